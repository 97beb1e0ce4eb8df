// The nonlinearity between the two linear layers of a feed-forward block, for the kernels that apply
// it in their epilogues.  The paper keeps the blocks of ViT / MLP-Mixer / BERT / GPT-2 as they are
// around the Monarch layers (Section 4) and does not write the nonlinearity down; those models use
// GELU, and this is the tanh form (GPT-2's):
//
//     gelu(v) = v/2 * (1 + tanh(u)) = v * s,   s = 1 / (1 + exp(-2u)),   u = sqrt(2/pi) * (v + 0.044715 v^3)
//     gelu'(v) = s + v * s * (1 - s) * d(2u)/dv
//
// fp32 throughout.  exp(-2u) is one v_exp_f32 (base 2, log2(e) folded into the polynomial).  From |v| = 16 on it is
// infinite or zero whatever the polynomial overflows to, so that s is exactly 0 or 1; in the gradient v is held to
// [-16, 16] (one v_med3_f32), or s (1 - s) = 0 would meet an infinite d(2u)/dv.  s (1 - s) stays two operations: as s
// - s s in one the last bit moves, and with it bf16 roundings of everything behind the gradient (1.7e-4 of the norm
// of a feed-forward block's).  In the epilogues that apply these, the vector units are what bounds them: in a loop of
// nothing else a value of gelu takes 39 clocks of a wave (47 with v clamped by maximum and minimum), of the gradient
// 59 (63).
#pragma once
#include <hip/hip_runtime.h>

namespace monarch {

// s(v) = 1/2 (1 + tanh u(v))
__device__ __forceinline__ float gelu_gate(float v)
{
    // -2u * log2(e) = v * (a + b v^2):  a = -2 sqrt(2/pi) log2(e),  b = a * 0.044715
    const float w = v * __builtin_fmaf(-0.10294324f, v * v, -2.3022082f);
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(w));
}

__device__ __forceinline__ float gelu_f(float v) { return v * gelu_gate(v); }

__device__ __forceinline__ float gelu_grad_f(float v)
{
    const float vc = __builtin_amdgcn_fmed3f(v, -16.f, 16.f);
    const float s = gelu_gate(vc);
    // d(2u)/dv = 2 sqrt(2/pi) (1 + 3 * 0.044715 v^2)
    return __builtin_fmaf(vc * (s * (1.0f - s)), __builtin_fmaf(0.21406445f, vc * vc, 1.5957692f), s);
}

}  // namespace monarch
