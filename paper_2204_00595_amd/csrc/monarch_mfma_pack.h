// Re-layout of the weights of the four-block layers in the fragment order of the packed-weight forward kernels
// (monarch_mfma_fwd_frag.hip): one thread builds one 16-byte piece.
//   RF1[kk][t][jt][lane][e] = R[kk][32*jt + lane%32][16*t + 8*(lane/32) + e]
//   LF2[c][lt][ks][lane][e] = L[c][32*lt + lane%32][4*(4*ks + e%4) + 2*(lane/32) + e/4]
#pragma once
#include "monarch_mfma_common.h"

namespace monarch {

__device__ __forceinline__ void pack_fwd_piece(const uint16_t* __restrict__ R, const uint16_t* __restrict__ L, uint16_t* __restrict__ RF1,
                                               uint16_t* __restrict__ LF2, int P, int Q, int S, int pc)
{
    const int nR = 4 * Q * P / 8, nL = 4 * S * Q / 8;  // 16-byte pieces per array
    if (pc < nR) {
        const int lane = pc & 63;
        int rest = pc >> 6;
        const int QT = Q / 32, T = P / 16;
        const int jt = rest % QT; rest /= QT;
        const int t = rest % T;
        const int kk = rest / T;
        const uint16_t* src = R + ((size_t)kk * Q + 32 * jt + (lane & 31)) * P + 16 * t + 8 * (lane >> 5);
        *reinterpret_cast<u32x4*>(RF1 + (size_t)pc * 8) = *reinterpret_cast<const u32x4*>(src);
    } else if (pc < nR + nL) {
        pc -= nR;
        const int lane = pc & 63;
        int rest = pc >> 6;
        const int KS = Q / 16, NLT = S / 32;
        const int ks = rest % KS; rest /= KS;
        const int lt = rest % NLT;
        const int c = rest / NLT;
        const int g = lane >> 5;
        const uint16_t* src = L + ((size_t)c * S + 32 * lt + (lane & 31)) * Q + 16 * ks;
        uint16_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = src[4 * (e & 3) + 2 * g + (e >> 2)];
        u32x4 o;
#pragma unroll
        for (int w = 0; w < 4; ++w) o[w] = (uint32_t)v[2 * w] | ((uint32_t)v[2 * w + 1] << 16);
        *reinterpret_cast<u32x4*>(LF2 + (size_t)pc * 8) = o;
    }
}

}  // namespace monarch
