// fp32 products on the bf16 matrix cores: an operand as three bf16 planes that add up to it.
#pragma once
#include "monarch_mfma_common.h"

namespace monarch {

// Operands are scaled up before they are split: every bit of an fp32 number, the denormal ones too, is then a multiple
// of 2^-125, so that each plane is a normal bf16 number or zero and nothing is lost at the lower end, whatever the
// other operand.  Numbers from 2^104 and results from 2^80 on become infinite, which the finished tile shows
// (planes_overflowed).
constexpr float kPlaneScale = 0x1p24f;
template <int SPLIT>  // operands that were split: 1 or 2
constexpr float kPlaneUnscale = SPLIT == 2 ? 0x1p-48f : 0x1p-24f;

// fp32 pair -> its three bf16 pairs: the (scaled) value rounded, what that leaves rounded, and the rest, which fits.
// The three add up to the value exactly.
__device__ __forceinline__ void split3(uint32_t a, uint32_t b, uint32_t out[3])
{
    float x = __uint_as_float(a) * kPlaneScale, y = __uint_as_float(b) * kPlaneScale;
#pragma unroll
    for (int w = 0; w < 3; ++w) {
        out[w] = pack_bf16x2(x, y);
        if (w < 2) {
            x -= __uint_as_float(out[w] << 16);
            y -= __uint_as_float(out[w] & 0xffff0000u);
        }
    }
}

// Products of the planes whose place values add up to less than 3; what the others add up to is at most 2^-24 of the
// product (2^-27.5 root mean square, where one rounding to fp32 is 2^-25.3).  `big` takes the product of the first
// planes, `small` the rest (they may be one).
template <int PA, int PB>
__device__ __forceinline__ void plane_products(const bf16x8 (&a)[PA], const bf16x8 (&b)[PB], f32x16& big, f32x16& small)
{
#pragma unroll
    for (int w = 2; w > 0; --w)
#pragma unroll
        for (int u = 0; u <= w; ++u)
            if (u < PA && w - u < PB) small = mfma32(a[u < PA ? u : 0], b[w - u < PB ? w - u : 0], small);
    big = mfma32(a[0], b[0], big);
}

// A result that is not finite: an infinity or NaN among the operands (an infinity times the zero planes of a number is
// no number), or something that the scale made infinite.
__device__ __forceinline__ bool planes_bad(float v) { return (__float_as_uint(v) << 1) >= (255u << 24); }

// Whether a lane of the wave holds one.  What is computed again then has to be chosen by rows of the batch: a row's
// result must not depend on the rows beside it.
template <int MT, int NT>
__device__ __forceinline__ bool planes_overflowed(const f32x16 (&acc)[MT][NT])
{
    uint32_t worst = 0;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t t = __float_as_uint(acc[i][j][r]) << 1;
                worst = t > worst ? t : worst;
            }
    return __any(worst >= (255u << 24));
}
template <int NT>
__device__ __forceinline__ bool planes_overflowed(const f32x16 (&acc)[NT])
{
    return planes_overflowed(reinterpret_cast<const f32x16(&)[1][NT]>(acc));
}
__device__ __forceinline__ bool planes_overflowed(const f32x16& acc)
{
    return planes_overflowed(reinterpret_cast<const f32x16(&)[1][1]>(acc));
}

// Tiles with a column (lane % 32) for each row of the batch: the results of the rows that hold something not finite
// become zero, for fp32 products to be added to them.  True in the lanes of these rows; the others keep their results
// and add products with zero.
__device__ __forceinline__ bool planes_clear(f32x16& acc)
{
    bool off = false;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float v = acc[r];
        off |= planes_bad(v);
    }
    const uint64_t m = __ballot(off);
    off = ((uint32_t)m | (uint32_t)(m >> 32)) >> (__lane_id() & 31) & 1;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float v = acc[r];
        acc[r] = off ? 0.f : v;
    }
    return off;
}

}  // namespace monarch
