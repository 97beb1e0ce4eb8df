// fp32 products on the bf16 matrix cores: an operand as three bf16 planes that add up to it.
#pragma once
#include "monarch_mfma_common.h"

namespace monarch {

// fp32 pair -> its three bf16 pairs: the value rounded, what that leaves rounded, and the rest, which fits.  The three add up to
// the value exactly, except where the last one is below bf16's smallest number (values below 2^-110) or the value is not finite.
__device__ __forceinline__ void split3(uint32_t a, uint32_t b, uint32_t out[3])
{
    float x = __uint_as_float(a), y = __uint_as_float(b);
#pragma unroll
    for (int w = 0; w < 3; ++w) {
        out[w] = pack_bf16x2(x, y);
        if (w < 2) {
            x -= __uint_as_float(out[w] << 16);
            y -= __uint_as_float(out[w] & 0xffff0000u);
        }
    }
}

// Products of the planes whose place values add up to less than 3; the others are below 2^-26 of the whole.  `big` takes the
// product of the first planes, `small` the rest (they may be one).
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

// Results of the split planes that are not what the fp32 matrix cores give: a value that is not finite (an infinity times the zero
// planes of a number is no number) and one so small that planes below bf16's smallest number may have been lost.  Exact zeros
// are right.  True if any lane of the wave holds such a value.
template <int MT, int NT>
__device__ __forceinline__ bool planes_doubtful(const f32x16 (&acc)[MT][NT])
{
    constexpr uint32_t kSmall = (127u - 80u) << 24, kWidth = (255u << 24) - kSmall;  // twice the bits of 2^-80, and from there to infinity
    uint32_t worst = 0;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t t = (__float_as_uint(acc[i][j][r]) << 1) - kSmall;
                worst = t > worst ? t : worst;
            }
    if (!__any(worst >= kWidth)) return false;
    bool off = false;  // most often these are the zeros of a ragged tile
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t t = __float_as_uint(acc[i][j][r]) << 1;
                off |= t != 0 && t - kSmall >= kWidth;
            }
    return __any(off);
}

__device__ __forceinline__ bool planes_doubtful(const f32x16& acc)
{
    return planes_doubtful(reinterpret_cast<const f32x16(&)[1][1]>(acc));
}
template <int NT>
__device__ __forceinline__ bool planes_doubtful(const f32x16 (&acc)[NT])
{
    return planes_doubtful(reinterpret_cast<const f32x16(&)[1][NT]>(acc));
}

}  // namespace monarch
