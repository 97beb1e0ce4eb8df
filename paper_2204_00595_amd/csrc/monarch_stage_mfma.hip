// Complex-valued Monarch multiply on the matrix cores (complex64, fp32 arithmetic), for square blocks
// p = q = s, a multiple of 8 from 16 to 64, and any k.  The paper's results hold over C (Notation Review); the steps
// are those of Section 3.3 with the permutations of Definition 3.1, the gradients those of monarch_complex.hip.
//
// A complex product is a real product of twice the size: with a vector stored as interleaved (re, im) pairs,
// y = W x over C is  y' = W' x'  over R, where W'[2j+e][2i+t] = (Wr, -Wi; Wi, Wr)[e][t].  The activations are
// therefore used exactly as they lie in memory, and the weights are expanded as they are loaded.
//
// One block-diagonal factor is one launch ("stage"), and the vector between the two factors goes through a
// workspace: at n = 4096 a row of it takes 32 KiB, so a 32-row tile does not fit LDS next to anything else.  A
// workgroup owns one block g and a share of the row tiles: its wave w keeps the expanded weights of 16 outputs
// (32 real rows, the M extent of the MFMA) in registers for the whole launch and streams 32-row
// activation tiles (the N extent) past them.
//   D (32 x 32): acc[r] = D[8*(r/4) + 4*(lane/32) + r%4][lane%32]: a lane holds whole complex outputs of one row.
//
// The products run on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16), both operands as three bf16 planes that add up
// to the fp32 values (monarch_planes.h): weights when they are loaded, activations on their way to LDS or, where a wave
// takes them from memory itself, in its registers.  A step contracts eight complex inputs with six MFMAs in place of
// sixteen fp32 MFMAs of twice the cycles.
// Rows with results that are not finite are computed again in fp32 (stage_finish; an infinity in one of every 32 rows,
// 64 complex blocks of 64, 2048 rows: forward 73 -> 210 us, backward 223 -> 525; 64 real blocks of 64, 12000 rows: 191
// -> 405 and 557 -> 2467).
// On the fp32 cores the contiguous stages took 54 us at 64 blocks of 64 and 2048 rows and were bound by them (69 to 74
// % busy); they take 37 to 40 now, for 134 MB each, 26 us at the rate of a copy.  What is left is one tile per
// workgroup in flight: the weights' planes take 96 registers, so two workgroups fit a CU.
// A second tile in flight took a workgroup's registers to the limit and 6 us more, a third workgroup spilled (62 us).
// Forward and backward together: 64 blocks of 64, 2048 rows: 389 -> 300 us; 48, 1500 rows: 212 -> 159; 32, 2048 rows:
// 103 -> 85; 64 real blocks of 64, 12000 rows: 895 -> 730.
//
// The permutation between the factors is an 8-byte transposition, so it is done where the pieces can be made
// long: the workspace holds the intermediate in tiles  T[row tile][block][index in block][32 rows]  (the
// producer writes, per output index, the 32 rows of its tile as one 256-byte run into the block the consumer
// will read; the consumer's tile is then one contiguous block).  Only the outer permutation (y[b][l*k + c], and
// dy read the same way) moves 8-byte pieces; the workgroups of one row range run on one XCD so that these meet in
// one L2.
//
// Weight gradients: dL[c] = dW[c]^T conj(U[c]),  dR[kk] = dY1[kk]^T conj(x[kk]),  contracted over the batch by the
// same MFMA (K = eight rows x two components), in the launch that computes the gradient of the factor's input
// (cboth_kernel); a workgroup owns one block and a share of the row tiles, the shares' partial results go to the
// workspace and are summed in a fixed order (no atomics).
//
// Real fp32 layers with square blocks of 32 or 64 run on the same kernels (template flag REAL): a float2 is then two
// consecutive values of a row, the activation side is unchanged, the weights are taken as stored and the
// permutations move single values (see cstage_kernel).
#include <type_traits>
#include "monarch_internal.h"
#include "monarch_device.h"
#include "monarch_mfma_common.h"
#include "monarch_planes.h"

namespace monarch {
namespace {

constexpr int kRT = 32;  // batch rows per tile
template <int Q>
constexpr int kTileWaves = (Q + 15) / 16;  // M tiles (16 outputs) of a block

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

enum : int { kInNat = 0, kInGather = 1, kInT = 2 };
enum : int { kOutTFwd = 0, kOutTBwd = 1, kOutNat = 2, kOutScatter = 3 };

// stage-1 output f = kk*q + j that lands at position g of the permuted vector (inverse of mid_dest)
__device__ __forceinline__ int mid_src(int g, int k, int q, bool perm_b)
{
    if (!perm_b) { const int j = g / k, kk = g - j * k; return kk * q + j; }
    const int c = g / q, r = g - c * q;
    return r * k + c;
}

// Element i of row `row` of a 32-row tile straight from memory, as the tiles below take it (zero past the end of the
// batch).
template <int P, int IN, bool REAL>
__device__ __forceinline__ float2 act_value(const float2* __restrict__ src, int64_t rt, int row, int g, int i, int k, int64_t ld, int64_t B)
{
    if constexpr (IN == kInT) return src[(((size_t)rt * k + g) * P + i) * kRT + row];
    const int64_t at = rt * kRT + row, r = at < B ? at : B - 1;
    float2 v;
    if constexpr (IN == kInNat) {
        v = src[r * ld + (size_t)g * P + i];
    } else if constexpr (!REAL) {
        v = src[r * ld + (size_t)i * k + g];
    } else {
        const float* f = reinterpret_cast<const float*>(src) + r * (2 * ld) + g;
        v = make_float2(f[(size_t)(2 * i) * k], f[(size_t)(2 * i + 1) * k]);
    }
    return at < B ? v : make_float2(0.f, 0.f);
}

// What lane (col, e = lane % 2) of the wave that owns M tile mt multiplies with input i of block g: its row of the
// expanded weights at the two components.  CONJT: the conjugate transpose of the stored block; REAL: the weights as
// they are (CONJT: transposed).
template <int P, int Q, bool CONJT, bool REAL>
__device__ __forceinline__ float2 weight_value(const float2* __restrict__ W, int g, int mt, int col, int i)
{
    if constexpr (REAL) {
        const float* Wf = reinterpret_cast<const float*>(W) + (size_t)g * (4 * P * Q);
        const int nw = 32 * mt + col;
        if constexpr (CONJT) return make_float2(Wf[(size_t)(2 * i) * (2 * Q) + nw], Wf[(size_t)(2 * i + 1) * (2 * Q) + nw]);
        return *reinterpret_cast<const float2*>(Wf + (size_t)nw * (2 * P) + 2 * i);
    } else {
        const int e = col & 1;
        int jw = 16 * mt + (col >> 1);
        if (Q % 16 != 0 && jw >= Q) jw = Q - 1;  // an output that does not exist
        const float2* Wg = W + (size_t)g * P * Q;
        constexpr float sgn = CONJT ? -1.f : 1.f;
        const float2 w = CONJT ? Wg[i * Q + jw] : Wg[jw * P + i];
        return make_float2(e ? sgn * w.y : w.x, e ? w.x : -sgn * w.y);
    }
}

// A lane's weights of an M tile as planes: step t contracts the inputs 8 t + 4 (lane / 32) .. + 3.
template <int P, int Q, bool CONJT, bool REAL>
__device__ __forceinline__ void load_weights(bf16x8 (&A)[P / 8][3], const float2* __restrict__ W, int g, int mt, int col, int kh)
{
#pragma unroll
    for (int t = 0; t < P / 8; ++t) {
        uint32_t w[4][3];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float2 v = weight_value<P, Q, CONJT, REAL>(W, g, mt, col, 8 * t + 4 * kh + c);
            split3(__float_as_uint(v.x), __float_as_uint(v.y), w[c]);
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) A[t][u] = as_bf16x8(u32x4{w[0][u], w[1][u], w[2][u], w[3][u]});
    }
}
// four complex values (REAL: pairs) -> planes
__device__ __forceinline__ void split_four(const float2 (&v)[4], bf16x8 (&b)[3])
{
    uint32_t w[4][3];
#pragma unroll
    for (int c = 0; c < 4; ++c) split3(__float_as_uint(v[c].x), __float_as_uint(v[c].y), w[c]);
#pragma unroll
    for (int u = 0; u < 3; ++u) b[u] = as_bf16x8(u32x4{w[0][u], w[1][u], w[2][u], w[3][u]});
}

// A finished tile: the planes' scale comes off, and rows with something not finite are computed again in fp32.
template <int P, int Q, int IN, bool CONJT, bool REAL>
__device__ __forceinline__ void stage_finish(f32x16& acc, const float2* __restrict__ in, const float2* __restrict__ W, int64_t rt, int g, int mt,
                                             int k, int64_t ld, int64_t B, int lane)
{
    const bool off = planes_overflowed(acc);
    acc *= kPlaneUnscale<2>;
    if (!off) return;
    const bool mine = planes_clear(acc);
    const int col = lane & 31, kh = lane >> 5;
    constexpr int U = P >= 48 ? 1 : 2;  // what the weights leave room for
#pragma clang loop unroll(disable)
    for (int u0 = 0; u0 < P / 2; u0 += U) {
        float2 w[U], x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            w[u] = weight_value<P, Q, CONJT, REAL>(W, g, mt, col, 2 * (u0 + u) + kh);
            x[u] = act_value<P, IN, REAL>(in, rt, col, g, 2 * (u0 + u) + kh, k, ld, B);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc = mfma_f32(w[u].x, mine ? x[u].x : 0.f, acc);
            acc = mfma_f32(w[u].y, mine ? x[u].y : 0.f, acc);
        }
    }
}

// A 32-row tile of one block's complex values, P per row, fetched into registers and later written to LDS.
//   kInNat:    src[row][g*P + i]
//   kInGather: src[row][i*k + g]
//   kInT:      src tile (rt, g): [i][32 rows], contiguous
// LDS: three bf16 planes (monarch_planes.h) of [row][2 P + 8], a row's components in order; the 16 bytes of padding
// make a row an odd number of 16-byte units, so that eight rows' pieces fall on different banks.  Rows past the end of
// the batch read as zeros (kInT: the producer wrote zeros there).
// REAL (real fp32 data, two consecutive values per float2): only the gathering form differs, whose pieces are then
// single floats, src[row][i'*k + g] for the 2P real indices i' of the block.
template <int P, int NTHR, int IN, bool REAL = false>
struct ActTile {
    static constexpr int kAll = (IN == kInGather) ? kRT * P : kRT * P / 2;
    static constexpr int kPieces = (kAll + NTHR - 1) / NTHR;  // per thread
    static __device__ __forceinline__ bool has(int idx) { return kAll % NTHR == 0 || idx < kAll; }
    static constexpr int kStride = 2 * P + 8, kPlane = kRT * kStride, kLen = 3 * kPlane;  // bf16 values
    static_assert(!REAL || kAll % NTHR == 0, "tile does not divide over the threads");
    u32x4 v[IN == kInGather ? (kPieces + 1) / 2 : kPieces];

    __device__ __forceinline__ void fetch(const float2* __restrict__ src, int64_t rt, int g, int k, int64_t ld, int64_t B, int tid)
    {
        const int64_t row0 = rt * kRT;
        if constexpr (IN == kInNat) {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / (P / 2), c2 = idx - row * (P / 2);
                v[n] = (has(idx) && row0 + row < B) ? ldg128(src + (row0 + row) * ld + (size_t)g * P + 2 * c2) : u32x4{0, 0, 0, 0};
            }
        } else if constexpr (IN == kInGather && REAL) {
            const float* srcf = reinterpret_cast<const float*>(src);
#pragma unroll
            for (int n = 0; n < 2 * kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / (2 * P), i = idx - row * (2 * P);
                float t = 0.f;
                if (row0 + row < B) t = srcf[(row0 + row) * (2 * ld) + (size_t)i * k + g];
                v[n / 4][n % 4] = __float_as_uint(t);
            }
        } else if constexpr (IN == kInGather) {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / P, i = idx - row * P;
                float2 t = make_float2(0.f, 0.f);
                if (has(idx) && row0 + row < B) t = src[(row0 + row) * ld + (size_t)i * k + g];
                if (n & 1) { v[n / 2].z = __float_as_uint(t.x); v[n / 2].w = __float_as_uint(t.y); }
                else { v[n / 2].x = __float_as_uint(t.x); v[n / 2].y = __float_as_uint(t.y); }
            }
        } else {
            const float2* tile = src + ((size_t)rt * k + g) * (P * kRT);
#pragma unroll
            for (int n = 0; n < kPieces; ++n)
                if (has(tid + n * NTHR)) v[n] = ldg128(tile + 2 * (tid + n * NTHR));
        }
    }

    __device__ __forceinline__ void to_lds(bf16_t* act, int tid) const
    {
        if constexpr (IN == kInNat) {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / (P / 2), c2 = idx - row * (P / 2);
                uint32_t a[3], b[3];
                split3(v[n].x, v[n].y, a);
                split3(v[n].z, v[n].w, b);
                if (!has(idx)) continue;
#pragma unroll
                for (int u = 0; u < 3; ++u) *reinterpret_cast<u32x2*>(act + u * kPlane + row * kStride + 4 * c2) = u32x2{a[u], b[u]};
            }
        } else if constexpr (IN == kInGather && REAL) {
#pragma unroll
            for (int n = 0; n < 2 * kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / (2 * P), i = idx - row * (2 * P);
                uint32_t a[3];
                split3(v[n / 4][n % 4], 0u, a);
#pragma unroll
                for (int u = 0; u < 3; ++u) act[u * kPlane + row * kStride + i] = (bf16_t)a[u];
            }
        } else if constexpr (IN == kInGather) {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / P, i = idx - row * P;
                const u32x4 w = v[n / 2];
                uint32_t a[3];
                if (n & 1) split3(w.z, w.w, a);
                else split3(w.x, w.y, a);
                if (!has(idx)) continue;
#pragma unroll
                for (int u = 0; u < 3; ++u) *reinterpret_cast<uint32_t*>(act + u * kPlane + row * kStride + 2 * i) = a[u];
            }
        } else {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, i = idx / (kRT / 2), row = 2 * (idx - i * (kRT / 2));
                uint32_t a[3], b[3];
                split3(v[n].x, v[n].y, a);
                split3(v[n].z, v[n].w, b);
                if (!has(idx)) continue;
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    *reinterpret_cast<uint32_t*>(act + u * kPlane + row * kStride + 2 * i) = a[u];
                    *reinterpret_cast<uint32_t*>(act + u * kPlane + (row + 1) * kStride + 2 * i) = b[u];
                }
            }
        }
    }

    // The tile in both orders at once, the one above and that of a weight-gradient operand (WgTile).
    template <typename TW>
    __device__ __forceinline__ void to_both(bf16_t* act, bf16_t* wg, int tid) const
    {
        constexpr int WS = TW::kStride, WP = TW::kPlane;
        if constexpr (IN == kInGather && REAL) {
#pragma unroll
            for (int n = 0; n < 2 * kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / (2 * P), i = idx - row * (2 * P);
                uint32_t a[3];
                split3(v[n / 4][n % 4], 0u, a);
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    act[u * kPlane + row * kStride + i] = (bf16_t)a[u];
                    wg[u * WP + i * WS + row] = (bf16_t)a[u];
                }
            }
        } else if constexpr (IN == kInGather) {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / P, i = idx - row * P;
                const u32x4 w = v[n / 2];
                uint32_t a[3];
                if (n & 1) split3(w.z, w.w, a);
                else split3(w.x, w.y, a);
                if (!has(idx)) continue;
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    *reinterpret_cast<uint32_t*>(act + u * kPlane + row * kStride + 2 * i) = a[u];
                    *reinterpret_cast<uint32_t*>(wg + u * WP + i * WS + 2 * row) = a[u];
                }
            }
        } else {
            static_assert(IN == kInT, "rows in their natural order are no operand of both");
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, i = idx / (kRT / 2), row = 2 * (idx - i * (kRT / 2));
                uint32_t a[3], b[3];
                split3(v[n].x, v[n].y, a);
                split3(v[n].z, v[n].w, b);
                if (!has(idx)) continue;
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    *reinterpret_cast<uint32_t*>(act + u * kPlane + row * kStride + 2 * i) = a[u];
                    *reinterpret_cast<uint32_t*>(act + u * kPlane + (row + 1) * kStride + 2 * i) = b[u];
                    if constexpr (REAL) {
                        *reinterpret_cast<uint32_t*>(wg + u * WP + 2 * i * WS + row) = pick_lo16(a[u], b[u]);
                        *reinterpret_cast<uint32_t*>(wg + u * WP + (2 * i + 1) * WS + row) = pick_hi16(a[u], b[u]);
                    } else {
                        *reinterpret_cast<u32x2*>(wg + u * WP + i * WS + 2 * row) = u32x2{a[u], b[u]};
                    }
                }
            }
        }
    }

    // the MFMA operand of step t: lane (row, h) the components 16 t + 8 h ..
    static __device__ __forceinline__ void read(bf16x8 (&b)[3], const bf16_t* act, int t, int lane)
    {
#pragma unroll
        for (int u = 0; u < 3; ++u) b[u] = as_bf16x8(lds128(act + u * kPlane + (lane & 31) * kStride + 16 * t + 8 * (lane >> 5)));
    }
};

// Where a lane's results go within a tile of the workspace (kOutTFwd, kOutTBwd): 32-bit byte offsets, which leave
// cstage_kernel room for a third workgroup.
template <int Q, int OUT, bool REAL>
struct TiledOut {
    static constexpr bool kTiled = OUT == kOutTFwd || OUT == kOutTBwd, kWhole = Q % 16 == 0;
    static constexpr int kOuts = kTiled ? (REAL ? 16 : 8) : 1;
    uint32_t off[kOuts];
    __device__ __forceinline__ void init(int g, int mt, int kh, int col, int k, bool pb)
    {
        if constexpr (!kTiled) return;
#pragma unroll
        for (int o = 0; o < kOuts; ++o) {
            constexpr int E = REAL ? 2 : 1;  // values per float2 of the output
            const int j = 16 * mt + 4 * (o / (2 * E)) + 2 * kh + o / E % 2, n = E * j + o % E;
            const int d = (OUT == kOutTFwd) ? mid_dest(g * E * Q + n, k, E * Q, pb) : mid_src(g * E * Q + n, k, E * Q, pb);
            const int blk = d / (E * Q), idx = d - blk * (E * Q);
            off[o] = (uint32_t)(((blk * Q + idx / E) * kRT + col) * E + idx % E) * (uint32_t)(8 / E);
        }
    }
    __device__ __forceinline__ void store(float2* __restrict__ out, const f32x16& acc, int64_t rt, int mt, int kh, int k) const
    {
        char* const to = reinterpret_cast<char*>(out + (size_t)rt * k * (Q * kRT));
#pragma unroll
        for (int o = 0; o < kOuts; ++o) {
            if (!kWhole && 16 * mt + 4 * (o / 2) + 2 * kh + o % 2 >= Q) continue;
            if constexpr (REAL) *reinterpret_cast<float*>(to + off[o]) = acc[o];
            else *reinterpret_cast<float2*>(to + off[o]) = make_float2(acc[2 * o], acc[2 * o + 1]);
        }
    }
};
// kOutNat: a tile's results through LDS [row][Q + 1], then out in whole rows
template <int Q, int NTHR>
struct NatOut {
    static constexpr int kStride = Q + 1, kLen = kRT * kStride;  // float2
    static __device__ __forceinline__ void put(float2* ost, const f32x16& acc, int mt, int kh, int col)
    {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (Q % 16 == 0 || 16 * mt + 4 * q4 + 2 * kh + h < Q)
                    ost[col * kStride + 16 * mt + 4 * q4 + 2 * kh + h] = make_float2(acc[4 * q4 + 2 * h], acc[4 * q4 + 2 * h + 1]);
    }
    static __device__ __forceinline__ void emit(const float2* ost, float2* __restrict__ out, int64_t rt, int g, int64_t ld, int64_t B, int tid)
    {
        constexpr int kAll = kRT * Q / 2, kPieces = (kAll + NTHR - 1) / NTHR;
#pragma unroll
        for (int n = 0; n < kPieces; ++n) {
            const int idx = tid + n * NTHR, r = idx / (Q / 2), c2 = idx - r * (Q / 2);
            if (kAll % NTHR != 0 && idx >= kAll) continue;
            const float2 v0 = ost[r * kStride + 2 * c2], v1 = ost[r * kStride + 2 * c2 + 1];
            if (rt * kRT + r < B)
                *reinterpret_cast<f32x4*>(out + (rt * kRT + r) * ld + (size_t)g * Q + 2 * c2) = f32x4{v0.x, v0.y, v1.x, v1.y};
        }
    }
};

// out[b][block g][n] = sum_m in[b][block g][m] * Wop[g][n][m],  n < Q, m < P;
// Wop[n][m] = W[g][n][m] (W stored [g][Q][P]) or, CONJT, conj(W[g][m][n]) (W stored [g][P][Q]).
//   kOutTFwd:    element (g, n) is stage-1 output f = g*Q + n; it goes to block c, index r of the permuted vector
//   kOutTBwd:    element (g, n) is position g*Q + n of the permuted vector; it goes to block kk, index j of stage 1
//   kOutNat:     out[row][g*Q + n]
//   kOutScatter: out[row][n*k + g], REAL: plus bias[n*k + g] where there is one
// Grid: k * nsplit workgroups of Q/16 waves; workgroup (g, split) takes the row tiles split, split + nsplit, ...
// (split = blockIdx % nsplit with nsplit a multiple of 8 keeps the blocks of one row range on one XCD).
// REAL: real fp32 data and weights, block sizes 2P -> 2Q.  A float2 is then two consecutive values of a row, which
// is what one pair of K = 2 steps contracts, so the activation side is unchanged; the weights are used as they are
// (CONJT: transposed), and since the permutations move single values, the two values of a result pair go to their
// places separately (in the tiled workspace, to the pair slot [index / 2][row][index % 2] of the consumer's block).
template <int P, int Q, int IN, int OUT, bool CONJT, bool REAL = false>
__global__ void __launch_bounds__(kTileWaves<Q> * 64, P >= 56 || IN == kInGather ? 2 : 3)
cstage_kernel(const float2* __restrict__ in, const float2* __restrict__ W, const float* __restrict__ bias, float2* __restrict__ out,
              int64_t B, int k, int nsplit, int perm_b)
{
    constexpr int NTHR = kTileWaves<Q> * 64;
    constexpr bool kWhole = Q % 16 == 0;  // else the last wave has outputs that do not exist
    using Tile = ActTile<P, NTHR, IN, REAL>;
    using Nat = NatOut<Q, NTHR>;
    // kOutNat: the barrier before the results leave LDS also frees the tile, so one buffer will do
    constexpr int kBufs = OUT == kOutNat ? 1 : 2;
    __shared__ __align__(16) bf16_t act[kBufs][Tile::kLen];
    __shared__ __align__(16) float2 ost[OUT == kOutNat ? Nat::kLen : 1];

    const int g = (int)blockIdx.x / nsplit, split = (int)blockIdx.x - g * nsplit;
    const int tid = threadIdx.x, lane = tid & 63, mt = tid >> 6;
    const int col = lane & 31, kh = lane >> 5;
    const int64_t ntiles = (B + kRT - 1) / kRT;
    const int64_t ld_in = (int64_t)k * P, ld_out = (int64_t)k * Q;
    const bool pb = perm_b != 0;

    bf16x8 A[P / 8][3];
    load_weights<P, Q, CONJT, REAL>(A, W, g, mt, col, kh);

    using Tiled = TiledOut<Q, OUT, REAL>;
    Tiled tiled;
    tiled.init(g, mt, kh, col, k, pb);

    Tile pre;
    int64_t rt = split;
    if (rt < ntiles) pre.fetch(in, rt, g, k, ld_in, B, tid);
    for (int it = 0; rt < ntiles; rt += nsplit, ++it) {
        bf16_t* a = act[kBufs == 2 ? it & 1 : 0];
        pre.to_lds(a, tid);
        lds_barrier();
        if (rt + nsplit < ntiles) pre.fetch(in, rt + nsplit, g, k, ld_in, B, tid);

        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int t = 0; t < P / 8; ++t) {
            bf16x8 xv[3];
            Tile::read(xv, a, t, lane);
            plane_products<3, 3>(A[t], xv, acc, acc);
        }
        stage_finish<P, Q, IN, CONJT, REAL>(acc, in, W, rt, g, mt, k, ld_in, B, lane);

        const int64_t row = rt * kRT + col;
        if constexpr (OUT == kOutNat) {
            Nat::put(ost, acc, mt, kh, col);
            lds_barrier();
            Nat::emit(ost, out, rt, g, ld_out, B, tid);
        } else if constexpr (Tiled::kTiled) {
            tiled.store(out, acc, rt, mt, kh, k);
        } else {
#pragma unroll
            for (int o = 0; o < 8; ++o) {
                const int j = 16 * mt + 4 * (o / 2) + 2 * kh + o % 2;
                if (!kWhole && j >= Q) continue;
                if (row >= B) continue;
                if constexpr (REAL) {
                    float* outf = reinterpret_cast<float*>(out) + row * (2 * ld_out) + g;
                    const int n0 = 2 * j * k, n1 = n0 + k;
                    outf[n0] = bias ? acc[2 * o] + bias[g + n0] : acc[2 * o];
                    outf[n1] = bias ? acc[2 * o + 1] + bias[g + n1] : acc[2 * o + 1];
                } else {
                    out[row * ld_out + (size_t)j * k + g] = make_float2(acc[2 * o], acc[2 * o + 1]);
                }
            }
        }
    }
}

// The two stages that touch the outer permutation (y[b][l*k + c] written, dy read the same way), for k a multiple
// of 8: eight blocks per workgroup, wave w = block 8*oct + w, every wave the same M tile (16 outputs) of its
// own block, so that the pieces of the permuted side are the eight blocks' values of one (row, l): 64 contiguous bytes
// instead of 8.  Workgroups that differ only in their M tile read the same activations (they sit on one XCD) and
// split them again, which costs less than the registers of a second M tile.
//
// cscatter8_kernel: tiled workspace -> y.  The activations of a wave's block are MFMA operands exactly as they lie
// in the workspace (lane = row, 512 contiguous bytes per wave load), so they go from global memory to registers
// directly, ahead of the MFMAs; the results are exchanged through LDS as [row][l][block].
template <int P, int Q>
struct Scatter8 {
    static constexpr int kRow = 16 * 8 + 1;  // values per row of the exchange buffer
    static constexpr size_t kLds = 2 * (size_t)kRT * kRow * sizeof(float2);
};

// REAL (see cstage_kernel): the pieces of y are the eight blocks' values of one (row, output), 32 bytes; a thread's are
// those of one output, so its four values of the bias stay in registers (training step, 64 blocks of 64 with a bias and
// without, us: 4000 rows 254.8 and 238.2, 16384 rows 912 and 842, what the bias's gradient takes; a pass over y of its
// own made that difference 40 and 185).
template <int P, int Q, bool REAL = false>
__global__ void __launch_bounds__(512)
cscatter8_kernel(const float2* __restrict__ T, const float2* __restrict__ W, const float* __restrict__ bias, float2* __restrict__ out,
                 int64_t B, int k, int nsplit)
{
    constexpr int MTG = kTileWaves<Q>;  // workgroups per (block octet, split)
    constexpr int STEPS = P / 8, NCH = STEPS >= 6 ? 2 : 1;  // pieces a tile's activations are fetched in
    constexpr int CH = (STEPS + NCH - 1) / NCH;              // steps of the first piece
    constexpr int OROW = Scatter8<P, Q>::kRow;
    extern __shared__ __align__(16) float2 ost8[];

    int bid = (int)blockIdx.x;
    const int split = bid % nsplit;
    bid /= nsplit;
    const int mt = bid % MTG, oct = bid / MTG;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int g = 8 * oct + w;
    const int col = lane & 31, kh = lane >> 5;
    const int64_t ntiles = (B + kRT - 1) / kRT;
    const int64_t ld_out = (int64_t)k * Q;

    bf16x8 A[STEPS][3];
    load_weights<P, Q, false, REAL>(A, W, g, mt, col, kh);
    auto load = [&](float2 (&buf)[CH][4], int64_t rt, int part) {
        const float2* src = T + ((size_t)rt * k + g) * (P * kRT) + (size_t)(8 * part * CH + 4 * kh) * kRT + col;
#pragma unroll
        for (int t = 0; t < CH; ++t)
            if (part * CH + t < STEPS) {
#pragma unroll
                for (int c = 0; c < 4; ++c) buf[t][c] = src[(8 * t + c) * kRT];
            }
    };
    f32x16 acc;
    auto zero = [&]() {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    };
    auto mma = [&](const float2 (&buf)[CH][4], auto which) {
        constexpr int part = decltype(which)::value;
#pragma unroll
        for (int t = 0; t < CH; ++t)
            if constexpr (part * CH < STEPS) {
                if (part * CH + t < STEPS) {
                    bf16x8 b[3];
                    split_four(buf[t], b);
                    plane_products<3, 3>(A[part * CH + t], b, acc, acc);
                }
            }
    };
    auto finish = [&](int64_t rt) { stage_finish<P, Q, kInT, false, REAL>(acc, T, W, rt, g, mt, k, 0, B, lane); };
    f32x4 bv = {0.f, 0.f, 0.f, 0.f};
    if constexpr (REAL) {
        if (bias) bv = *reinterpret_cast<const f32x4*>(bias + (size_t)(32 * mt + (tid >> 1 & 31)) * k + 8 * oct + 4 * (tid & 1));
    }
    // the results of one tile: exchange through LDS buffer it & 1 (one barrier per tile), then the 64-byte (REAL:
    // 32-byte) pieces of y
    auto emit = [&](int64_t rt, int it) {
        float2* o = ost8 + (it & 1) * (kRT * OROW);
        if constexpr (REAL) {
            // [row][32 outputs][8 blocks] floats in the same space; acc[r] is output 8*(r/4) + 4*kh + r%4
            float* of = reinterpret_cast<float*>(o);
#pragma unroll
            for (int r = 0; r < 16; ++r) of[col * (2 * OROW) + (8 * (r / 4) + 4 * kh + (r % 4)) * 8 + w] = acc[r];
            lds_barrier();
            float* outf = reinterpret_cast<float*>(out);
#pragma unroll
            for (int n = 0; n < 4; ++n) {  // 32 rows x 32 outputs x 2 halves of the eight blocks, 16 bytes each
                const int idx = tid + n * 512, part = idx & 1, nl = (idx >> 1) & 31, r = idx >> 6;
                const float2 v0 = *reinterpret_cast<const float2*>(of + r * (2 * OROW) + nl * 8 + 4 * part);
                const float2 v1 = *reinterpret_cast<const float2*>(of + r * (2 * OROW) + nl * 8 + 4 * part + 2);
                if (rt * kRT + r < B)
                    *reinterpret_cast<f32x4*>(outf + (rt * kRT + r) * (2 * ld_out) + (size_t)(32 * mt + nl) * k + 8 * oct + 4 * part) =
                        bias ? f32x4{v0.x + bv.x, v0.y + bv.y, v1.x + bv.z, v1.y + bv.w} : f32x4{v0.x, v0.y, v1.x, v1.y};
            }
        } else {
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    o[col * OROW + (4 * q4 + 2 * kh + h) * 8 + w] = make_float2(acc[4 * q4 + 2 * h], acc[4 * q4 + 2 * h + 1]);
            lds_barrier();
#pragma unroll
            for (int n = 0; n < 4; ++n) {  // 32 rows x 16 outputs x 4 pairs of blocks, 16 bytes each
                const int idx = tid + n * 512, c2 = idx & 3, ll = (idx >> 2) & 15, r = idx >> 6;
                const float2 v0 = o[r * OROW + ll * 8 + 2 * c2], v1 = o[r * OROW + ll * 8 + 2 * c2 + 1];
                if (rt * kRT + r < B && (Q % 16 == 0 || 16 * mt + ll < Q))
                    *reinterpret_cast<f32x4*>(out + (rt * kRT + r) * ld_out + (size_t)(16 * mt + ll) * k + 8 * oct + 2 * c2) =
                        f32x4{v0.x, v0.y, v1.x, v1.y};
            }
        }
    };

    // two register sets: the next piece of the activations (a whole tile, or half of one where the weights leave less
    // room) is on its way while the current one is multiplied
    typedef std::integral_constant<int, 0> First;
    typedef std::integral_constant<int, 1> Second;
    float2 xa[CH][4], xb[CH][4];
    int64_t rt = split;
    if (rt < ntiles) load(xa, rt, 0);
    if constexpr (NCH == 1) {
        for (int it = 0; rt < ntiles; it += 2) {
            if (rt + nsplit < ntiles) load(xb, rt + nsplit, 0);
            zero();
            mma(xa, First());
            finish(rt);
            emit(rt, it);
            rt += nsplit;
            if (rt >= ntiles) break;
            if (rt + nsplit < ntiles) load(xa, rt + nsplit, 0);
            zero();
            mma(xb, First());
            finish(rt);
            emit(rt, it + 1);
            rt += nsplit;
        }
    } else {
        for (int it = 0; rt < ntiles; rt += nsplit, ++it) {
            zero();
            load(xb, rt, 1);
            mma(xa, First());
            if (rt + nsplit < ntiles) load(xa, rt + nsplit, 0);
            mma(xb, Second());
            finish(rt);
            emit(rt, it);
        }
    }
}

// cgather8_kernel: dy (read through the outer permutation) -> tiled workspace, weights conj(L[c])^T.  The eight
// blocks' values of 32 rows x 16 inputs come in as 64-byte pieces and are laid out in LDS as one plane per block,
// [row][16 + 2]; a wave takes its operands from its own plane.  Four (P = 64) such chunks make a tile; the next
// chunk is fetched into registers while the current one is multiplied.
template <int P>
struct Gather8 {
    static constexpr int kPlane = kRT * 18 + 2;
    static constexpr size_t kLds = 2 * (size_t)8 * kPlane * sizeof(float2);
};

// REAL (see cstage_kernel): the pieces of dy are 32 bytes (eight blocks' values of one (row, input)), a chunk is
// 32 inputs = 16 pairs, and the weights are L[c]^T as stored.  MTW: M tiles of a wave (launch_gather8).
template <int P, int Q, bool REAL, int MTW>
__global__ void __launch_bounds__(512)
cgather8_kernel(const float2* __restrict__ in, const float2* __restrict__ W, float2* __restrict__ out,
                int64_t B, int k, int nsplit, int perm_b)
{
    constexpr int MTG = kTileWaves<Q> / MTW;
    constexpr int NCHUNK = (P + 15) / 16;
    constexpr int PLANE = Gather8<P>::kPlane;
    extern __shared__ __align__(16) float2 gat8[];

    int bid = (int)blockIdx.x;
    const int split = bid % nsplit;
    bid /= nsplit;
    const int mt0 = bid % MTG * MTW, oct = bid / MTG;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = 8 * oct + w;
    const int col = lane & 31, kh = lane >> 5;
    const int64_t ntiles = (B + kRT - 1) / kRT;
    const int64_t ld_in = (int64_t)k * P;
    const bool pb = perm_b != 0;

    bf16x8 A[MTW][P / 8][3];
#pragma unroll
    for (int m = 0; m < MTW; ++m) load_weights<P, Q, true, REAL>(A[m], W, g, mt0 + m, col, kh);
    constexpr int kOuts = REAL ? 16 : 8, E = REAL ? 2 : 1;  // as in cstage_kernel
    uint32_t off[MTW][kOuts];
#pragma unroll
    for (int o = 0; o < MTW * kOuts; ++o) {
        const int j = 16 * (mt0 + o / kOuts) + 4 * (o % kOuts / (2 * E)) + 2 * kh + o / E % 2;
        const int d = mid_src(g * E * Q + E * j + o % E, k, E * Q, pb), blk = d / (E * Q), idx = d - blk * (E * Q);
        off[o / kOuts][o % kOuts] = (uint32_t)(((blk * Q + idx / E) * kRT + col) * E + idx % E) * (uint32_t)(8 / E);
    }
    u32x4 pre[4];
    auto fetch = [&](int64_t rt, int ch) {
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int idx = tid + n * 512;
            const int64_t row = rt * kRT + (idx >> 6);
            if constexpr (REAL) {
                const int part = idx & 1, il = (idx >> 1) & 31;
                const float* srcf = reinterpret_cast<const float*>(in);
                pre[n] = row < B ? ldg128(srcf + row * (2 * ld_in) + (size_t)(32 * ch + il) * k + 8 * oct + 4 * part) : u32x4{0, 0, 0, 0};
            } else {
                const int c2 = idx & 3, ll = (idx >> 2) & 15;
                pre[n] = row < B && (P % 16 == 0 || 16 * ch + ll < P)
                             ? ldg128(in + row * ld_in + (size_t)(16 * ch + ll) * k + 8 * oct + 2 * c2) : u32x4{0, 0, 0, 0};
            }
        }
    };
    auto to_lds = [&](float2* buf) {
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int idx = tid + n * 512, r = idx >> 6;
            if constexpr (REAL) {
                const int part = idx & 1, il = (idx >> 1) & 31;
                float* bf = reinterpret_cast<float*>(buf);
#pragma unroll
                for (int t = 0; t < 4; ++t) bf[(4 * part + t) * (2 * PLANE) + r * 36 + il] = __uint_as_float(pre[n][t]);
            } else {
                const int c2 = idx & 3, ll = (idx >> 2) & 15;
                buf[(2 * c2) * PLANE + r * 18 + ll] = make_float2(__uint_as_float(pre[n].x), __uint_as_float(pre[n].y));
                buf[(2 * c2 + 1) * PLANE + r * 18 + ll] = make_float2(__uint_as_float(pre[n].z), __uint_as_float(pre[n].w));
            }
        }
    };

    int64_t rt = split;
    if (rt < ntiles) fetch(rt, 0);
    int cnt = 0;
    for (; rt < ntiles; rt += nsplit) {
        f32x16 acc[MTW];
#pragma unroll
        for (int r = 0; r < MTW * 16; ++r) acc[r / 16][r % 16] = 0.f;
#pragma unroll
        for (int ch = 0; ch < NCHUNK; ++ch, ++cnt) {
            float2* buf = gat8 + (cnt & 1) * (8 * PLANE);
            to_lds(buf);
            lds_barrier();
            if (ch + 1 < NCHUNK) fetch(rt, ch + 1);
            else if (rt + nsplit < ntiles) fetch(rt + nsplit, 0);
            const float2* mine = buf + w * PLANE;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (2 * ch + u >= P / 8) continue;  // the last chunk of a block that is no multiple of 16
                float2 xv[4];
#pragma unroll
                for (int c = 0; c < 4; c += 2) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(mine + col * 18 + 8 * u + 4 * kh + c);
                    xv[c] = make_float2(v.x, v.y);
                    xv[c + 1] = make_float2(v.z, v.w);
                }
                bf16x8 b[3];
                split_four(xv, b);
#pragma unroll
                for (int m = 0; m < MTW; ++m) plane_products<3, 3>(A[m][2 * ch + u], b, acc[m], acc[m]);
            }
        }
        char* const to = reinterpret_cast<char*>(out + (size_t)rt * k * (Q * kRT));
#pragma unroll
        for (int m = 0; m < MTW; ++m) {
            stage_finish<P, Q, kInGather, true, REAL>(acc[m], in, W, rt, g, mt0 + m, k, ld_in, B, lane);
#pragma unroll
            for (int o = 0; o < kOuts; ++o) {
                if (!REAL && Q % 16 != 0 && 16 * (mt0 + m) + 4 * (o / 2) + 2 * kh + o % 2 >= Q) continue;
                if constexpr (REAL) *reinterpret_cast<float*>(to + off[m][o]) = acc[m][o];
                else *reinterpret_cast<float2*>(to + off[m][o]) = make_float2(acc[m][2 * o], acc[m][2 * o + 1]);
            }
        }
    }
}

// dy, read through the outer permutation, in tiles dW[row tile][block][l][32 rows]: the operand of the stage that makes
// dY1 and of the weight gradient.  A workgroup moves 64 consecutive values of 32 rows through LDS (REAL: the 64 blocks
// from g0 of one pair of inputs, 2 x 64 floats), reading 512 bytes (2 x 256) of a row and writing runs of 256 bytes.
// Bound by memory (2048 x 4096 complex values: 28 us, 4.8 TB/s).  REAL with a number of blocks that is no multiple of
// four loads single values: a piece of four would start anywhere, and the last one of the last row would end past the
// tensor.
template <bool REAL>
__global__ void __launch_bounds__(256)
ctile_kernel(const float2* __restrict__ in, float2* __restrict__ out, int64_t B, int k, int P, int chunks)
{
    constexpr int kRow = 65;  // float2 (REAL: two rows of 65 floats, the first and the second input)
    __shared__ float2 buf[kRT * kRow];
    const int64_t rt = blockIdx.x / chunks;
    const int ch = (int)(blockIdx.x - rt * chunks), tid = threadIdx.x;
    const int per = (k + 63) / 64, pair = REAL ? ch / per : 0, g0 = REAL ? (ch - pair * per) * 64 : 0;
    const int j0 = 64 * ch, n = k * P;  // complex: flat position l * k + c
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int idx = tid + 256 * u, row = idx >> 5, c = idx & 31;
        const int64_t r = rt * kRT + row;
        bool in_row;
        size_t at;
        if constexpr (REAL) {
            in_row = g0 + 4 * (c & 15) < k;
            at = (size_t)r * (2 * n) + (size_t)(2 * pair + (c >> 4)) * k + g0 + 4 * (c & 15);
        } else {
            in_row = j0 + 2 * c < n;
            at = (size_t)r * (2 * n) + 2 * (j0 + 2 * c);
        }
        const float* p = reinterpret_cast<const float*>(in) + at;
        if (!REAL || k % 4 == 0) {
            v[u] = r < B && in_row ? ldg128(p) : u32x4{0, 0, 0, 0};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[u][e] = r < B && g0 + 4 * (c & 15) + e < k ? __float_as_uint(p[e]) : 0u;
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int idx = tid + 256 * u, row = idx >> 5, c = idx & 31;
        if constexpr (REAL) {
            float* b = reinterpret_cast<float*>(buf) + row * (2 * kRow) + (c >> 4) * kRow + 4 * (c & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = __uint_as_float(v[u][e]);
        } else {
            buf[row * kRow + 2 * c] = make_float2(__uint_as_float(v[u].x), __uint_as_float(v[u].y));
            buf[row * kRow + 2 * c + 1] = make_float2(__uint_as_float(v[u].z), __uint_as_float(v[u].w));
        }
    }
    lds_barrier();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int idx = tid + 256 * u, row = 2 * (idx & 15), j = idx >> 4;
        float2 a, b;
        size_t at;
        if constexpr (REAL) {
            if (g0 + j >= k) continue;
            const float* f = reinterpret_cast<const float*>(buf) + row * (2 * kRow) + j;
            a = make_float2(f[0], f[kRow]);
            b = make_float2(f[2 * kRow], f[3 * kRow]);
            at = (((size_t)rt * k + g0 + j) * P + pair) * kRT + row;
        } else {
            if (j0 + j >= n) continue;
            const int l = (j0 + j) / k, c = j0 + j - l * k;
            a = buf[row * kRow + j];
            b = buf[(row + 1) * kRow + j];
            at = (((size_t)rt * k + c) * P + l) * kRT + row;
        }
        *reinterpret_cast<f32x4*>(out + at) = f32x4{a.x, a.y, b.x, b.y};
    }
}

// part[z][g][ma][nb] = sum over the rows b of the tiles z, z + Z, ... of  A[b][g][ma] * conj(Bv[b][g][nb])
// A: dW (kInT or kInGather) or dY1 (kInT);  Bv: U (kInT) or x (kInNat).  M = 2*MA real rows (re and im of the
// result), N = NB columns, K = (row, component): with B'[(b,t)][nb] = component t of Bv[b][nb],
//   A'[2ma][(b,0)] = ar,  A'[2ma][(b,1)] = ai,  A'[2ma+1][(b,0)] = ai,  A'[2ma+1][(b,1)] = -ar.
// Wave w owns the 16 values ma = 16w .. 16w+15 and every column.  LDS holds each operand as three bf16 planes
// (monarch_planes.h) [idx][32 rows x 2 components + 8], the layout of an MFMA operand; the A rows 2ma+1 are made from
// 2ma on the way out of LDS.
template <int LEN, int NTHR, int MODE, bool REAL = false>
struct WgTile {
    static constexpr int kAll = kRT * LEN / 2;
    static constexpr int kPieces = (kAll + NTHR - 1) / NTHR;
    static __device__ __forceinline__ bool has(int idx) { return kAll % NTHR == 0 || idx < kAll; }
    static_assert(!REAL || kAll % NTHR == 0, "tile does not divide over the threads");
    static constexpr int kStride = REAL ? kRT + 8 : 2 * kRT + 8, kPlane = (REAL ? 2 : 1) * LEN * kStride, kLen = 3 * kPlane;  // bf16 values
    u32x4 v[kPieces];

    __device__ __forceinline__ void fetch(const float2* __restrict__ src, int64_t rt, int g, int k, int64_t ld, int64_t B, int tid)
    {
        const int64_t row0 = rt * kRT;
        if constexpr (MODE == kInNat) {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR;
                const int row = REAL ? 2 * (idx / LEN) + (idx & 1) : idx / (LEN / 2), c2 = REAL ? (idx % LEN) >> 1 : idx % (LEN / 2);
                v[n] = (has(idx) && row0 + row < B) ? ldg128(src + (row0 + row) * ld + (size_t)g * LEN + 2 * c2) : u32x4{0, 0, 0, 0};
            }
        } else {
            const float2* tile = src + ((size_t)rt * k + g) * (LEN * kRT);
#pragma unroll
            for (int n = 0; n < kPieces; ++n)
                if (has(tid + n * NTHR)) v[n] = ldg128(tile + 2 * (tid + n * NTHR));
        }
    }

    // one dword (two values next to each other in a row of LDS) to its place in each plane
    static __device__ __forceinline__ void put(bf16_t* p, uint32_t x, uint32_t y)
    {
        uint32_t w[3];
        split3(x, y, w);
#pragma unroll
        for (int u = 0; u < 3; ++u) *reinterpret_cast<uint32_t*>(p + u * kPlane) = w[u];
    }
    static __device__ __forceinline__ void put2(bf16_t* p, uint32_t x, uint32_t y, uint32_t z, uint32_t w)
    {
        uint32_t a[3], b[3];
        split3(x, y, a);
        split3(z, w, b);
#pragma unroll
        for (int u = 0; u < 3; ++u) *reinterpret_cast<u32x2*>(p + u * kPlane) = u32x2{a[u], b[u]};
    }
    __device__ __forceinline__ void to_lds(bf16_t* t, int tid) const
    {
        if constexpr (MODE == kInNat && REAL) {
            // of the four values of a piece an even lane takes two, an odd lane the other two, each of both lanes' rows
            const bool odd = tid & 1;
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, row = 2 * (idx / LEN), c2 = (idx % LEN) >> 1;
                uint32_t a[2], b[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const uint32_t mine = odd ? v[n][2 + c] : v[n][c], give = odd ? v[n][c] : v[n][2 + c];
                    const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)give, 0xB1, 0xf, 0xf, true);  // lane ^ 1
                    a[c] = odd ? got : mine;
                    b[c] = odd ? mine : got;
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) put(t + (4 * c2 + 2 * odd + c) * kStride + row, a[c], b[c]);
            }
        } else if constexpr (MODE == kInNat) {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, row = idx / (LEN / 2), c2 = idx - row * (LEN / 2);
                if (!has(idx)) continue;
                put(t + 2 * c2 * kStride + 2 * row, v[n].x, v[n].y);
                put(t + (2 * c2 + 1) * kStride + 2 * row, v[n].z, v[n].w);
            }
        } else {
#pragma unroll
            for (int n = 0; n < kPieces; ++n) {
                const int idx = tid + n * NTHR, i = idx / (kRT / 2), row = 2 * (idx - i * (kRT / 2));
                if (!has(idx)) continue;
                if constexpr (REAL) {
                    put(t + 2 * i * kStride + row, v[n].x, v[n].z);
                    put(t + (2 * i + 1) * kStride + row, v[n].y, v[n].w);
                } else {
                    put2(t + i * kStride + 2 * row, v[n].x, v[n].y, v[n].z, v[n].w);
                }
            }
        }
    }

    // the MFMA operand of step s: lane half h the values 16 s + 8 h .. of its row idx
    static __device__ __forceinline__ void read(bf16x8 (&b)[3], const bf16_t* t, int idx, int s, int h)
    {
#pragma unroll
        for (int u = 0; u < 3; ++u) b[u] = as_bf16x8(lds128(t + u * kPlane + idx * kStride + 16 * s + 8 * h));
    }
};

// REAL: real fp32 operands, two consecutive values per float2: out[g][ma'][nb'] = sum_b A[b][g][ma'] * Bv[b][g][nb']
// for the 2*MA x 2*NB real indices; a K = 2 step contracts two batch rows, each lane picking its component of the
// pair.
template <int MA, int NB, int AMODE, int BMODE, bool REAL>
struct WgradSums {
    static constexpr int NTHR = kTileWaves<MA> * 64, NTN = REAL ? (2 * NB + 31) / 32 : (NB + 31) / 32;
    using TA = WgTile<MA, NTHR, AMODE == kInGather ? kInT : AMODE, REAL>;
    using TB = WgTile<NB, NTHR, BMODE, REAL>;
    f32x16 acc[NTN];

    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int nt = 0; nt < NTN; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;
    }
    static __device__ __forceinline__ int row_of(int mt, int col)
    {
        const int ma = 16 * mt + (col >> 1);
        return MA % 16 != 0 && ma >= MA ? MA - 1 : ma;  // a row that does not exist
    }
    __device__ __forceinline__ void add_tile(const bf16_t* ta, const bf16_t* tb, int mt, int lane)
    {
        const int col = lane & 31, kh = lane >> 5, e = lane & 1, ma = row_of(mt, col);
        const uint32_t turn = e ? 0x01000302u : 0x03020100u, flip = e ? 0x80000000u : 0u;  // (ar, ai) or (ai, -ar)
#pragma unroll
        for (int s = 0; s < (REAL ? 2 : 4); ++s) {
            bf16x8 av[3];
            TA::read(av, ta, REAL ? 32 * mt + col : ma, s, kh);
            if constexpr (!REAL) {
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    u32x4 w = __builtin_bit_cast(u32x4, av[u]);
#pragma unroll
                    for (int c = 0; c < 4; ++c) w[c] = __builtin_amdgcn_perm(w[c], w[c], turn) ^ flip;
                    av[u] = as_bf16x8(w);
                }
            }
#pragma unroll
            for (int nt = 0; nt < NTN; ++nt) {
                int nb = 32 * nt + col;
                if (!REAL && NB % 32 != 0 && nb >= NB) nb = NB - 1;  // a column that does not exist
                bf16x8 bv[3];
                TB::read(bv, tb, nb, s, kh);
                plane_products<3, 3>(av, bv, acc[nt], acc[nt]);
            }
        }
    }
    // the sums of the tiles z, z + Z, ...: unscaled, what is not finite computed again in fp32, and out
    __device__ __forceinline__ void finish(const float2* __restrict__ A, const float2* __restrict__ Bv, float2* __restrict__ part, int64_t B,
                                           int k, int g, int z, int Z, int64_t lda, int64_t ldb, int mt, int lane)
    {
        const int col = lane & 31, kh = lane >> 5, e = lane & 1, ma = row_of(mt, col);
        const int64_t ntiles = (B + kRT - 1) / kRT;
        const bool off = planes_overflowed(acc);
#pragma unroll
        for (int nt = 0; nt < NTN; ++nt) acc[nt] *= kPlaneUnscale<2>;
        if (off) {
#pragma unroll
            for (int nt = 0; nt < NTN; ++nt) {
                if (!planes_overflowed(acc[nt])) continue;
                const bool mine = planes_clear(acc[nt]);
                int nb = REAL ? 16 * nt + (col >> 1) : 32 * nt + col;
                if (nb >= NB) nb = NB - 1;
#pragma clang loop unroll(disable)
                for (int64_t t = z; t < ntiles; t += Z)
#pragma clang loop unroll(disable)
                    for (int u0 = 0; u0 < kRT / 2; u0 += 2) {
                        float2 av[2], bv[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            av[u] = act_value<MA, AMODE, REAL>(A, t, 2 * (u0 + u) + kh, g, ma, k, lda, B);
                            bv[u] = act_value<NB, BMODE, REAL>(Bv, t, 2 * (u0 + u) + kh, g, nb, k, ldb, B);
                            if (!mine) bv[u] = make_float2(0.f, 0.f);
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            if constexpr (REAL) {
                                acc[nt] = mfma_f32(e ? av[u].y : av[u].x, e ? bv[u].y : bv[u].x, acc[nt]);
                            } else {
                                acc[nt] = mfma_f32(e ? av[u].y : av[u].x, bv[u].x, acc[nt]);
                                acc[nt] = mfma_f32(e ? -av[u].x : av[u].y, bv[u].y, acc[nt]);
                            }
                        }
                    }
            }
        }
        if constexpr (REAL) {
            // acc[nt][r]: row 32*mt + 8*(r/4) + 4*kh + r%4, column 32*nt + col of the (2*MA) x (2*NB) block
            float* o = reinterpret_cast<float*>(part) + ((size_t)z * k + g) * (4 * MA * NB);
#pragma unroll
            for (int nt = 0; nt < NTN; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    o[(size_t)(32 * mt + 8 * (r / 4) + 4 * kh + (r % 4)) * (2 * NB) + 32 * nt + col] = acc[nt][r];
        } else {
            float2* o = part + ((size_t)z * k + g) * (MA * NB);
#pragma unroll
            for (int nt = 0; nt < NTN; ++nt) {
                const int nb = 32 * nt + col;
                if (NB % 32 != 0 && nb >= NB) continue;
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (MA % 16 == 0 || 16 * mt + 4 * q4 + 2 * kh + h < MA) o[(16 * mt + 4 * q4 + 2 * kh + h) * NB + nb] = make_float2(acc[nt][4 * q4 + 2 * h], acc[nt][4 * q4 + 2 * h + 1]);
            }
        }
    }
};

// One factor's share of the backward in one launch: the gradient of its input, out = in W~ (cstage_kernel), and that of
// its weights, part[z] = sum over its tiles of in^T conj(other) (WgradSums).  `in` comes from memory once for both; a
// workgroup owns one block g and the row tiles z, z + Z, ..., and splits a tile of `in` into planes in both orders.
// LDS: `in` as rows (where the results take their place on the way out in rows), `in` and `other` as weight-gradient
// operands; 79.5 KiB at complex blocks of 64, so that two workgroups fit a CU.  In two launches `in` came twice and was
// split twice.  Backward, with the sums of both gradients in one launch: 64 complex blocks of 64, 2048 rows 208 -> 187
// us, 500 rows 86 -> 71; 48 of 48, 2048 rows 139 -> 110; 16 of 16, 64 rows 23.6 -> 15.5; real blocks, 64 of 64, 4000
// rows 192 -> 179, 16384 rows 723 -> 604; 32 of 32, 400 rows 29.6 -> 21.6, 16384 rows 188 -> 162.
template <int M, int IN, int OUT, int OTHER, bool REAL>
__global__ void __launch_bounds__(kTileWaves<M> * 64, 2)
cboth_kernel(const float2* __restrict__ in, const float2* __restrict__ W, const float2* __restrict__ other, float2* __restrict__ out,
             float2* __restrict__ part, int64_t B, int k, int Z, int perm_b)
{
    constexpr int NTHR = kTileWaves<M> * 64;
    using Tile = ActTile<M, NTHR, IN, REAL>;
    using Sums = WgradSums<M, M, IN, OTHER, REAL>;
    using Nat = NatOut<M, NTHR>;
    using Tiled = TiledOut<M, OUT, REAL>;
    static_assert(OUT != kOutNat || Nat::kLen * sizeof(float2) <= Tile::kLen * sizeof(bf16_t), "the results take the place of the rows");
    extern __shared__ __align__(16) bf16_t both_lds[];
    bf16_t *const act = both_lds, *const ta = act + Tile::kLen, *const tb = ta + Sums::TA::kLen;
    float2* const ost = reinterpret_cast<float2*>(act);

    const int g = (int)blockIdx.x / Z, z = (int)blockIdx.x - g * Z;
    const int tid = threadIdx.x, lane = tid & 63, mt = tid >> 6;
    const int col = lane & 31, kh = lane >> 5;
    const int64_t ntiles = (B + kRT - 1) / kRT, ld = (int64_t)k * M;

    bf16x8 A[M / 8][3];
    load_weights<M, M, true, REAL>(A, W, g, mt, col, kh);
    Tiled tiled;
    tiled.init(g, mt, kh, col, k, perm_b != 0);
    Sums sums;
    sums.zero();
    Tile pa;
    typename Sums::TB pb;
    int64_t rt = z;
    if (rt < ntiles) {
        pa.fetch(in, rt, g, k, ld, B, tid);
        pb.fetch(other, rt, g, k, ld, B, tid);
    }
    for (; rt < ntiles; rt += Z) {
        lds_barrier();
        pa.template to_both<typename Sums::TA>(act, ta, tid);
        pb.to_lds(tb, tid);
        lds_barrier();
        if (rt + Z < ntiles) {
            pa.fetch(in, rt + Z, g, k, ld, B, tid);
            pb.fetch(other, rt + Z, g, k, ld, B, tid);
        }
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int t = 0; t < M / 8; ++t) {
            bf16x8 xv[3];
            Tile::read(xv, act, t, lane);
            plane_products<3, 3>(A[t], xv, acc, acc);
        }
        stage_finish<M, M, IN, true, REAL>(acc, in, W, rt, g, mt, k, ld, B, lane);
        if constexpr (OUT == kOutNat) {
            lds_barrier();
            Nat::put(ost, acc, mt, kh, col);
        } else {
            tiled.store(out, acc, rt, mt, kh, k);
        }
        sums.add_tile(ta, tb, mt, lane);
        if constexpr (OUT == kOutNat) {
            lds_barrier();
            Nat::emit(ost, out, rt, g, ld, B, tid);
        }
    }
    sums.finish(in, other, part, B, k, g, z, Z, ld, ld, mt, lane);
}

struct SumJob {
    const f32x4* part;
    f32x4* out;
};
// out[e] = part[0][e] + part[1][e] + ... + part[Z-1][e], in that order, for both gradients; e counts float4s
__global__ void __launch_bounds__(256) csum_kernel(const SumJob first, const SumJob second, size_t n4, int Z)
{
    const f32x4* const part = blockIdx.y ? second.part : first.part;
    f32x4* const out = blockIdx.y ? second.out : first.out;
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n4) return;
    f32x4 s = part[e];
    int z = 1;
    for (; z + 8 <= Z; z += 8) {  // eight loads in flight, added in order
        f32x4 t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = part[(size_t)(z + u) * n4 + e];
#pragma unroll
        for (int u = 0; u < 8; ++u) { s.x += t[u].x; s.y += t[u].y; s.z += t[u].z; s.w += t[u].w; }
    }
    for (; z < Z; ++z) {
        const f32x4 t = part[(size_t)z * n4 + e];
        s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    out[e] = s;
}

int64_t tiles_of(const Problem& pb) { return (pb.B + kRT - 1) / kRT; }
size_t t_bytes(const Problem& pb, bool real) { return align_up((size_t)tiles_of(pb) * kRT * pb.kq() * (real ? sizeof(float) : sizeof(float2)), 256); }

// workgroups of one block: about `target_waves` in all, a multiple of 8, at most one per tile.  A workgroup loads and
// splits a block's weights before its first tile, so there are no more of them than stay resident: eight waves a CU (64
// complex blocks of 64, 2048 rows, forward and backward: 317 us with sixteen, 302 with eight), four for real layers,
// whose batches are the long ones (64 real blocks of 64, 12000 rows: 834 with sixteen, 807 with eight, 745 with four),
// but eight where single values are gathered (x M, 2 blocks of 64, 12000 rows: 17.5 us with four, 16.3 with eight)
int splits_for(const Problem& pb, int waves_per_wg, int target_waves)
{
    int64_t n = (target_waves / waves_per_wg + pb.k - 1) / pb.k;
    n = (n + 7) / 8 * 8;
    const int64_t t = tiles_of(pb);
    if (n > t) n = t;
    return (int)(n < 1 ? 1 : n);
}

// Batch chunks of the weight gradients: 512 workgroups, no more than two of which fit a CU at blocks of 64 (with 1024,
// 64 complex blocks of 64, 2048 rows, backward 194 -> 206 us, 48 112 -> 123, 64 real blocks of 64, 12000 rows 10 % more).
int wgrad_chunks(const Problem& pb)
{
    int64_t z = (512 + pb.k - 1) / pb.k;
    z = (z + 7) / 8 * 8;
    const int64_t t = tiles_of(pb);
    if (z > t) z = t;
    return (int)(z < 1 ? 1 : z);
}
// Real blocks of 32 have workgroups of one wave: twice as many of them where each then still has two tiles (32 blocks,
// 4000 rows, backward 58 -> 48 us, 16384 rows 197 -> 162; 20 blocks, 2000 rows, two tiles each before, 33 -> 37).
int real_chunks(const Problem& pb)
{
    const int z = wgrad_chunks(pb);
    return pb.p == 32 && tiles_of(pb) >= 4 * z ? 2 * z : z;
}

template <int M, int IN, int OUT, bool CONJT, bool REAL = false>
int launch_stage(const Problem& pb, const void* in, const void* W, void* out, hipStream_t st)
{
    const int nsplit = splits_for(pb, kTileWaves<M>, REAL && IN != kInGather ? 1024 : 2048);
    const int64_t grid = (int64_t)pb.k * nsplit;
    if (grid > 0x7fffffffLL) return -2;
    hipLaunchKernelGGL((cstage_kernel<M, M, IN, OUT, CONJT, REAL>), dim3((unsigned)grid), dim3(64 * kTileWaves<M>), 0, st, (const float2*)in,
                       (const float2*)W, REAL && OUT == kOutScatter ? (const float*)pb.bias : nullptr, (float2*)out, pb.B, pb.k, nsplit,
                       pb.perm_b() ? 1 : 0);
    return hip_status(hipGetLastError());
}

// the eight-blocks-per-workgroup stages: about one workgroup per CU, a multiple of 8 per (block octet, M tile); their
// weights take 12 registers a step of 8 inputs (32 real blocks of 32, 8000 rows, forward and backward: 144 us with
// two, 133 with one)
int splits8_for(const Problem& pb, int mtiles)
{
    int64_t n = (256 + (pb.k / 8) * mtiles - 1) / ((pb.k / 8) * mtiles);
    n = (n + 7) / 8 * 8;
    const int64_t t = tiles_of(pb);
    if (n > t) n = t;
    return (int)(n < 1 ? 1 : n);
}

template <int M, bool REAL = false>
int launch_scatter8(const Problem& pb, const void* T, const void* W, void* out, hipStream_t st)
{
    constexpr int MTG = kTileWaves<M>;
    const int nsplit = splits8_for(pb, MTG);
    const int64_t grid = (int64_t)(pb.k / 8) * MTG * nsplit;
    if (grid > 0x7fffffffLL) return -2;
    auto kern = cscatter8_kernel<M, M, REAL>;
    constexpr size_t lds = Scatter8<M, M>::kLds;
    if (allow_dynamic_lds((const void*)kern, lds) != hipSuccess) return -4;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), lds, st, (const float2*)T, (const float2*)W,
                       REAL ? (const float*)pb.bias : nullptr, (float2*)out, pb.B, pb.k, nsplit);
    return hip_status(hipGetLastError());
}

template <int M, bool REAL, int MTW>
int launch_gather8_tiles(const Problem& pb, const void* in, const void* W, void* out, hipStream_t st)
{
    constexpr int MTG = kTileWaves<M> / MTW;
    const int nsplit = splits8_for(pb, MTG);
    const int64_t grid = (int64_t)(pb.k / 8) * MTG * nsplit;
    if (grid > 0x7fffffffLL) return -2;
    auto kern = cgather8_kernel<M, M, REAL, MTW>;
    constexpr size_t lds = Gather8<M>::kLds;
    if (allow_dynamic_lds((const void*)kern, lds) != hipSuccess) return -4;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), lds, st, (const float2*)in, (const float2*)W,
                       (float2*)out, pb.B, pb.k, nsplit, pb.perm_b() ? 1 : 0);
    return hip_status(hipGetLastError());
}

// One M tile a wave, whose workgroups read the same rows once for each; two, with all the registers there are, for
// the real layers with blocks of 64 whose rows take more than 64 MB, so that they come from memory once (x M, 64
// blocks: 2000 rows, 33 MB, 39 us with one and 43 with two; 6000 rows 128 and 106, 30000 rows 616 and 485; 32 blocks,
// 6000 rows, 49 MB, 52 and 53, 12000 rows 122 and 100).
template <int M, bool REAL = false>
int launch_gather8(const Problem& pb, const void* in, const void* W, void* out, hipStream_t st)
{
    if constexpr (REAL && M == 32) {
        if (pb.B * pb.n_out() * (int64_t)sizeof(float) > (64LL << 20)) return launch_gather8_tiles<M, REAL, 2>(pb, in, W, out, st);
    }
    return launch_gather8_tiles<M, REAL, 1>(pb, in, W, out, st);
}

template <int M, int IN, int OUT, int OTHER, bool REAL>
int launch_both(const Problem& pb, const void* in, const void* W, const void* other, void* out, void* part, int Z, hipStream_t st)
{
    const int64_t grid = (int64_t)pb.k * Z;
    if (grid > 0x7fffffffLL) return -2;
    auto kern = cboth_kernel<M, IN, OUT, OTHER, REAL>;
    using Sums = WgradSums<M, M, IN, OTHER, REAL>;
    constexpr size_t lds = (size_t)(ActTile<M, Sums::NTHR, IN, REAL>::kLen + Sums::TA::kLen + Sums::TB::kLen) * sizeof(bf16_t);
    if (allow_dynamic_lds((const void*)kern, lds) != hipSuccess) return -4;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(Sums::NTHR), lds, st, (const float2*)in, (const float2*)W, (const float2*)other,
                       (float2*)out, (float2*)part, pb.B, pb.k, Z, pb.perm_b() ? 1 : 0);
    return hip_status(hipGetLastError());
}

// How dy gets to the backward's first factor: gathered by its workgroups in pieces of one value, or laid out in tiles by
// a launch of its own (ctile_kernel), which costs a pass over it.  Up to seven blocks leave that launch's lanes little
// to do.  Otherwise the pieces lose where they come from memory again and again: with many blocks from 4.5 MB on, with
// large complex blocks, and else beyond 18 MB.  Whole backward with the launch and without: 7 complex blocks of 64,
// 2048 rows 53.0 and 45.8 us; 32 of 32, 500 rows (4.1 MB) 30.7 and 27.5, 2048 rows 56.2 and 53.1; 48 of 48, 500 rows
// 54.9 and 53.0; 24 of 24, 6000 rows (28 MB) 78.7 and 74.8; 64 of 64, 64 rows 32.4 and 30.9, 200 rows (6.5 MB) 47.7 and
// 49.7; 12 of 64, 1500 rows (9 MB) 63.3 and 66.4; real blocks, 16 of 32, 8000 rows 52.1 and 47.0; 20 of 32, 2000 rows
// 33.0 and 29.3; 32 of 32, 1000 rows (4.1 MB) 29.2 and 27.0, 2500 rows (10 MB) 40.1 and 42.0; 64 of 64, 256 rows 39.5
// and 37.7, 330 rows (5.4 MB) 45.1 and 47.3.
template <int M, bool REAL>
bool gathers(const Problem& pb)
{
    const bool far = REAL ? pb.k >= 32 : pb.k > 48 || M >= 56;
    const size_t bytes = (size_t)pb.B * pb.n_out() * (REAL ? sizeof(float) : sizeof(float2));
    return pb.B == 0 || pb.k < 8 || bytes <= (far ? (size_t)9 << 19 : (size_t)18 << 20);
}

template <int M, bool REAL = false>
int launch_tile(const Problem& pb, const void* in, void* out, hipStream_t st)
{
    const int chunks = REAL ? M * ((pb.k + 63) / 64) : (pb.k * M + 63) / 64;
    const int64_t grid = tiles_of(pb) * chunks;
    if (grid > 0x7fffffffLL) return -2;
    hipLaunchKernelGGL(ctile_kernel<REAL>, dim3((unsigned)grid), dim3(256), 0, st, (const float2*)in, (float2*)out, pb.B, pb.k, M, chunks);
    return hip_status(hipGetLastError());
}

template <int M>
int run_fwd(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    int rc = launch_stage<M, kInNat, kOutTFwd, false>(pb, x, R, ws, st);
    if (rc) return rc;
    if (pb.k % 8 == 0) return launch_scatter8<M>(pb, ws, L, y, st);
    return launch_stage<M, kInT, kOutScatter, false>(pb, ws, L, y, st);
}

template <int M>
int run_fwd_h(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    int rc = pb.k % 8 == 0 ? launch_gather8<M>(pb, x, L, ws, st)
                           : launch_stage<M, kInGather, kOutTBwd, true>(pb, x, L, ws, st);
    if (rc) return rc;
    return launch_stage<M, kInT, kOutNat, true>(pb, ws, R, y, st);
}

template <int M, bool REAL = false>
int run_bwd(const Problem& pb, const void* dy, const void* x, const void* R, const void* L, void* dx, void* dR, void* dL,
            void* ws, hipStream_t st)
{
    const size_t mid = t_bytes(pb, REAL);
    char* const w = (char*)ws;
    void *const Ut = w, *const dWt = w + mid, *const dY1t = w + 2 * mid;
    const int Z = REAL && pb.ws_bytes >= real32_mfma_workspace(pb, 1) ? real_chunks(pb) : wgrad_chunks(pb);
    // the second factor's partial sums take the place of U and dW, which the first has read: Z <= the row tiles of 32,
    // so that Z M^2 k values fit two times 32 M k for each
    void* const partL = Z > 1 ? (void*)(w + 3 * mid) : dL;
    void* const partR = Z > 1 ? (void*)w : dR;
    int rc = launch_stage<M, kInNat, kOutTFwd, false, REAL>(pb, x, R, Ut, st);
    if (rc) return rc;
    if (gathers<M, REAL>(pb)) {
        rc = launch_both<M, kInGather, kOutTBwd, kInT, REAL>(pb, dy, L, Ut, dY1t, partL, Z, st);
    } else {
        rc = launch_tile<M, REAL>(pb, dy, dWt, st);
        if (!rc) rc = launch_both<M, kInT, kOutTBwd, kInT, REAL>(pb, dWt, L, Ut, dY1t, partL, Z, st);
    }
    if (!rc) rc = launch_both<M, kInT, kOutNat, kInNat, REAL>(pb, dY1t, R, x, dx, partR, Z, st);
    if (rc || Z == 1) return rc;
    const size_t n4 = (size_t)pb.k * M * M / (REAL ? 1 : 2);  // float4s of one gradient: (2M)^2 floats, or M^2 complex values, per block
    hipLaunchKernelGGL(csum_kernel, dim3((unsigned)((n4 + 255) / 256), 2), dim3(256), 0, st, SumJob{(const f32x4*)partL, (f32x4*)dL},
                       SumJob{(const f32x4*)partR, (f32x4*)dR}, n4, Z);
    return hip_status(hipGetLastError());
}

// ---- real fp32 layers with square blocks of 32 or 64 on the same kernels (REAL): M = block size / 2 ----
template <int M>
int run_real_fwd(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    int rc = launch_stage<M, kInNat, kOutTFwd, false, true>(pb, x, R, ws, st);
    if (rc) return rc;
    if (pb.k % 8 == 0) return launch_scatter8<M, true>(pb, ws, L, y, st);
    return launch_stage<M, kInT, kOutScatter, false, true>(pb, ws, L, y, st);
}

template <int M>
int run_real_fwd_t(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    int rc = pb.k % 8 == 0 ? launch_gather8<M, true>(pb, x, L, ws, st)
                           : launch_stage<M, kInGather, kOutTBwd, true, true>(pb, x, L, ws, st);
    if (rc) return rc;
    return launch_stage<M, kInT, kOutNat, true, true>(pb, ws, R, y, st);
}

}  // namespace

bool real32_mfma_supported(const Problem& pb)
{
    return pb.dtype == 0 && pb.p == pb.q && pb.q == pb.s && (pb.p == 32 || pb.p == 64);
}

// pass: 0 forward, 1 backward, 2 transposed multiply
static size_t real32_bwd_bytes(const Problem& pb, int Z)
{
    return 3 * t_bytes(pb, true) + (Z > 1 ? align_up((size_t)Z * pb.n_L() * sizeof(float), 256) : 0);
}
size_t real32_mfma_workspace(const Problem& pb, int pass)
{
    return pass != 1 ? t_bytes(pb, true) : real32_bwd_bytes(pb, real_chunks(pb));
}
size_t real32_mfma_bwd_least(const Problem& pb) { return real32_bwd_bytes(pb, wgrad_chunks(pb)); }

int real32_mfma_fwd(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    return pb.p == 32 ? run_real_fwd<16>(pb, x, R, L, y, ws, st) : run_real_fwd<32>(pb, x, R, L, y, ws, st);
}

int real32_mfma_fwd_t(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    return pb.p == 32 ? run_real_fwd_t<16>(pb, x, R, L, y, ws, st) : run_real_fwd_t<32>(pb, x, R, L, y, ws, st);
}

int real32_mfma_bwd(const Problem& pb, const void* dy, const void* x, const void* R, const void* L, void* dx, void* dR,
                    void* dL, void* ws, hipStream_t st)
{
    if (pb.B == 0) {
        const int rc = launch_fill_zero_f32((float*)dR, pb.n_R(), st);
        return rc ? rc : launch_fill_zero_f32((float*)dL, pb.n_L(), st);
    }
    return pb.p == 32 ? run_bwd<16, true>(pb, dy, x, R, L, dx, dR, dL, ws, st) : run_bwd<32, true>(pb, dy, x, R, L, dx, dR, dL, ws, st);
}

bool complex_mfma_supported(const Problem& pb)
{
    return pb.p == pb.q && pb.q == pb.s && pb.p >= 16 && pb.p <= 64 && pb.p % 8 == 0;
}

// pass: 0 forward, 1 backward, 2 conjugate-transpose forward
size_t complex_mfma_workspace(const Problem& pb, int pass)
{
    if (pass != 1) return t_bytes(pb, false);
    const int Z = wgrad_chunks(pb);
    return 3 * t_bytes(pb, false) + (Z > 1 ? align_up((size_t)Z * pb.n_L() * sizeof(float2), 256) : 0);
}

int complex_mfma_fwd(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    switch (pb.p) {
        case 16: return run_fwd<16>(pb, x, R, L, y, ws, st);
        case 24: return run_fwd<24>(pb, x, R, L, y, ws, st);
        case 32: return run_fwd<32>(pb, x, R, L, y, ws, st);
        case 40: return run_fwd<40>(pb, x, R, L, y, ws, st);
        case 48: return run_fwd<48>(pb, x, R, L, y, ws, st);
        case 56: return run_fwd<56>(pb, x, R, L, y, ws, st);
        case 64: return run_fwd<64>(pb, x, R, L, y, ws, st);
        default: return -2;
    }
}

int complex_mfma_fwd_h(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    switch (pb.p) {
        case 16: return run_fwd_h<16>(pb, x, R, L, y, ws, st);
        case 24: return run_fwd_h<24>(pb, x, R, L, y, ws, st);
        case 32: return run_fwd_h<32>(pb, x, R, L, y, ws, st);
        case 40: return run_fwd_h<40>(pb, x, R, L, y, ws, st);
        case 48: return run_fwd_h<48>(pb, x, R, L, y, ws, st);
        case 56: return run_fwd_h<56>(pb, x, R, L, y, ws, st);
        case 64: return run_fwd_h<64>(pb, x, R, L, y, ws, st);
        default: return -2;
    }
}

int complex_mfma_bwd(const Problem& pb, const void* dy, const void* x, const void* R, const void* L, void* dx, void* dR,
                     void* dL, void* ws, hipStream_t st)
{
    switch (pb.p) {
        case 16: return run_bwd<16>(pb, dy, x, R, L, dx, dR, dL, ws, st);
        case 24: return run_bwd<24>(pb, dy, x, R, L, dx, dR, dL, ws, st);
        case 32: return run_bwd<32>(pb, dy, x, R, L, dx, dR, dL, ws, st);
        case 40: return run_bwd<40>(pb, dy, x, R, L, dx, dR, dL, ws, st);
        case 48: return run_bwd<48>(pb, dy, x, R, L, dx, dR, dL, ws, st);
        case 56: return run_bwd<56>(pb, dy, x, R, L, dx, dR, dL, ws, st);
        case 64: return run_bwd<64>(pb, dy, x, R, L, dx, dR, dL, ws, st);
        default: return -2;
    }
}

}  // namespace monarch
