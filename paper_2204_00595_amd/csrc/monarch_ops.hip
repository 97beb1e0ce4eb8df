// Shape-generic multiply on the matrix cores, fp32 and bf16: any k, any block sizes from 16 up, both readings of the
// mid permutation.  It serves the calls that bring a workspace on every shape without a kernel of its own (fp32
// Transformer layers, block sizes that are multiples of nothing); without a workspace, or below 16, the SIMT kernels
// of monarch_generic.hip run.
//
// Every step of Section 3.3 and every adjoint of one is a batched contraction whose operands lie in memory with three
// element strides each (block, row, contraction index), and the permutations are nothing but such strides:
//   step 1         U[b][j*k + kk]  = sum_i x[b][kk*p + i] R[kk][j][i]       (default reading: U is the permuted vector)
//   step 2, 3      y[b][l*k + c]   = sum_r U[b][c*q + r] L[c][l][r]
//   backward       dU[b][c*q + r]  = sum_l dy[b][l*k + c] L[c][l][r]
//                  dx[b][kk*p + i] = sum_j dU[b][j*k + kk] R[kk][j][i]
//                  dL[c][l][r]     = sum_b dy[b][l*k + c] U[b][c*q + r],   dR likewise from dU and x
// With MONARCH_FLAG_PERM_B the vector between the factors is kept in stage-1 order and the strides on either side of it
// change places.  So there is one contraction, ops_gemm: O[g][m][n] = sum_k A[g][m][k] B[g][n][k].
//
// Precision: U and dU are fp32 for both types, as in the SIMT kernels; bf16 layers are rounded once, when a result is
// stored.
// Everything runs on the bf16 matrix cores, which are exact in the products and add them in fp32.  An fp32 operand is
// taken as three bf16 planes that add up to it exactly (split3), and a product of two such operands as the six largest
// products of planes (three where the other operand is bf16).  An accumulator takes one rounding per 16 contraction
// indices and product of planes, so the results are closer to float64 than those of v_mfma_f32_32x32x2_f32 with one per
// 2 (normal operands, 192 indices: 2.0e-7 against 2.5e-7; with the small products in a sum of their own, as the weight
// gradients have them, 0.8e-7).  What the planes cannot hold (infinities, operands from 2^104 and results from 2^80 on)
// is found in the finished tile; those rows of it are then computed again in fp32 (op_redo).  With an infinity in one
// of every 32 rows that costs: 768 -> 768 fp32, 12608 rows, forward 82 -> 322 us and backward 230 -> 539, 1024 -> 4096
// fp32, 8000 rows, 169 -> 832 and 409 -> 1187.
//
// What bounds it: a product of two fp32 operands costs the matrix cores 6/14.4 of its time on the fp32 cores (2058
// against 143 TFLOP/s in a loop of MFMAs alone), and what is left is the vector work of splitting (5.5 instructions an
// element, once per tile that takes it) and LDS.  Neither is near its rate: the chunks are a chain of load, split,
// barrier and multiply, and what hides it is the number of workgroups on a CU.  So a chunk is 16 contraction indices,
// one MFMA deep: 64 x 64 tiles then take 30 KB of LDS, five to a CU, where chunks of 32 leave two (4096 -> 1024 fp32,
// 8000 rows, whole step: 660 us on the fp32 matrix cores, 674 in planes with chunks of 32, 455 with 16); few workgroups
// take chunks of 32 (launch_chunks).  Small and odd bf16 layers are bound by the memory system.  The intermediate goes
// through memory (for most shapes it stays in the last-level cache): a fused kernel would hold all k blocks of a row
// tile, which leaves the large shapes one 16-row tile per CU. Measured, training step: 768 -> 768 fp32, k = 4, 12608
// rows: 4369 us on the SIMT kernels, 297 on the fp32 matrix cores, 256 in planes, with the weights laid out as planes
// and large tiles for their gradients 210 to 217 (one contraction of 3.7 GFLOP takes 34 us, 38 where its rows come
// interleaved, the two weight gradients 55); 196 -> 256 bf16, blocks of 49 and 64, 32768 rows: 458, 121, 96, now 86 to
// 93 us; 2048 -> 512 fp32, 3000 rows: 137, in planes 112.
#include <algorithm>
#include <type_traits>
#include "monarch_internal.h"
#include "monarch_device.h"
#include "monarch_mfma_common.h"
#include "monarch_colsum.h"
#include "monarch_planes.h"

namespace monarch {
namespace {

constexpr int kCUs = 256;

typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr int kStep = 16;  // contraction indices of an MFMA

// How an operand is taken: kPieces16, 16-byte pieces along the contiguous index, all of them aligned and inside;
// kPiecesAny, 16-byte pieces along it wherever they start (gfx950 loads from any address), a piece that crosses the
// limit being read from the elements that end there and shifted into place on its way to LDS; kElements, single
// elements at any stride.
enum Take { kElements, kPiecesAny, kPieces16 };

// One operand: element (g, row, k) at p[g*g_s + row*r_s + k*k_s].
struct OpOperand {
    const void* p;
    int64_t g_s, r_s, k_s;
    Take take;
};
struct OpDesc {
    OpOperand a, b;
    void* o;           // output, or the partial tiles [split][g][m][n] (fp32)
    int64_t o_g, o_m, o_n;  // element (g, m, n) goes to g*o_g + m*o_m + n*o_n ...
    int o_mid;         // ... or, 1: to the stage-1 position of element g*N + n of the permuted vector (default reading)
    int o_turn;        // long batches: how a result's neighbours in memory are found (RowsStore)
    const void* bias;  // added to o at the offset g*o_g + n*o_n (may be null)
    int64_t M, K;
    int N, G;
    int tiles_m, tiles_n;
    int nouter, deal;  // row tiles (or batch chunks); 1: they are dealt to the XCDs
    int64_t k_chunk;   // contraction indices per batch chunk (K when the contraction is not split)
    int blocks;        // workgroups
};

// Buffer accesses: the base is uniform, a lane adds a 32-bit offset, and a lane whose offset is kNowhere reads zero or
// writes nothing.  So a ragged tile needs no branch around a load -- with branches the compiler cannot count the
// loads in flight and waits for all of them at the first use, which undoes the prefetching.
constexpr uint32_t kNowhere = 0xffffffffu, kBufferBytes = 0x7fffffffu;  // ops_supported keeps a tile's extent below 2 GiB
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void* p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, kBufferBytes, 0x00020000);
}

template <typename T>
struct TileDrop {
    // v without its first n elements (zeros follow); a piece with nothing inside was loaded as zeros
    static __device__ __forceinline__ u32x4 drop(u32x4 v, int n)
    {
        const int bytes = n * (int)sizeof(T);
        if (bytes & 8) v = u32x4{v[2], v[3], 0u, 0u};
        if (bytes & 4) v = u32x4{v[1], v[2], v[3], 0u};
        if constexpr (sizeof(T) == 2) {
            const uint32_t s = (bytes & 2) * 8;
            v = u32x4{__builtin_amdgcn_alignbit(v[1], v[0], s), __builtin_amdgcn_alignbit(v[2], v[1], s),
                      __builtin_amdgcn_alignbit(v[3], v[2], s), v[3] >> s};
        }
        return v;
    }
};

// A C x O tile of an operand (C: extent along the index with the unit or smallest stride, O: along the other one) on
// its way from memory to LDS [o][c], row stride LSTR elements: bf16 as it is, fp32 as three planes of SZ elements.
// Elements past the limits read as zeros.  Single elements are loaded with consecutive lanes on consecutive c (at a
// stride of 16 bytes a load takes the L1 31 cycles, at 32 bytes 60), and neighbouring lanes exchange them so that each
// has two for a dword.
template <typename T, int C, int O, int LSTR, Take TAKE, int SZ, int THREADS>
struct OpTile {
    static constexpr bool VEC = TAKE != kElements, kSplit = sizeof(T) == 4;
    static constexpr int V = VEC ? 16 / (int)sizeof(T) : 1;          // elements per piece
    static constexpr int PPO = C / V;                                // pieces per o
    static constexpr int kPieces = PPO * O;
    static constexpr int NP = (kPieces + THREADS - 1) / THREADS;   // per thread
    static constexpr int kDwords = VEC ? 4 : 1;
    static_assert(C % V == 0 && LSTR * 2 % 16 == 0, "tile");
    static constexpr bool kEven = THREADS % PPO == 0;  // a thread's pieces share c and step in o by a uniform amount
    static_assert(VEC || (kEven && kPieces % THREADS == 0 && NP % 2 == 0), "element-wise tiles divide over the threads");
    uint32_t r[NP * kDwords];
    int over[TAKE == kPiecesAny ? (kEven ? 1 : NP) : 1];  // elements of a piece past the limit

    __device__ __forceinline__ void fetch(const T* base, uint32_t os, uint32_t cs, int olim, int clim, int tid)
    {
        // the piece that ends at the limit may start before `base`, which is not the start of its row there
        constexpr uint32_t kBack = TAKE == kPiecesAny ? 16 : 0;
        const auto rs = buffer_at(reinterpret_cast<const char*>(base) - kBack);
        const int o0 = tid / PPO, c0 = (tid % PPO) * V;
        const uint32_t v0 = (o0 * os + c0 * cs) * (uint32_t)sizeof(T) + kBack;
#pragma unroll
        for (int n = 0; n < NP; ++n) {
            const int idx = tid + n * THREADS;
            const int o = kEven ? o0 + n * (THREADS / PPO) : idx / PPO, c = kEven ? c0 : (idx % PPO) * V;
            uint32_t vo = kEven ? v0 : (o * os + c * cs) * (uint32_t)sizeof(T) + kBack;
            const uint32_t so = kEven ? n * (THREADS / PPO) * os * (uint32_t)sizeof(T) : 0u;
            bool in = o < olim && c < clim;
            if constexpr (kPieces % THREADS != 0) in = in && idx < kPieces;
            if constexpr (TAKE == kPiecesAny) {
                const int past = c + V > clim ? c + V - clim : 0;
                over[kEven ? 0 : n] = past;
                vo -= past * (uint32_t)sizeof(T);
            }
            const uint32_t at = in ? vo : kNowhere;
            if constexpr (VEC) {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, at, so, 0);
#pragma unroll
                for (int w = 0; w < 4; ++w) r[4 * n + w] = v[w];
            } else if constexpr (sizeof(T) == 4) {
                r[n] = __builtin_amdgcn_raw_buffer_load_b32(rs, at, so, 0);
            } else {
                r[n] = __builtin_amdgcn_raw_buffer_load_b16(rs, at, so, 0);
            }
        }
    }
    __device__ __forceinline__ void store(bf16_t* lds, int tid) const
    {
        if constexpr (VEC) {
#pragma unroll
            for (int n = 0; n < NP; ++n) {
                const int idx = tid + n * THREADS, o = idx / PPO, c = (idx % PPO) * V;
                u32x4 v = {r[4 * n], r[4 * n + 1], r[4 * n + 2], r[4 * n + 3]};
                if constexpr (TAKE == kPiecesAny) v = TileDrop<T>::drop(v, over[kEven ? 0 : n]);
                if (kPieces % THREADS == 0 || idx < kPieces) {
                    if constexpr (kSplit) {
                        uint32_t lo[3], hi[3];
                        split3(v[0], v[1], lo);
                        split3(v[2], v[3], hi);
#pragma unroll
                        for (int w = 0; w < 3; ++w) *reinterpret_cast<u32x2*>(lds + w * SZ + o * LSTR + c) = u32x2{lo[w], hi[w]};
                    } else {
                        *reinterpret_cast<u32x4*>(lds + o * LSTR + c) = v;
                    }
                }
            }
        } else {
            // of the elements n and n + 1 an even lane takes n of both lanes, an odd lane n + 1
            const bool odd = tid & 1;
            bf16_t* const to = lds + (tid / PPO + (odd ? THREADS / PPO : 0)) * LSTR + (tid % PPO & ~1);
#pragma unroll
            for (int n = 0; n < NP; n += 2) {
                const uint32_t mine = odd ? r[n + 1] : r[n], give = odd ? r[n] : r[n + 1];
                const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)give, 0xB1, 0xf, 0xf, true);  // lane ^ 1
                const uint32_t a = odd ? got : mine, b = odd ? mine : got;
                bf16_t* const p = to + n * (THREADS / PPO) * LSTR;
                if constexpr (kSplit) {
                    uint32_t v[3];
                    split3(a, b, v);
#pragma unroll
                    for (int w = 0; w < 3; ++w) *reinterpret_cast<uint32_t*>(p + w * SZ) = v[w];
                } else {
                    *reinterpret_cast<uint32_t*>(p) = a | b << 16;
                }
            }
        }
    }
};

// LDS row strides: contraction-contiguous tiles [row][KC] + 16 bytes (eight lanes of a b128 read then start in eight
// different bank groups); row-contiguous tiles [k][rows]: odd multiples of 64 bytes, so that the four rows a half
// wave of the transposing read touches fall on disjoint bank quarters.
template <bool RC, int ROWS, int KC>
constexpr int op_lstr()
{
    if (!RC) return KC + 8;
    return ROWS % 64 == 32 ? ROWS : ROWS + 32;
}

__device__ __forceinline__ u32x2 op_lds_tr16(const bf16_t* p)
{
    s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(const_cast<bf16_t*>(p)));
    return __builtin_bit_cast(u32x2, v);
}

// The MFMA operands of the contraction indices k0 .. k0 + 15 for the 32 rows from r0, from PL planes of SZ elements:
// lane (row = lane % 32, h = lane / 32) holds the indices k0 + 8 h .. of its row.
template <bool RC, int LSTR, int PL, int SZ>
struct OpFrag {
    bf16x8 v[PL];
    __device__ __forceinline__ void read(const bf16_t* lds, int r0, int k0, int lane)
    {
#pragma unroll
        for (int w = 0; w < PL; ++w) {
            if constexpr (!RC) {
                v[w] = as_bf16x8(lds128(lds + w * SZ + (r0 + (lane & 31)) * LSTR + k0 + 8 * (lane >> 5)));
            } else {
                // transposing read: within 16 lanes, lane i gets element i % 4 of lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4
                const int G = lane >> 4, j = lane & 15;
                const bf16_t* p = lds + w * SZ + (k0 + 8 * (G >> 1) + (j >> 2)) * LSTR + r0 + 16 * (G & 1) + 4 * (j & 3);
                const u32x2 lo = op_lds_tr16(p), hi = op_lds_tr16(p + 4 * LSTR);
                v[w] = as_bf16x8(u32x4{lo[0], lo[1], hi[0], hi[1]});
            }
        }
    }
};
template <int WM_, int WN_, int MT_, int NT_, int CHUNK_ = 16>
struct OpCfg {  // WM x WN waves, each MT x NT tiles of 32 x 32; CHUNK: contraction indices of a chunk where planes are multiplied
    static constexpr int WM = WM_, WN = WN_, MT = MT_, NT = NT_, CHUNK = CHUNK_;
    static constexpr int TM = WM * MT * 32, TN = WN * NT * 32;
};

// Rows of wave (wm, wn)'s 32 x 32 tiles that hold something not finite, again on the fp32 matrix cores, straight from
// memory, sixteen contraction indices to a partial sum.  The other rows keep their results: their operand is zero here
// (a weight that is not finite leaves no other rows).  All tile sizes have the same groups of 32 columns, so that a
// row's result depends neither on the rows beside it nor on the tile that was picked for the batch.
template <typename T>
__device__ __forceinline__ float op_element(__amdgpu_buffer_rsrc_t rs, uint32_t at, uint32_t scalar)
{
    if constexpr (sizeof(T) == 4) return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, at, scalar, 0));
    else return bf16_to_f32((bf16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, at, scalar, 0));
}
template <typename TA, typename TB, int MT, int NT>
__device__ __forceinline__ void op_redo(const OpDesc& d, int g, int64_t m0, int n0, int mlim, int nlim, int wm, int wn, int64_t k_lo, int64_t k_len,
                                        int lane, f32x16 (&acc)[MT][NT])
{
    wm = __builtin_amdgcn_readfirstlane(wm) * (MT * 32);  // uniform, for the addresses to be
    wn = __builtin_amdgcn_readfirstlane(wn) * (NT * 32);
    mlim -= wm;
    nlim -= wn;
    const TA* pa = static_cast<const TA*>(d.a.p) + g * d.a.g_s + (m0 + wm) * d.a.r_s + k_lo * d.a.k_s;
    const TB* pb = static_cast<const TB*>(d.b.p) + g * d.b.g_s + (int64_t)(n0 + wn) * d.b.r_s + k_lo * d.b.k_s;
    const int row = lane & 31, h = lane >> 5;
    const uint32_t a_2k = 2u * (uint32_t)d.a.k_s * (uint32_t)sizeof(TA), b_2k = 2u * (uint32_t)d.b.k_s * (uint32_t)sizeof(TB);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            uint32_t bad = 0;  // rows
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float v = acc[i][j][r];
                const uint64_t off = __ballot(planes_bad(v));
                if ((uint32_t)off) bad |= 1u << (8 * (r / 4) + r % 4);
                if ((uint32_t)(off >> 32)) bad |= 1u << (8 * (r / 4) + 4 + r % 4);
            }
            if (!bad) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float v = acc[i][j][r];
                acc[i][j][r] = bad >> (8 * (r / 4) + 4 * h + r % 4) & 1 ? 0.f : v;
            }
            const bool a_in = i * 32 + row < mlim && (bad >> row & 1), b_in = j * 32 + row < nlim;
            const uint32_t a_at = (uint32_t)((i * 32 + row) * (int)d.a.r_s + h * (int)d.a.k_s) * (uint32_t)sizeof(TA);
            const uint32_t b_at = (uint32_t)((j * 32 + row) * (int)d.b.r_s + h * (int)d.b.k_s) * (uint32_t)sizeof(TB);
#pragma clang loop unroll(disable)
            for (int64_t k = 0; k < k_len; k += 16) {
                const auto ra = buffer_at(pa + k * d.a.k_s), rb = buffer_at(pb + k * d.b.k_s);
                const int left = k_len - k < 16 ? (int)(k_len - k) : 16;
                f32x16 sum;
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[r] = 0.f;
#pragma clang loop unroll(disable)
                for (int u0 = 0; u0 < 8; u0 += 4) {
                    float a[4], b[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool in = 2 * (u0 + u) + h < left;
                        a[u] = op_element<TA>(ra, a_in && in ? a_at : kNowhere, (u0 + u) * a_2k);
                        b[u] = op_element<TB>(rb, b_in && in ? b_at : kNowhere, (u0 + u) * b_2k);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u], b[u], sum, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] += sum[r];
            }
        }
}

template <typename TO, bool PARTIAL, int MT, int NT>
__device__ __forceinline__ void op_store(const OpDesc& d, const f32x16 (&acc)[MT][NT], int outer, int g, int64_t m0, int n0,
                                         int mlim, int nlim, int wm, int wn, int lane)
{
    const int col = lane & 31, rh = 4 * (lane >> 5);
    using OT = typename std::conditional<PARTIAL, float, TO>::type;
    OT* O = static_cast<OT*>(d.o);
    uint32_t o_m = (uint32_t)d.o_m;
    if constexpr (PARTIAL) {
        O += (((int64_t)outer * d.G + g) * d.M + m0) * d.N;
        o_m = (uint32_t)d.N;
    } else {
        O += m0 * d.o_m;
    }
    const auto out = buffer_at(O);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int n = (wn * NT + j) * 32 + col;
        uint32_t off = (uint32_t)(n0 + n);
        float bv = 0.f;
        if constexpr (!PARTIAL) {
            off = (uint32_t)g * (uint32_t)d.o_g + off * (uint32_t)d.o_n;
            if (d.o_mid) {
                const uint32_t f = (uint32_t)(g * d.N + n0 + n), jj = f / (uint32_t)d.G;
                off = (f - jj * (uint32_t)d.G) * (uint32_t)d.N + jj;
            }
            if (d.bias) {
                const uint32_t at = n < nlim ? off * (uint32_t)sizeof(TO) : kNowhere;
                if constexpr (sizeof(TO) == 4) bv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(buffer_at(d.bias), at, 0, 0));
                else bv = bf16_to_f32((bf16_t)__builtin_amdgcn_raw_buffer_load_b16(buffer_at(d.bias), at, 0, 0));
            }
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = (wm * MT + i) * 32 + 8 * (r / 4) + rh + r % 4;
                const uint32_t at = m < mlim && n < nlim ? (m * o_m + off) * (uint32_t)sizeof(OT) : kNowhere;
                const float v = acc[i][j][r] + bv;
                if constexpr (sizeof(OT) == 4) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), out, at, 0, 0);
                else __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(v), out, at, 0, 0);
            }
    }
}

// One workgroup, `bid` of d.blocks.  TA, TB, TO: element types of the operands and the output in memory.  RA / RB: the
// operand's row index (not the contraction) is the contiguous one.  PARTIAL: fp32 partial tiles of a split contraction
// instead of the output.
// Workgroup order: the row tile (PARTIAL: the batch chunk) is dealt to the XCDs, and the blocks and column tiles of one
// row tile follow each other on that XCD: strided operands and outputs of the k blocks share their cache lines, which
// then meet in one L2.
template <typename TA, typename TB, typename TO, class Cfg, bool RA, bool RB, bool PARTIAL, Take AV, Take BV>
struct OpGemm {
    static constexpr bool kSplit = sizeof(TA) == 4 || sizeof(TB) == 4;
    static constexpr int PA = sizeof(TA) == 2 ? 1 : 3, PB = sizeof(TB) == 2 ? 1 : 3, kThreads = Cfg::WM * Cfg::WN * 64;
    static constexpr int KC = kSplit ? Cfg::CHUNK : 32, LA = op_lstr<RA, Cfg::TM, KC>(), LB = op_lstr<RB, Cfg::TN, KC>();
    static constexpr int SZA = RA ? KC * LA : Cfg::TM * LA, SZB = RB ? KC * LB : Cfg::TN * LB;
    static constexpr int SZ = PA * SZA + PB * SZB;
    static constexpr size_t kLds = 2 * sizeof(bf16_t) * (size_t)SZ;
    static __device__ void run(const OpDesc& d, int bid, unsigned char* op_lds);
};
template <typename TA, typename TB, typename TO, class Cfg, bool RA, bool RB, bool PARTIAL, Take AV, Take BV>
__device__ __forceinline__ void OpGemm<TA, TB, TO, Cfg, RA, RB, PARTIAL, AV, BV>::run(const OpDesc& d, int bid, unsigned char* op_lds)
{
    constexpr int MT = Cfg::MT, NT = Cfg::NT, TM = Cfg::TM, TN = Cfg::TN;
    using TileA = OpTile<TA, RA ? TM : KC, RA ? KC : TM, LA, AV, SZA, kThreads>;
    using TileB = OpTile<TB, RB ? TN : KC, RB ? KC : TN, LB, BV, SZB, kThreads>;
    bf16_t* const lds = reinterpret_cast<bf16_t*>(op_lds);

    const int inner = d.G * d.tiles_n * (PARTIAL ? d.tiles_m : 1);
    const int seq = d.deal ? bid >> 3 : bid;
    const int outer = d.deal ? (seq / inner) * 8 + (bid & 7) : seq / inner;
    if (outer >= d.nouter) return;
    int in = seq % inner;
    const int g = in % d.G;
    in /= d.G;
    const int tn = in % d.tiles_n;
    const int tm = PARTIAL ? in / d.tiles_n : outer;
    const int64_t m0 = (int64_t)tm * TM;
    const int n0 = tn * TN;
    const int64_t k_lo = PARTIAL ? (int64_t)outer * d.k_chunk : 0;
    const int64_t k_len = PARTIAL ? (d.K - k_lo < d.k_chunk ? d.K - k_lo : d.k_chunk) : d.K;
    const int mlim = d.M - m0 < TM ? (int)(d.M - m0) : TM, nlim = d.N - n0 < TN ? d.N - n0 : TN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % Cfg::WM, wn = wave / Cfg::WM;
    const TA* pa = static_cast<const TA*>(d.a.p) + g * d.a.g_s + m0 * d.a.r_s + k_lo * d.a.k_s;
    const TB* pb = static_cast<const TB*>(d.b.p) + g * d.b.g_s + (int64_t)n0 * d.b.r_s + k_lo * d.b.k_s;
    const uint32_t a_o = (uint32_t)(RA ? d.a.k_s : d.a.r_s), a_c = (uint32_t)(RA ? d.a.r_s : d.a.k_s);
    const uint32_t b_o = (uint32_t)(RB ? d.b.k_s : d.b.r_s), b_c = (uint32_t)(RB ? d.b.r_s : d.b.k_s);

    // Partial tiles, whose sums run over hundreds of rows, keep the small products apart: a single sum left the fp32
    // weight gradients of some hundred rows further off float64 than the SIMT kernels, which add up 16 rows at a
    // time.
    constexpr int SUMS = PARTIAL && kSplit ? 2 : 1;
    f32x16 sums[SUMS][MT][NT];
#pragma unroll
    for (int u = 0; u < SUMS; ++u)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) sums[u][i][j][r] = 0.f;

    // two chunks are on their way from memory while one is multiplied: with one, a chunk's time on the matrix cores
    // (0.4 to 0.9 us) does not cover a load's
    struct Stage {
        TileA a;
        TileB b;
    };
    Stage s0, s1;
    auto fetch = [&](Stage& s, int64_t kk) {
        const int64_t left = k_len - kk;
        const int klim = left < KC ? (left > 0 ? (int)left : 0) : KC;
        s.a.fetch(pa + kk * d.a.k_s, a_o, a_c, RA ? klim : mlim, RA ? mlim : klim, tid);
        s.b.fetch(pb + kk * d.b.k_s, b_o, b_c, RB ? klim : nlim, RB ? nlim : klim, tid);
        __builtin_amdgcn_sched_barrier(0);  // in this order: the wait for a chunk counts the loads behind it
    };
    auto put = [&](const Stage& s, int buf) {
        s.a.store(lds + buf * SZ, tid);
        s.b.store(lds + buf * SZ + PA * SZA, tid);
    };
    auto multiply = [&](auto which, int64_t kk) {
        constexpr int buf = decltype(which)::value;
        const bf16_t* la = lds + buf * SZ;
        const bf16_t* lb = la + PA * SZA;
        const int left = (int)(k_len - kk < KC ? k_len - kk : KC);
#pragma unroll
        for (int t = 0; t < KC / kStep; ++t) {
            if (t * kStep < left) {
                OpFrag<RA, LA, PA, SZA> af[MT];
                OpFrag<RB, LB, PB, SZB> bf[NT];
#pragma unroll
                for (int i = 0; i < MT; ++i) af[i].read(la, (wm * MT + i) * 32, t * kStep, lane);
#pragma unroll
                for (int j = 0; j < NT; ++j) bf[j].read(lb, (wn * NT + j) * 32, t * kStep, lane);
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) {
                        plane_products<PA, PB>(af[i].v, bf[j].v, sums[0][i][j], sums[SUMS - 1][i][j]);
                    }
            }
        }
    };
    // chunk c is multiplied from LDS buffer c % 2; chunk c + 1 goes there from its registers at the end of step c, and
    // chunk c + 3 is requested into the registers so freed
    fetch(s0, 0);
    fetch(s1, KC);
    put(s0, 0);
    fetch(s0, 2 * KC);
    lds_barrier();
    for (int64_t kk = 0; kk < k_len; kk += 2 * KC) {
        multiply(std::integral_constant<int, 0>(), kk);
        if (kk + KC >= k_len) break;
        put(s1, 1);
        fetch(s1, kk + 3 * KC);
        lds_barrier();
        multiply(std::integral_constant<int, 1>(), kk + KC);
        if (kk + 2 * KC >= k_len) break;
        put(s0, 0);
        fetch(s0, kk + 4 * KC);
        lds_barrier();
    }

    auto& acc = sums[0];
    if constexpr (SUMS > 1) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc[i][j][r] += sums[1][i][j][r];
                }
    }
    if constexpr (kSplit) {
        const bool off = planes_overflowed(acc);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] *= kPlaneUnscale<PA / 3 + PB / 3>;
        if (off) op_redo<TA, TB>(d, g, m0, n0, mlim, nlim, wm, wn, k_lo, k_len, lane, acc);
    }
    op_store<TO, PARTIAL, MT, NT>(d, acc, outer, g, m0, n0, mlim, nlim, wm, wn, lane);
}

template <class G>
__global__ void __launch_bounds__(G::kThreads, 2)
ops_gemm_kernel(const OpDesc d)
{
    extern __shared__ __align__(16) unsigned char op_lds[];
    G::run(d, (int)blockIdx.x, op_lds);
}
// two contractions, the workgroups of the second behind those of the first
template <class G0, class G1>
__global__ void __launch_bounds__(G0::kThreads, 2)
ops_gemm_pair_kernel(const OpDesc d0, const OpDesc d1)
{
    extern __shared__ __align__(16) unsigned char op_lds[];
    const int bid = (int)blockIdx.x;
    const bool second = bid >= d0.blocks;
    if constexpr (std::is_same<G0, G1>::value) {
        const OpDesc& d = second ? d1 : d0;
        G0::run(d, second ? bid - d0.blocks : bid, op_lds);
    } else {
        if (second) G1::run(d1, bid - d0.blocks, op_lds);
        else G0::run(d0, bid, op_lds);
    }
}

// ---- long batches: the weights as planes, laid out once per call ----
//
// A workgroup has 64 rows of four neighbouring blocks, two waves a block, each with half of the columns of its tile (64
// NT).  The rows are split on their way into LDS, once for all columns of the tile, and interleaved blocks are read and
// written in whole lines; the weights come as planes in fragment order (ops_planes_kernel) straight into registers, a
// K-step ahead, so that nothing but the rows is split in the loop and nothing but the rows passes through LDS.  The sums
// are those of OpGemm, in the same order: a call that takes this kernel gives the same bits.
// 768 -> 768 fp32, 12608 rows, per contraction: 42 to 50 us in 64 x 64 tiles, 33 here (37 with interleaved rows).  Of
// these the matrix cores alone take 16 (six products, 197 of 256 CUs, the clock that ordinary numbers leave them), storing
// the results, which nothing overlaps with one workgroup to a CU, 9, the first rows and the launch 5.
struct PlaneJob {
    const void* src;
    bf16_t* dst;    // [g][tile of 32 rows n][K-step][plane][lane][8]
    int N, K, n_s, k_s;  // element (g, n, k) at g*N*K + n*n_s + k*k_s
    int tiles_n, steps, blocks;
};
// CW > 0: workgroups behind those of the weights run the first pass of the bias gradient, CW columns to a lane
template <typename T, int CW>
__global__ void __launch_bounds__(256)
ops_planes_kernel(const PlaneJob j0, const PlaneJob j1, const PlaneJob j2, int G, const ColsumJob cj)
{
    constexpr int PL = sizeof(T) == 4 ? 3 : 1;
    const int b01 = j0.blocks + j1.blocks, b012 = b01 + j2.blocks, block = (int)blockIdx.x;
    if constexpr (CW > 0) {
        if (block >= b012) {
            colsum_partial_body<T, CW>(cj, block - b012);
            return;
        }
    }
    const PlaneJob j = block < j0.blocks ? j0 : block < b01 ? j1 : j2;
    const int bid = block < j0.blocks ? block : block < b01 ? block - j0.blocks : block - b01;
    const int idx = bid * 256 + (int)threadIdx.x, lane = idx & 63, tile = idx >> 6;
    const int ks = tile % j.steps, nt = tile / j.steps % j.tiles_n, g = tile / j.steps / j.tiles_n;
    if (g >= G) return;
    const int n = nt * 32 + (lane & 31), k0 = ks * kStep + 8 * (lane >> 5);
    const T* const p = static_cast<const T*>(j.src) + (size_t)g * j.N * j.K + (size_t)n * j.n_s + (size_t)k0 * j.k_s;
    T v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = n < j.N && k0 + e < j.K ? p[(size_t)e * j.k_s] : T(0);
    bf16_t* const to = j.dst + ((size_t)tile * PL * 64 + lane) * 8;
    u32x4 o[PL];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if constexpr (PL == 3) {
            uint32_t s[3];
            split3(__float_as_uint(v[2 * w]), __float_as_uint(v[2 * w + 1]), s);
#pragma unroll
            for (int u = 0; u < 3; ++u) o[u][w] = s[u];
        } else {
            o[0][w] = (uint32_t)v[2 * w] | (uint32_t)v[2 * w + 1] << 16;
        }
    }
#pragma unroll
    for (int u = 0; u < PL; ++u) *reinterpret_cast<u32x4*>(to + (size_t)u * 512) = o[u];
}

constexpr int kRows = 64, kRowsThreads = 512;
// 64 rows x 32 of an operand whose blocks are interleaved (element (g, k) at k*G + g), on their way to LDS: a thread has
// four k of a row for four neighbouring blocks, in pieces of four elements, and turns them in registers.
template <typename T, int LSTR, int SZ>
struct QuadTile {
    static constexpr int kWords = sizeof(T);  // dwords of a piece
    u32x4 r[sizeof(T)];  // fp32: a piece each; bf16: two
    __device__ __forceinline__ void fetch(const T* base, uint32_t os, uint32_t cs, int olim, int clim, int tid)
    {
        const int o = tid >> 3, c = (tid & 7) * 4;
        const auto rs = buffer_at(base);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const uint32_t at = o < olim && c + n < clim ? (o * os + (c + n) * cs) * (uint32_t)sizeof(T) : kNowhere;
            if constexpr (sizeof(T) == 4) {
                r[n] = __builtin_amdgcn_raw_buffer_load_b128(rs, at, 0, 0);
            } else {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, at, 0, 0);
                r[n >> 1][2 * (n & 1)] = v[0];
                r[n >> 1][2 * (n & 1) + 1] = v[1];
            }
        }
    }
    // lds: the first of four slots, `slot` elements apart
    __device__ __forceinline__ void store(bf16_t* lds, int slot, int tid) const
    {
        bf16_t* const to = lds + (tid >> 3) * LSTR + (tid & 7) * 4;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if constexpr (sizeof(T) == 4) {
                uint32_t lo[3], hi[3];
                split3(r[0][g], r[1][g], lo);
                split3(r[2][g], r[3][g], hi);
#pragma unroll
                for (int w = 0; w < 3; ++w) *reinterpret_cast<u32x2*>(to + g * slot + w * SZ) = u32x2{lo[w], hi[w]};
            } else {
                const uint32_t a = r[0][g >> 1], b = r[0][2 + (g >> 1)], c = r[1][g >> 1], e = r[1][2 + (g >> 1)];
                *reinterpret_cast<u32x2*>(to + g * slot) = g & 1 ? u32x2{pick_hi16(a, b), pick_hi16(c, e)} : u32x2{pick_lo16(a, b), pick_lo16(c, e)};
            }
        }
    }
};

// A finished workgroup's results, eight rows of its four blocks at a time, by way of LDS, so that what lies side by side
// in memory leaves together: kTurnNone, four columns of a block; kTurnBlocks, the four blocks of a column (element (g, n)
// at n*G + g); kTurnMid, four columns G apart of a block (the stage-1 position of the permuted vector), kTurnMidAny, one
// of them, a lane the next.  Straight from the accumulators (kTurnDirect) single elements leave, G or more apart: 768 ->
// 768 fp32, 12608 rows, 44 to 50 us for a contraction that takes 34 this way.
enum Turn { kTurnDirect, kTurnNone, kTurnBlocks, kTurnMid, kTurnMidAny };
template <typename TO, int NT>
struct RowsStore {
    static constexpr int NW = 64 * NT, STR = NW + 4, TILE = 8 * 4 * STR;
    static constexpr size_t kLds = 2 * sizeof(float) * (size_t)TILE;
    // E: elements of a piece
    template <int E>
    static __device__ __forceinline__ void run(const OpDesc& d, const f32x16 (&acc)[2][NT], int g0, int tn, int64_t m0, int mlim, int slot, int half,
                                               int tid, int lane, float* lds)
    {
        constexpr int U = 4 * NT / E, PB = NW / E;  // pieces of a thread and of a block's eight rows / 8
        const int col = half * (NT * 32) + (lane & 31), h = lane >> 5, G = d.G, step = d.o_turn == kTurnBlocks ? STR : d.o_turn == kTurnMid ? G : 1;
        const auto out = buffer_at(static_cast<TO*>(d.o) + m0 * d.o_m), bias = buffer_at(d.bias);
        int from[U], row[U];  // place in LDS; row of the eight (kRows: a piece that does not exist)
        uint32_t to[U];
        float add[U][E];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = tid + u * kRowsThreads, r = idx / (4 * PB), rest = idx % (4 * PB);
            int c = rest / PB, n = rest % PB * E;
            if (d.o_turn == kTurnBlocks) {
                c = 0;
                n = rest;
            } else if (d.o_turn != kTurnNone) {
                const int w = NW / G / E, t = rest % PB;
                n = t % w * (E * G) + t / w;
            }
            const int g = g0 + c, at = tn * NW + n;
            from[u] = (r * 4 + c) * STR + n;
            row[u] = at < d.N ? r : kRows;
            if (d.o_turn >= kTurnMid) {
                const uint32_t f = (uint32_t)(g * d.N + at);
                to[u] = f % (uint32_t)G * (uint32_t)d.N + f / (uint32_t)G;
            } else {
                to[u] = (uint32_t)g * (uint32_t)d.o_g + (uint32_t)at * (uint32_t)d.o_n;
            }
#pragma unroll
            for (int e = 0; e < E; ++e) add[u][e] = 0.f;
            if (E == 4 && d.bias) {
                const uint32_t b = row[u] < kRows ? to[u] * (uint32_t)sizeof(TO) : kNowhere;
                if constexpr (sizeof(TO) == 4) {
                    const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(bias, b, 0, 0));
#pragma unroll
                    for (int e = 0; e < E; ++e) add[u][e] = v[e];
                } else {
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(bias, b, 0, 0);
#pragma unroll
                    for (int e = 0; e < E; ++e) add[u][e] = __uint_as_float(e & 1 ? v[e >> 1] & 0xffff0000u : v[e >> 1] << 16);
                }
            }
        }
        lds_barrier();  // the last chunk has been read
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            float* const tile = lds + (s & 1) * TILE;
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) tile[((4 * h + e) * 4 + slot) * STR + col + j * 32] = acc[s >> 2][j][4 * (s & 3) + e];
            lds_barrier();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float* const p = tile + from[u];
                const int m = s * 8 + row[u];
                const uint32_t at = m < mlim ? ((uint32_t)m * (uint32_t)d.o_m + to[u]) * (uint32_t)sizeof(TO) : kNowhere;
                if constexpr (E == 1) {
                    static_assert(E != 1 || sizeof(TO) == 4, "between the factors");
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(p[0]), out, at, 0, 0);
                } else {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < E; ++e) v[e] = p[e * step] + add[u][e];
                    if constexpr (sizeof(TO) == 4) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), out, at, 0, 0);
                    else __builtin_amdgcn_raw_buffer_store_b64(u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])}, out, at, 0, 0);
                }
            }
        }
    }
};

template <typename TA, typename TB, typename TO, int NT, Take AV, bool QUAD>
struct RowsGemm {
    static constexpr bool kSplit = sizeof(TA) == 4 || sizeof(TB) == 4;
    static constexpr int PA = sizeof(TA) == 2 ? 1 : 3, PB = sizeof(TB) == 2 ? 1 : 3;
    // chunks of 16 indices where that lets a second workgroup on the CU (49 x 49 blocks bf16, 32768 rows: 17 and 15 us)
    static constexpr int KC = PA == 3 && NT == 1 && !QUAD ? 16 : 32, LSTR = KC + 8, SZ = kRows * LSTR, SLOT = PA * SZ, BUF = 4 * SLOT;
    static constexpr size_t kLds = std::max(2 * sizeof(bf16_t) * (size_t)BUF, RowsStore<TO, NT>::kLds);
};
template <typename TA, typename TB, typename TO, int NT, Take AV, bool QUAD>
__global__ void __launch_bounds__(kRowsThreads, 2)
ops_rows_kernel(const OpDesc d, const bf16_t* __restrict__ planes, int steps)
{
    using S = RowsGemm<TA, TB, TO, NT, AV, QUAD>;
    constexpr int PA = S::PA, PB = S::PB, KC = S::KC, MT = 2, NF = NT * PB;
    static_assert(!QUAD || KC == 32, "the tile of QuadTile");
    using TileA = std::conditional_t<QUAD, QuadTile<TA, S::LSTR, S::SZ>, OpTile<TA, KC, kRows, S::LSTR, AV, S::SZ, 128>>;
    extern __shared__ __align__(16) unsigned char op_lds[];
    bf16_t* const lds = reinterpret_cast<bf16_t*>(op_lds);

    const int inner = d.G / 4 * d.tiles_n, bid = (int)blockIdx.x, seq = d.deal ? bid >> 3 : bid;
    const int tm = d.deal ? (seq / inner) * 8 + (bid & 7) : seq / inner;
    if (tm >= d.nouter) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), slot = wave >> 1, half = wave & 1;
    const int g0 = seq % inner % (d.G / 4) * 4, g = g0 + slot, tn = seq % inner / (d.G / 4);
    const int64_t m0 = (int64_t)tm * kRows;
    const int n0 = tn * (64 * NT), K = (int)d.K;
    const int mlim = d.M - m0 < kRows ? (int)(d.M - m0) : kRows, nlim = d.N - n0 < 64 * NT ? d.N - n0 : 64 * NT;

    // rows: the 128 threads of a slot have its block; QUAD: all threads have the four blocks of the workgroup
    const TA* pa = static_cast<const TA*>(d.a.p) + (QUAD ? g0 : g) * d.a.g_s + m0 * d.a.r_s;
    TileA s0, s1;
    // requests stay where they are written: moved to their use, as the compiler would, they are waited for at once
    auto pin = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto fetch = [&](TileA& s, int kk) {
        const int left = K - kk, klim = left < KC ? (left > 0 ? left : 0) : KC;
        s.fetch(pa + (int64_t)kk * d.a.k_s, (uint32_t)d.a.r_s, QUAD ? (uint32_t)d.a.k_s : 1u, mlim, klim, QUAD ? tid : tid & 127);
        pin();
    };
    auto put = [&](const TileA& s, int buf) {
        if constexpr (QUAD) s.store(lds + buf * S::BUF, S::SLOT, tid);
        else s.store(lds + buf * S::BUF + slot * S::SLOT, tid & 127);
    };
    // fragments of a K-step: tiles past the last column take the last one's
    const int nt_all = (d.N + 31) / 32;
    uint32_t w_at[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int nt = tn * 2 * NT + half * NT + j, in = nt < nt_all ? nt : nt_all - 1;
        w_at[j] = (uint32_t)(((g * nt_all + in) * steps) * PB) * 1024u;
    }
    const auto rw = buffer_at(planes);
    u32x4 w0[NF], w1[NF];
    auto load = [&](u32x4 (&w)[NF], int ks) {
        const uint32_t at = (uint32_t)(ks < steps ? ks : steps - 1) * (PB * 1024u);
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int u = 0; u < PB; ++u) w[j * PB + u] = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16u, w_at[j] + at + u * 1024u, 0);
        pin();
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    auto multiply = [&](const u32x4 (&w)[NF], int buf, int t) {
        OpFrag<false, S::LSTR, PA, S::SZ> af[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) af[i].read(lds + buf * S::BUF + slot * S::SLOT, i * 32, t * kStep, lane);
        // the order of plane_products in every tile
#pragma unroll
        for (int v = 2; v >= 0; --v)
#pragma unroll
            for (int u = 0; u <= v; ++u)
                if (u < PA && v - u < PB) {
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < NT; ++j)
                            acc[i][j] = mfma32(af[i].v[u < PA ? u : 0], as_bf16x8(w[j * PB + (v - u < PB ? v - u : 0)]), acc[i][j]);
                }
        __builtin_amdgcn_sched_barrier(0);
    };
    load(w0, 0);
    fetch(s0, 0);
    fetch(s1, KC);
    put(s0, 0);
    lds_barrier();
    // a chunk that is not the last one; fragments of the next K-step, then rows, whose wait leaves them in flight
    auto chunk = [&](auto which, TileA& mine, const TileA& next, u32x4 (&even)[NF], u32x4 (&odd)[NF], int kk) {
        constexpr int buf = decltype(which)::value;
        load(odd, kk / kStep + 1);
        fetch(mine, kk + 2 * KC);
        multiply(even, buf, 0);
        if constexpr (KC > kStep) {
            load(even, kk / kStep + 2);
            multiply(odd, buf, 1);
        }
        put(next, buf ^ 1);
        lds_barrier();
    };
    auto& w2 = KC > kStep ? w0 : w1;  // fragments of the second chunk of two
    auto& w3 = KC > kStep ? w1 : w0;
    int kk = 0, buf = 0;
    for (; kk + 2 * KC < K; kk += 2 * KC) {
        chunk(std::integral_constant<int, 0>(), s0, s1, w0, w1, kk);
        chunk(std::integral_constant<int, 1>(), s1, s0, w2, w3, kk + KC);
    }
    if (kk + KC < K) {
        chunk(std::integral_constant<int, 0>(), s0, s1, w0, w1, kk);
        kk += KC;
        buf = 1;
    }
    if constexpr (KC > kStep) {
        load(w1, kk / kStep + 1);
        multiply(w0, buf, 0);
        if (kStep < K - kk) multiply(w1, buf, 1);
    } else if (buf) {
        multiply(w1, 1, 0);
    } else {
        multiply(w0, 0, 0);
    }
    if constexpr (S::kSplit) {
        const bool off = planes_overflowed(acc);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] *= kPlaneUnscale<PA / 3 + PB / 3>;
        if (off) op_redo<TA, TB>(d, g, m0, n0, mlim, nlim, 0, half, 0, K, lane, acc);
    }
    float* const turn = reinterpret_cast<float*>(op_lds);
    if (d.o_turn == kTurnDirect) {
        op_store<TO, false, MT, NT>(d, acc, tm, g, m0, n0, mlim, nlim, 0, half, lane);
        return;
    }
    if constexpr (sizeof(TO) == 4) {
        if (d.o_turn == kTurnMidAny) {
            RowsStore<TO, NT>::template run<1>(d, acc, g0, tn, m0, mlim, slot, half, tid, lane, turn);
            return;
        }
    }
    RowsStore<TO, NT>::template run<4>(d, acc, g0, tn, m0, mlim, slot, half, tid, lane, turn);
}

// out[e] = sum over the batch chunks of P[z][e], for both gradients.  WAVES = 1: a thread per element.  WAVES > 1,
// for many chunks: a workgroup owns 64 elements, wave w adds the chunks w, w + WAVES, ..., the sums of the waves are
// added in order.  Workgroups from `blocks01` on run the second pass of the bias gradient.  Bound by latency: the
// 128 chunks of blocks of 49 x 49 and 64 x 49 took 11.7 us with a thread per element and the bias pass 6.7 us in a
// launch of its own, together 5.3; at 16 chunks of 192 x 192 a thread per element takes 5.1 us, 16 waves 13.
constexpr int kSumWaves = 16, kManyChunks = 32;
struct OpSum {
    const float* P;
    void* out;
    int64_t n;
    int nz;
};
template <typename OT, int WAVES>
__global__ void __launch_bounds__(WAVES > 1 ? WAVES * 64 : 256)
ops_sum_kernel(OpSum s0, OpSum s1, int64_t blocks0, int64_t blocks01, ColsumJob cj)
{
    constexpr int kOwn = WAVES > 1 ? 64 : 256;  // elements of a workgroup
    if ((int64_t)blockIdx.x >= blocks01) {
        colsum_final_body<OT, (WAVES > 1 ? WAVES * 64 : 256)>(cj, (int)((int64_t)blockIdx.x - blocks01));
        return;
    }
    const bool second = (int64_t)blockIdx.x >= blocks0;
    const OpSum& s = second ? s1 : s0;
    const int tx = threadIdx.x % kOwn, wave = threadIdx.x / kOwn;
    const int64_t i = ((int64_t)blockIdx.x - (second ? blocks0 : 0)) * kOwn + tx;
    const bool live = i < s.n;
    float v = 0.f;
    if (live) {
#pragma unroll 4
        for (int z = wave; z < s.nz; z += WAVES) v += s.P[z * s.n + i];
    }
    if constexpr (WAVES > 1) {
        __shared__ float part[WAVES - 1][64];
        if (wave > 0) part[wave - 1][tx] = v;
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int w = 0; w < WAVES - 1; ++w) v += part[w][tx];
    }
    if (live) Elem<OT>::store(static_cast<OT*>(s.out) + i, v);
}
template <typename OT>
int launch_sum(const OpSum& s0, const OpSum& s1, const ColsumJob* cj, hipStream_t st)
{
    const bool many = s0.nz >= kManyChunks;
    const int64_t own = many ? 64 : 256, b0 = (s0.n + own - 1) / own, b01 = b0 + (s1.n + own - 1) / own;
    const dim3 grid((unsigned)(b01 + (cj ? colsum_final_blocks(*cj) : 0)));
    const ColsumJob job = cj ? *cj : ColsumJob{};
    if (many) hipLaunchKernelGGL((ops_sum_kernel<OT, kSumWaves>), grid, dim3(kSumWaves * 64), 0, st, s0, s1, b0, b01, job);
    else hipLaunchKernelGGL((ops_sum_kernel<OT, 1>), grid, dim3(256), 0, st, s0, s1, b0, b01, job);
    return hip_status(hipGetLastError());
}

// ---- host side ----

// 16-byte pieces along the contiguous index need every other stride, the extent and the base to be multiples of a
// piece. Otherwise they are taken wherever they start (no extent is shorter than a piece: blocks have at least 16
// elements).
Take take_of(const void* p, int64_t s1, int64_t s2, int64_t contiguous_stride, int64_t extent, int esize)
{
    const int v = 16 / esize;
    if (contiguous_stride != 1) return kElements;
    return (uintptr_t)p % 16 == 0 && s1 % v == 0 && s2 % v == 0 && extent % v == 0 ? kPieces16 : kPiecesAny;
}

template <class G>
int launch_one(const OpDesc& d, hipStream_t st)
{
    auto kernel = ops_gemm_kernel<G>;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), G::kLds)) return hip_status(e);
    hipLaunchKernelGGL(kernel, dim3((unsigned)d.blocks), dim3(G::kThreads), G::kLds, st, d);
    return hip_status(hipGetLastError());
}
template <class G0, class G1>
int launch_pair(const OpDesc& d0, const OpDesc& d1, hipStream_t st)
{
    constexpr size_t lds = G0::kLds > G1::kLds ? G0::kLds : G1::kLds;
    auto kernel = ops_gemm_pair_kernel<G0, G1>;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds)) return hip_status(e);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(d0.blocks + d1.blocks)), dim3(G0::kThreads), lds, st, d0, d1);
    return hip_status(hipGetLastError());
}

using Cfg128x128 = OpCfg<2, 2, 2, 2>;
using Cfg128x96 = OpCfg<4, 1, 1, 3>;
using Cfg128x64 = OpCfg<2, 2, 2, 1>;
using Cfg64x64 = OpCfg<2, 2, 1, 1>;
using Cfg64x128 = OpCfg<2, 2, 1, 2>;
using Cfg192x192 = OpCfg<6, 2, 1, 3>;  // twelve waves
struct TileSize {
    int m, n;
};
constexpr int kTileSizes = 5;
constexpr TileSize kTiles[kTileSizes] = {{128, 128}, {128, 96}, {128, 64}, {64, 64}, {64, 128}};

// Chunks of 32 indices where planes are multiplied by no more workgroups than then run at the same time, one or two
// to a CU: nothing but the next chunks hides a chunk's way from memory there, and half as many take less time, with
// the same results bit for bit. x M in fp32, blocks of 256 and 1024, chunks of 16 and 32: 3000 rows 114.5 and 76.4
// us; x M^T, 40 rows 20.7 and 17.4, 2000 rows 51.2 and 49.1.  Beyond, chunks of 16 leave room for more workgroups
// (blocks of 40 x 128 and 128 x 257, k = 3, 8000 rows, x M: 31.0 and 43.6 us).
template <typename TA, typename TB, typename TO, class Cfg, bool RB, Take AV, Take BV>
int launch_chunks(const OpDesc& d, hipStream_t st)
{
    if constexpr (sizeof(TA) == 4 || sizeof(TB) == 4) {
        using Few = OpGemm<TA, TB, TO, OpCfg<Cfg::WM, Cfg::WN, Cfg::MT, Cfg::NT, 32>, false, RB, false, AV, BV>;
        if (d.blocks <= kCUs * (kMaxLdsBytes / 2 >= Few::kLds ? 2 : 1)) return launch_one<Few>(d, st);
    }
    return launch_one<OpGemm<TA, TB, TO, Cfg, false, RB, false, AV, BV>>(d, st);
}
template <typename TA, typename TB, typename TO, bool RB, Take AV, Take BV>
int launch_tile(int cfg, const OpDesc& d, hipStream_t st)
{
    if constexpr (AV != kElements) {
        switch (cfg) {
            case 0: return launch_chunks<TA, TB, TO, Cfg128x128, RB, AV, BV>(d, st);
            case 1: return launch_chunks<TA, TB, TO, Cfg128x96, RB, AV, BV>(d, st);
            case 2: return launch_chunks<TA, TB, TO, Cfg128x64, RB, AV, BV>(d, st);
        }
    } else if (cfg == 4) {
        return launch_chunks<TA, TB, TO, Cfg64x128, RB, AV, BV>(d, st);
    }
    return launch_chunks<TA, TB, TO, Cfg64x64, RB, AV, BV>(d, st);
}
// The two kinds of contraction of the data path with the ways of taking that occur: both operands in aligned pieces,
// both in pieces from anywhere, or A element by element (it is strided in the backward, and in the forward under
// MONARCH_FLAG_PERM_B).
template <typename TA, typename TB, typename TO>
int launch_op(bool w_rc, int cfg, const OpDesc& d, hipStream_t st)
{
    const bool aligned = d.b.take == kPieces16;
    if (!w_rc) {
        if (d.a.take == kElements) return launch_tile<TA, TB, TO, false, kElements, kPiecesAny>(cfg, d, st);
        return aligned && d.a.take == kPieces16 ? launch_tile<TA, TB, TO, false, kPieces16, kPieces16>(cfg, d, st)
                                                : launch_tile<TA, TB, TO, false, kPiecesAny, kPiecesAny>(cfg, d, st);
    }
    if (d.a.take == kElements) {
        return aligned ? launch_tile<TA, TB, TO, true, kElements, kPieces16>(cfg, d, st)
                       : launch_tile<TA, TB, TO, true, kElements, kPiecesAny>(cfg, d, st);
    }
    return aligned && d.a.take == kPieces16 ? launch_tile<TA, TB, TO, true, kPieces16, kPieces16>(cfg, d, st)
                                            : launch_tile<TA, TB, TO, true, kPiecesAny, kPiecesAny>(cfg, d, st);
}
// dL from dy and U, dR from dU and x: T is the layer's type, U and dU are fp32
template <typename T, class Cfg, Take AV, Take BV>
int launch_wgrad_tile(const OpDesc& d0, const OpDesc& d1, hipStream_t st)
{
    return launch_pair<OpGemm<T, float, float, Cfg, true, true, true, kElements, BV>, OpGemm<float, T, float, Cfg, true, true, true, AV, BV>>(d0, d1, st);
}
template <typename T, Take AV, Take BV>
int launch_wgrad_take(int cfg, const OpDesc& d0, const OpDesc& d1, hipStream_t st)
{
    switch (cfg) {
        case 0: return launch_wgrad_tile<T, Cfg64x64, AV, BV>(d0, d1, st);
        case 1: return launch_wgrad_tile<T, Cfg128x128, AV, BV>(d0, d1, st);
        default: return launch_wgrad_tile<T, Cfg192x192, AV, BV>(d0, d1, st);
    }
}
template <typename T>
int launch_wgrad(int cfg, const OpDesc& d0, const OpDesc& d1, hipStream_t st)
{
    const Take b = d0.b.take < d1.b.take ? d0.b.take : d1.b.take;
    if (b == kElements) return launch_wgrad_take<T, kElements, kElements>(cfg, d0, d1, st);
    return b == kPieces16 && d1.a.take == kPieces16 ? launch_wgrad_take<T, kPieces16, kPieces16>(cfg, d0, d1, st)
                                                     : launch_wgrad_take<T, kPiecesAny, kPiecesAny>(cfg, d0, d1, st);
}

int64_t tiles(int64_t n, int t) { return (n + t - 1) / t; }

// The tile that finishes first under a simple model: up to 256 workgroups run one per CU; beyond, rounds of two per CU
// that share it.  A workgroup costs its (padded) tile plus a fixed share for filling and draining the pipeline.
// Operands taken element by element keep to 64 rows, whose workgroups hold more of the strided loads in flight, and
// to 128 columns where there are more than 64, since every column tile loads them again (1024 -> 4096 fp32, 8000
// rows: step 559 us with 64 x 64, 521 with 64 x 128, 560 with 128 x 64).  Not where 128 columns would leave half of
// the CUs idle (x M, blocks of 256 and 1024, 40 rows: 55.2 us with 64 x 128, 41.6 with 64 x 64; from there up to a
// workgroup per CU it depends: 192 of them, blocks of 256 and 1024, 60.0 and 54.3 us, blocks of 96 19.1 and 21.3).
int pick_tile(int64_t M, int N, int G, bool pieces)
{
    if (!pieces) return N > 64 && tiles(M, 64) * tiles(N, 128) * G > kCUs / 2 ? 4 : 3;
    int best = 3;
    double best_t = 1e30;
    for (int c = 0; c < 4; ++c) {
        const double wgs = (double)tiles(M, kTiles[c].m) * tiles(N, kTiles[c].n) * G;
        const double pairs = wgs / 512, rounds = wgs <= 256 ? 0.5 : pairs < 4 ? (double)((int64_t)(pairs + 0.999)) : pairs;
        const double t = rounds * (kTiles[c].m * kTiles[c].n + 2048);
        if (t < best_t) {
            best_t = t;
            best = c;
        }
    }
    return best;
}

// What a contraction reads and writes: the rows of the blocks interleaved on the way in or out, or on neither side.
enum Sides { kPlain, kSpreadOut, kSpreadIn };
// Columns per wave (NT tiles of 32) of the kernel with the weights laid out as planes.
int rows_tile(int N) { return N <= 64 ? 1 : tiles(N, 192) * 192 <= tiles(N, 128) * 128 ? 3 : 2; }
// Where that kernel gains.  It reads and writes an interleaved side in whole lines and splits a row once instead of
// once per 64 columns; its workgroups run one to a CU, so that it loses where the last round of them is far from full,
// and the weights are a launch of 3 to 5 us before it.  us, contractions of 64-column tiles first: 768 -> 768 fp32 x
// M^T 12608 rows 80 and 67, 8192 rows (half a round) 47 and 58; x M 83 and 73; 768 -> 3072 12608 rows 166 and 155, x M
// 182 and 140; 1024 -> 1024 fp32 x M^T 16384 rows (two rounds of 128 columns) 133 and 126, 8192 rows and 1024 -> 4096
// at 2048 (one round) 70 and 67, 50 and 55; with 96 of 128 columns: 384 -> 384 16384 rows 36 and 45; 40 x 33 blocks, k
// = 8, bf16, 16384 rows 29 and 20, x M 35 and 25; in fp32 x M 22 and 26 at 8192 rows.
// kBeside: where it gains less than the launch costs, another contraction of the call has to share it, which takes no
// more time for it.  Those are the ones with neither side interleaved (fp32, four blocks, 12608 rows: 132 x 16, alone
// in the call, 18 and 23; 16384 rows, 160 x 72 41 and 47; beside another, 12608 rows, 170 x 180 82 and 76; two rounds
// of them no better than 64-column tiles there either, more than one column tile worse, 3072 -> 768 x M 146 and 163;
// bf16 with fp32 rows gains alone where the round is nearly full, 14000 rows, 150 x 120 40 and 35), one round of 64
// columns (bf16, four blocks of 49 x 49, 16384 rows 22 and 27, of 60 x 80 21 and 28; both contractions of sixteen of 56
// x 56, 4096 rows, 37 and 22), and the second factor of bf16 layers with four blocks in 128 columns (240 x 200, 24000
// rows 83 and 94; beside another, 128 x 128, 32768 rows 55 and 54).
enum Gain { kNever, kBeside, kAlone };
Gain rows_gain(const Problem& pb, int N, int K, Sides sides, bool wide)  // wide: the rows are fp32
{
    if (pb.k % 4) return kNever;
    const int nt = rows_tile(N);
    const bool bf16 = pb.dtype == 1;
    const int64_t cols = tiles(N, 64 * nt), wgs = tiles(pb.B, kRows) * (pb.k / 4) * cols, slots = tiles(wgs, kCUs) * kCUs;
    const bool full = 10 * wgs >= 9 * slots, rounds = slots > kCUs;
    if (nt == 3) {
        if (4 * wgs < 3 * slots) return kNever;
        if (sides != kPlain) return kAlone;
        if (cols > 1 || rounds) return kNever;
        return bf16 && wide && K >= 40 && 5 * wgs >= 4 * slots ? kAlone : kBeside;
    }
    if (!full) return kNever;
    if (nt == 1) {
        if ((N <= 48 && pb.k <= 4) || (!bf16 && sides != kSpreadOut)) return kNever;
        return sides != kPlain && (rounds || (sides == kSpreadIn && pb.k > 4)) ? kAlone : kBeside;
    }
    if (sides == kPlain || !rounds || 5 * N < 4 * 128 * cols) return kNever;
    return bf16 && wide && sides == kSpreadOut && pb.k == 4 ? kBeside : kAlone;
}
// a weight (k blocks, N x K) as planes, bytes
size_t plane_bytes(const Problem& pb, int N, int K)
{
    return (size_t)pb.k * (size_t)tiles(N, 32) * (size_t)tiles(K, kStep) * (pb.dtype == 0 ? 3 : 1) * 1024;
}
struct Planes {  // of the weights of one call, in its workspace; those the call has no use for are null
    bf16_t* w[3] = {nullptr, nullptr, nullptr};
    PlaneJob job[3] = {};
    int n = 0;
    int gain = 0;  // kAlone, or the sum of several kBeside: the launch pays
    size_t bytes = 0;
    // the next weight, element (g, n, k) at g*N*K + n*n_s + k*k_s
    void add(const Problem& pb, const void* src, int N, int K, int n_s, int k_s, Sides sides, bool wide)
    {
        const size_t b = plane_bytes(pb, N, K);
        const Gain one = b < (1u << 30) ? rows_gain(pb, N, K, sides, wide) : kNever;
        if (one) {
            PlaneJob& j = job[n];
            j = PlaneJob{src, reinterpret_cast<bf16_t*>(bytes), N, K, n_s, k_s, (int)tiles(N, 32), (int)tiles(K, kStep), 0};
            j.blocks = (int)tiles((int64_t)pb.k * j.tiles_n * j.steps, 4);
            bytes += b;
        }
        gain += one;
        ++n;
    }
    Planes done() const { return gain >= kAlone ? *this : Planes{}; }
    // `at`: room for them, or null; cj (may be null): the first pass of the bias gradient with them
    int launch(const Problem& pb, void* at, const ColsumJob* cj, hipStream_t st)
    {
        const int blocks = at ? job[0].blocks + job[1].blocks + job[2].blocks : 0;
        if (!blocks) return cj ? launch_colsum_partial(pb, *cj, st) : 0;
        for (int i = 0; i < n; ++i)
            if (job[i].blocks) w[i] = job[i].dst = reinterpret_cast<bf16_t*>(static_cast<char*>(at) + reinterpret_cast<size_t>(job[i].dst));
        const int cw = cj ? rowcol_cw(cj->n_out) : 0;
        auto kernel = pb.dtype == 0 ? (cw == 4 ? ops_planes_kernel<float, 4> : cw ? ops_planes_kernel<float, 1> : ops_planes_kernel<float, 0>)
                                    : (cw == 4 ? ops_planes_kernel<bf16_t, 4> : cw ? ops_planes_kernel<bf16_t, 1> : ops_planes_kernel<bf16_t, 0>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks + (cj ? colsum_partial_blocks(*cj) : 0))), dim3(256), 0, st, job[0], job[1], job[2], pb.k,
                           cj ? *cj : ColsumJob{});
        return hip_status(hipGetLastError());
    }
};

template <typename TA, typename TB, typename TO, int NT, Take AV, bool QUAD>
int launch_rows_one(const OpDesc& d, const bf16_t* planes, hipStream_t st)
{
    auto kernel = ops_rows_kernel<TA, TB, TO, NT, AV, QUAD>;
    constexpr size_t lds = RowsGemm<TA, TB, TO, NT, AV, QUAD>::kLds;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds)) return hip_status(e);
    hipLaunchKernelGGL(kernel, dim3((unsigned)d.blocks), dim3(kRowsThreads), lds, st, d, planes, (int)tiles(d.K, kStep));
    return hip_status(hipGetLastError());
}
template <typename TA, typename TB, typename TO, int NT>
int launch_rows_take(const OpDesc& d, const bf16_t* planes, hipStream_t st)
{
    switch (d.a.take) {
        case kElements: return launch_rows_one<TA, TB, TO, NT, kElements, true>(d, planes, st);
        case kPiecesAny: return launch_rows_one<TA, TB, TO, NT, kPiecesAny, false>(d, planes, st);
        default: return launch_rows_one<TA, TB, TO, NT, kPieces16, false>(d, planes, st);
    }
}
template <typename TA, typename TB, typename TO>
int launch_rows(int nt, const OpDesc& d, const bf16_t* planes, hipStream_t st)
{
    switch (nt) {
        case 1: return launch_rows_take<TA, TB, TO, 1>(d, planes, st);
        case 2: return launch_rows_take<TA, TB, TO, 2>(d, planes, st);
        default: return launch_rows_take<TA, TB, TO, 3>(d, planes, st);
    }
}

// Where the row tiles (batch chunks) do not come out even over the eight XCDs, whole ones per XCD would leave some of
// them idle: the workgroups are then numbered straight through.
void deal(OpDesc& d, int nouter, int inner)
{
    const int64_t even = tiles(nouter, 8) * 8;
    d.nouter = nouter;
    d.deal = 5 * even <= 6 * nouter;
    d.blocks = (int)((d.deal ? even : nouter) * inner);
}

// element (g, row, k) of an operand; `rc`: its row index is the contiguous one
OpOperand operand(const void* p, int64_t g_s, int64_t r_s, int64_t k_s, bool rc, int64_t rows, int64_t K, int esize)
{
    return OpOperand{p, g_s, r_s, k_s,
                     rc ? take_of(p, g_s, k_s, r_s, rows, esize) : take_of(p, g_s, r_s, k_s, K, esize)};
}

// One step of the data path: O (rows x blocks x N) = A x W per block; W, and one of A and O, are of the layer's type.
template <typename TA, typename TW, typename TO>
int data_op(const Problem& pb, const void* a, int64_t a_g, int64_t a_k, int64_t lda, int K, const void* w, bool w_rc, int N,
            const bf16_t* planes, void* o, int64_t o_g, int64_t o_n, int64_t ldo, const void* bias, hipStream_t st, bool o_mid = false)
{
    OpDesc d{};
    d.a = operand(a, a_g, lda, a_k, false, pb.B, K, sizeof(TA));
    d.b = w_rc ? operand(w, (int64_t)K * N, 1, N, true, N, K, sizeof(TW)) : operand(w, (int64_t)K * N, K, 1, false, N, K, sizeof(TW));
    d.o = o;
    d.o_g = o_g;
    d.o_m = ldo;
    d.o_n = o_n;
    d.o_mid = o_mid ? 1 : 0;
    d.bias = bias;
    d.M = pb.B;
    d.K = K;
    d.N = N;
    d.G = pb.k;
    d.k_chunk = K;
    if (planes) {
        const int nt = rows_tile(N);
        d.tiles_n = (int)tiles(N, 64 * nt);
        const bool whole = N % 4 == 0 && ldo % 4 == 0;  // pieces of four elements begin at multiples of their size
        if (o_mid) d.o_turn = whole && N % (4 * d.G) == 0 && 64 * nt % (4 * d.G) == 0 ? kTurnMid : 64 * nt % d.G == 0 ? kTurnMidAny : kTurnDirect;
        else if (o_n == 1) d.o_turn = whole && o_g % 4 == 0 ? kTurnNone : kTurnDirect;
        else d.o_turn = o_g == 1 && o_n == d.G && d.G % 4 == 0 ? kTurnBlocks : kTurnDirect;
        deal(d, (int)tiles(d.M, kRows), d.G / 4 * d.tiles_n);
        return launch_rows<TA, TW, TO>(nt, d, planes, st);
    }
    const int cfg = pick_tile(d.M, N, d.G, d.a.take != kElements);
    d.tiles_m = (int)tiles(d.M, kTiles[cfg].m);
    d.tiles_n = (int)tiles(N, kTiles[cfg].n);
    deal(d, d.tiles_m, d.tiles_n * d.G);
    return launch_op<TA, TW, TO>(w_rc, cfg, d, st);
}

// Tiles and batch chunks of the weight-gradient contractions.  64 x 64, about four workgroups per CU over both
// contractions (768 -> 768 fp32: 131 us with two, 104 with four; 128 x 64 gained nothing anywhere: 96 x 384 blocks,
// 4096 rows, backward 64 us and 73).  Larger tiles, 128 x 128 two to a CU and 192 x 192 (twelve waves) one to a CU,
// where they cover no more than the small ones and their chunks still have 256 rows: every value is split half or a
// third as often (768 -> 768 fp32, 12608 rows, both contractions 77 us in 64 x 64 tiles, 53 in 192 x 192, of which the
// matrix cores alone take 30; backward 176 and 152, at 1024 rows 41 and 48; 1024 -> 4096 in 128 x 128 tiles, 12608 rows
// 617 and 564, 4096 rows 212 and 201; 128 x 512 blocks, 4096 rows 83 and 94).  At least 128 rows each, and whole sets
// of eight, since a chunk belongs to an XCD (4096 -> 1024 fp32 with three chunks: three XCDs busy, 1088 us; with eight
// 465 us).  In steps of 32 rows: in steps of 64 the chunks were up to a fifth longer than an even share, and the launch
// waits for the longest (backward of 12 fp32 blocks of 48 x 48 and 48 x 192, 3231 rows 105 us and 85, of 12 of 80 x 80
// and 80 x 150 133 and 119; two of 64 shapes lost 3 and 5 %).  One set of eight small tiles stays in steps of 64: 32
// gain 1 to 3 % there, and a batch would ask for as much room as a slightly longer one.
struct WgradPlan {
    int cfg;
    int nz;
    int64_t rows;  // per chunk
};
constexpr int kWgradTiles[] = {64, 128, 192}, kWgradGroups[] = {4 * kCUs, 2 * kCUs, kCUs};
size_t part_bytes(const Problem& pb, int nz) { return align_up((size_t)nz * (pb.n_R() + pb.n_L()) * 4, 256); }
WgradPlan wgrad_plan(const Problem& pb, size_t room = SIZE_MAX)  // room: bytes for the partial sums; one chunk is the least
{
    const int M[2] = {pb.s, pb.q}, N[2] = {pb.q, pb.p};
    const int64_t rows = pb.B > 0 ? pb.B : 1, most = tiles(rows, 128);
    WgradPlan pl{};
    int64_t z = 1, least = 0;  // batch chunks; what the small tiles cover
    for (int c = 0; c < 3; ++c) {
        const int t = kWgradTiles[c];
        int64_t count = 0;
        for (int i = 0; i < 2; ++i) count += tiles(M[i], t) * tiles(N[i], t);
        int64_t nz = tiles(kWgradGroups[c], (int)(count * pb.k));
        if (nz > 1) nz = tiles(nz, 8) * 8;  // whole sets of the eight XCDs
        nz = std::min(nz, most);
        if (c == 0) least = count * t * t;
        if (c > 0 && (10 * count * t * t > 11 * least || rows < 256 * nz)) continue;
        pl.cfg = c;
        z = nz;
    }
    for (;; z = pl.nz - 1) {
        const int step = pl.cfg == 0 && z <= 8 ? 64 : 32;
        pl.rows = tiles(tiles(rows, (int)z), step) * step;
        pl.nz = (int)tiles(rows, (int)pl.rows);
        if (part_bytes(pb, pl.nz) <= room || pl.nz == 1) return pl;
    }
}

size_t mid_bytes(const Problem& pb) { return align_up((size_t)(pb.B > 0 ? pb.B : 1) * pb.kq() * sizeof(float), 256); }

// element strides of the vector between the factors: kept permuted (default reading) or in stage-1 order (PERM_B)
struct Mid {
    int64_t s1_g, s1_n;  // seen from stage 1: (kk, j)
    int64_t s2_g, s2_n;  // seen from stage 2: (c, r)
};
Mid mid(const Problem& pb)
{
    if (!pb.perm_b()) return Mid{1, pb.k, pb.q, 1};
    return Mid{pb.q, 1, 1, pb.k};
}

template <typename T>
int stage1(const Problem& pb, const void* x, const void* R, const bf16_t* planes, void* U, hipStream_t st)
{
    const Mid m = mid(pb);
    return data_op<T, T, float>(pb, x, pb.p, 1, pb.n_in, pb.p, R, false, pb.q, planes, U, m.s1_g, m.s1_n, pb.kq(), nullptr, st);
}
template <typename T>
int fwd_typed(const Problem& pb, const void* x, const void* R, const void* L, const Planes& pl, void* y, void* U, hipStream_t st)
{
    if (int rc = stage1<T>(pb, x, R, pl.w[0], U, st)) return rc;
    const Mid m = mid(pb);
    return data_op<float, T, T>(pb, U, m.s2_g, m.s2_n, pb.kq(), pb.q, L, false, pb.s, pl.w[1], y, 1, pb.k, pb.n_out(), pb.bias, st);
}
template <typename T>
int fwd_t_typed(const Problem& pb, const void* x, const void* R, const void* L, const Planes& pl, void* y, void* dU, hipStream_t st)
{
    // the vector between the factors in stage-1 order: written in short pieces once, read in long ones twice (dx, dR)
    if (int rc = data_op<T, T, float>(pb, x, 1, pb.k, pb.n_out(), pb.s, L, true, pb.q, pl.w[0], dU, 1, pb.k, pb.kq(), nullptr, st, !pb.perm_b()))
        return rc;
    return data_op<float, T, T>(pb, dU, pb.q, 1, pb.kq(), pb.q, R, true, pb.p, pl.w[1], y, pb.p, 1, pb.n_in, nullptr, st);
}

// The weights that the forward and the data path of the backward (recompute: with step 1 again) want as planes.
Planes fwd_planes(const Problem& pb, const void* R, const void* L)
{
    Planes pl;
    pl.add(pb, R, pb.q, pb.p, pb.p, 1, pb.perm_b() ? kPlain : kSpreadOut, pb.dtype == 0);
    pl.add(pb, L, pb.s, pb.q, pb.q, 1, pb.perm_b() ? kSpreadIn : kSpreadOut, true);
    return pl.done();
}
Planes fwd_t_planes(const Problem& pb, const void* R, const void* L, bool recompute)
{
    Planes pl;
    pl.add(pb, L, pb.q, pb.s, 1, pb.q, kSpreadIn, pb.dtype == 0);
    pl.add(pb, R, pb.p, pb.q, 1, pb.p, kPlain, true);
    if (recompute) pl.add(pb, R, pb.q, pb.p, pb.p, 1, pb.perm_b() ? kPlain : kSpreadOut, pb.dtype == 0);
    return pl.done();
}
int run_fwd_t(const Problem& pb, const void* x, const void* R, const void* L, const Planes& pl, void* y, void* dU, hipStream_t st)
{
    return pb.dtype == 0 ? fwd_t_typed<float>(pb, x, R, L, pl, y, dU, st) : fwd_t_typed<bf16_t>(pb, x, R, L, pl, y, dU, st);
}

}  // namespace

// Blocks below 16 would leave most of every 32 x 32 tile empty; the index arithmetic of a tile is 32-bit.
bool ops_supported(const Problem& pb)
{
    if (pb.flags & 4u) return false;  // MONARCH_FLAG_GENERIC: the SIMT kernels
    if (pb.p < 16 || pb.q < 16 || pb.s < 16) return false;
    if (pb.n_in > (1 << 20) || pb.kq() > (1 << 20) || pb.n_out() > (1 << 20)) return false;  // 32-bit offsets inside a tile
    const int64_t rows = pb.B > 0 ? pb.B : 1;
    const int widest = pb.p > pb.q ? (pb.p > pb.s ? pb.p : pb.s) : (pb.q > pb.s ? pb.q : pb.s);
    return (tiles(rows, 64) + 8) * tiles(widest, 32) * pb.k < (1LL << 30);
}

// The vector between the factors, then the weights as planes; with room for the vector alone (`least`) the weights are
// taken as they are, which gives the same bits.
size_t ops_fwd_workspace(const Problem& pb) { return mid_bytes(pb) + fwd_planes(pb, nullptr, nullptr).bytes; }
size_t ops_fwd_least(const Problem& pb) { return mid_bytes(pb); }

// U: the vector between the factors (mid_bytes), left there for ops_bwd; pb.ws_bytes from there on
int ops_fwd(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* U, hipStream_t st)
{
    Planes pl = fwd_planes(pb, R, L);
    if (int rc = pl.launch(pb, pb.ws_bytes >= mid_bytes(pb) + pl.bytes ? static_cast<char*>(U) + mid_bytes(pb) : nullptr, nullptr, st)) return rc;
    return pb.dtype == 0 ? fwd_typed<float>(pb, x, R, L, pl, y, U, st) : fwd_typed<bf16_t>(pb, x, R, L, pl, y, U, st);
}

size_t ops_fwd_t_workspace(const Problem& pb) { return mid_bytes(pb) + fwd_t_planes(pb, nullptr, nullptr, false).bytes; }
size_t ops_fwd_t_least(const Problem& pb) { return mid_bytes(pb); }

// y = x M: the dx path on its own
int ops_fwd_t(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* dU, hipStream_t st)
{
    Planes pl = fwd_t_planes(pb, R, L, false);
    if (int rc = pl.launch(pb, pb.ws_bytes >= mid_bytes(pb) + pl.bytes ? static_cast<char*>(dU) + mid_bytes(pb) : nullptr, nullptr, st)) return rc;
    return run_fwd_t(pb, x, R, L, pl, y, dU, st);
}

// U, dU, then the weights as planes, over which the partial sums of the weight gradients are written afterwards
size_t ops_bwd_workspace(const Problem& pb)
{
    const size_t part = part_bytes(pb, wgrad_plan(pb).nz), planes = fwd_t_planes(pb, nullptr, nullptr, true).bytes;
    return 2 * mid_bytes(pb) + (part > planes ? part : planes);
}
size_t ops_bwd_least(const Problem& pb) { return 2 * mid_bytes(pb) + part_bytes(pb, 1); }

int ops_bwd(const Problem& pb, const void* dy, const void* x, const void* R, const void* L, void* dx, void* dR, void* dL,
            void* ws, hipStream_t st)
{
    if (pb.B == 0) {
        const bool f = pb.wgrad_f32();
        int rc = f ? launch_fill_zero_f32((float*)dR, pb.n_R(), st) : launch_fill_zero_u16((uint16_t*)dR, pb.n_R(), st);
        if (rc) return rc;
        return f ? launch_fill_zero_f32((float*)dL, pb.n_L(), st) : launch_fill_zero_u16((uint16_t*)dL, pb.n_L(), st);
    }
    const WgradPlan pl = wgrad_plan(pb, pb.ws_bytes - 2 * mid_bytes(pb));
    Planes planes = fwd_t_planes(pb, R, L, !pb.saved);
    ColsumJob cj{};
    if (pb.dbias) cj = make_colsum_job(pb, dy, pb.dbias, pb.colsum_ws);
    const ColsumJob* bias_sum = pb.dbias ? &cj : nullptr;
    char* w = static_cast<char*>(ws);
    const void* U = pb.saved;
    if (int rc = planes.launch(pb, pb.ws_bytes >= 2 * mid_bytes(pb) + planes.bytes ? w + 2 * mid_bytes(pb) : nullptr, bias_sum, st)) return rc;
    if (!U) {
        if (int rc = pb.dtype == 0 ? stage1<float>(pb, x, R, planes.w[2], w, st) : stage1<bf16_t>(pb, x, R, planes.w[2], w, st)) return rc;
        U = w;
    }
    void* dU = w + mid_bytes(pb);
    if (int rc = run_fwd_t(pb, dy, R, L, planes, dx, dU, st)) return rc;

    const Mid m = mid(pb);
    const int e = (int)pb.esize();
    float* P = reinterpret_cast<float*>(w + 2 * mid_bytes(pb));
    OpDesc d[2] = {};
    d[0].a = operand(dy, 1, pb.k, pb.n_out(), true, pb.s, pb.B, e);
    d[0].b = operand(U, m.s2_g, m.s2_n, pb.kq(), true, pb.q, pb.B, sizeof(float));
    d[1].a = operand(dU, pb.q, 1, pb.kq(), true, pb.q, pb.B, sizeof(float));
    d[1].b = operand(x, pb.p, 1, pb.n_in, true, pb.p, pb.B, e);
    const int M[2] = {pb.s, pb.q}, N[2] = {pb.q, pb.p};
    for (int i = 0; i < 2; ++i) {
        d[i].o = i ? P + (size_t)pl.nz * pb.n_L() : P;
        d[i].M = M[i];
        d[i].N = N[i];
        d[i].K = pb.B;
        d[i].G = pb.k;
        d[i].tiles_m = (int)tiles(M[i], kWgradTiles[pl.cfg]);
        d[i].tiles_n = (int)tiles(N[i], kWgradTiles[pl.cfg]);
        d[i].k_chunk = pl.rows;
        deal(d[i], pl.nz, d[i].tiles_m * d[i].tiles_n * pb.k);
    }
    const int rc = pb.dtype == 0 ? launch_wgrad<float>(pl.cfg, d[0], d[1], st) : launch_wgrad<bf16_t>(pl.cfg, d[0], d[1], st);
    if (rc) return rc;
    const OpSum s0{P, dL, (int64_t)pb.n_L(), pl.nz}, s1{P + (size_t)pl.nz * pb.n_L(), dR, (int64_t)pb.n_R(), pl.nz};
    return pb.wgrad_f32() ? launch_sum<float>(s0, s1, bias_sum, st) : launch_sum<bf16_t>(s0, s1, bias_sum, st);
}

}  // namespace monarch
