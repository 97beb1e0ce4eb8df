// bf16 kernels for the square Monarch matrix of Definition 3.1 with m = 64 (n = 4096,
// k = q = s = p = 64): fused forward, and the backward data path.
//
// Per batch row the input is a 64 x 64 matrix X[kk][i].  Step 1 of Section 3.3 multiplies
// row kk by R[kk], the permutation turns the result Y1[kk][j] into U[c][r] = Y1[r][c], step 2
// multiplies row c of U (column c of Y1) by L[c], and step 3 writes y[l*64 + c] = W[c][l].  So
// every output block needs one column from every input block: a workgroup has to own whole rows,
// 8 KiB each in bf16.  A workgroup (8 waves) owns 32 rows.
//
// "Block stage": wave w multiplies blocks 8w .. 8w+7 of a block-diagonal factor with its rows and
// keeps the 32 x 512 results packed in registers (pairs of blocks per dword), because the full
// 256 KiB intermediate does not fit in LDS.  The intermediate is exchanged in two halves (output
// columns < 32, then >= 32): a half is written to LDS as T[b][col][block] (block fastest, 16-byte
// writes of the wave's eight blocks), which is exactly the operand order of the next factor for
// its block number `col`: the transposition P^T costs no data movement of its own.
//
// "Column stage": wave (cg, lt) multiplies the eight blocks 32h + 8cg .. +7 of the next factor,
// output rows 32lt .. 32lt+31, with the half in LDS.
//
// MFMA operands are loaded from global memory in operand layout.  Which contraction index sits
// in which K-slot is free as long as both operands agree, so lane group g of K-step u takes
// indices 32g + 8u .. +7: every lane then reads 64 contiguous bytes of its row.
// Everything that goes back to global memory is first transposed through LDS so that it is
// written in full 128-byte lines (16-byte pieces scattered over lines cost 2-3x the time).
//
// Backward (adjoints of steps 3, 2, P^T, 1; the paper leaves them to automatic differentiation,
// Section 4):
//   u           block stage (x, R) -> U to the workspace (dL needs it), unless the forward kept it
//   stage L     dy, U -> dU (to the workspace), dL's partial sums and the bias gradient's
//   stage R     dU, x -> dx and dR's partial sums        (both: bwd_sq64_stage_kernel)
//   reduce      the sums over the batch chunks (monarch_mfma_wgrad.hip)
// What bounds it: memory.  U, dU and the inputs are read and written 8 times in all (1.07 GB at 16384 rows); the
// transposed dy, dY1 and separate weight-gradient products that this replaced moved 1.47 GB (training step, 16384 rows:
// 379 -> 325 us; the backward alone 311 -> 260, at 1000 rows 61 -> 52, at 64 rows 51 -> 43).
// The transposed multiply transposes its input rows and runs both adjoint steps in one kernel.
#include "monarch_internal.h"
#include "monarch_mfma_common.h"
#include "monarch_mfma_stage1.h"
#include "monarch_lds_tr.h"
#include "monarch_colsum.h"

namespace monarch {

namespace {

constexpr int M64 = 64, N64 = 4096;
constexpr int SQ_BM = 32;                          // rows per workgroup
constexpr int SQ_ROWB = 32 * 128 + 16;             // bytes per row of the exchange buffer (32 cols x 64 blocks + pad)
constexpr size_t SQ_LDS = (size_t)SQ_BM * SQ_ROWB; // 131584 bytes

struct Lane {
    int wave, lane, ln, g;
};

// Block stage.  act: the lane's row, at column 32*g; W[block][out][in] (64 x 64 each).
// Results: bf16 pairs (block even, block odd) of T[b = ln][block][col], col = 32*jt + 8*(i/4) + 4*g + i%4.
// The half col < 32 goes to the exchange buffer as it is produced (LDS must be idle), the half
// col >= 32 is returned in pk1[i][t2].
// PACKED: W is the factor in fragment order (pack64_kernel): a weight operand is then one contiguous
// 1 KiB read per wave instruction instead of 32 lines touched twice.
template <bool PACKED>
__device__ __forceinline__ void block_stage(const Lane& t_, const uint16_t* __restrict__ act_row,
                                            const uint16_t* __restrict__ W, unsigned char* ldsb, u32x4 (&pk1)[16])
{
    const int wave = t_.wave, ln = t_.ln, g = t_.g;
    const uint16_t* arow = act_row + (size_t)wave * 8 * M64;
    const uint16_t* Wrow = PACKED ? W + ((size_t)wave * 8 * 8 * 64 + t_.lane) * 8
                                  : W + ((size_t)wave * 8 * M64 + ln) * M64 + 32 * g;
    u32x4 xa[2][4], ra[2][4];
    auto load_x = [&](int t, int s) {
#pragma unroll
        for (int u = 0; u < 4; ++u) xa[s][u] = ldg128(arow + t * M64 + 8 * u);
    };
    auto load_r = [&](int t, int jt) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            ra[jt][u] = PACKED ? ldg128(Wrow + (size_t)((t * 2 + jt) * 4 + u) * 512)
                               : ldg128(Wrow + ((size_t)t * M64 + 32 * jt) * M64 + 8 * u);
    };
    load_x(0, 0);
    load_r(0, 0);
    load_r(0, 1);
    f32x16 ev[2];
    u32x2 q0[16];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int s = t & 1;
        __builtin_amdgcn_sched_barrier(0);  // pins the prefetch distance
        if (t + 1 < 8) load_x(t + 1, s ^ 1);
#pragma unroll
        for (int jt = 0; jt < 2; ++jt) {
            __builtin_amdgcn_sched_barrier(0);
            f32x16 acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = mfma32(as_bf16x8(ra[jt][u]), as_bf16x8(xa[s][u]), acc);
            __builtin_amdgcn_sched_barrier(0);
            if (t + 1 < 8) load_r(t + 1, jt);
            if ((t & 1) == 0) {
                ev[jt] = acc;
            } else if (jt == 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i) pk1[i][t >> 1] = pack_bf16x2(ev[1][i], acc[i]);
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) q0[i][(t >> 1) & 1] = pack_bf16x2(ev[0][i], acc[i]);
                if ((t & 3) == 3) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int jl = 8 * (i >> 2) + 4 * g + (i & 3);
                        *reinterpret_cast<u32x2*>(ldsb + (size_t)ln * SQ_ROWB + jl * 128 + 16 * wave + 8 * (t >> 2)) =
                            q0[i];
                    }
                }
            }
        }
    }
}

// second half of the block-stage results -> exchange buffer
__device__ __forceinline__ void exchange_write(const Lane& t_, unsigned char* ldsb, const u32x4 (&pk1)[16])
{
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int jl = 8 * (i >> 2) + 4 * t_.g + (i & 3);
        *reinterpret_cast<u32x4*>(ldsb + (size_t)t_.ln * SQ_ROWB + jl * 128 + 16 * t_.wave) =
            pk1[i];
    }
}

// Column stage for half h: eight blocks c = 32h + 8cg + cc of W2[c][out][in], output tile lt.
// acc(cc) = D[out = 32*lt + 8*(i/4) + 4*g + i%4][b = ln]; `sink(cc, acc)` consumes it.
template <bool PACKED, typename Sink>
__device__ __forceinline__ void column_stage(const Lane& t_, const uint16_t* __restrict__ W2, const unsigned char* ldsb,
                                             int h, Sink&& sink)
{
    const int cg = t_.wave & 3, lt = t_.wave >> 2;
    const unsigned char* ub = ldsb + (size_t)t_.ln * SQ_ROWB + (8 * cg) * 128 + 64 * t_.g;
    // packed: fragment (block c, tile lt, K-step u) at ((c*2 + lt)*4 + u) * 512 elements, + lane * 8
    const uint16_t* Wrow = PACKED ? W2 + ((size_t)((32 * h + 8 * cg) * 2 + lt) * 4 * 64 + t_.lane) * 8
                                  : W2 + (((size_t)(32 * h + 8 * cg)) * M64 + 32 * lt + t_.ln) * M64 + 32 * t_.g;
    constexpr size_t BLK = PACKED ? 8 * 512 : (size_t)M64 * M64;  // elements between consecutive blocks c
    constexpr size_t KST = PACKED ? 512 : 8;                       // elements between consecutive K-steps u
    u32x4 la[2][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) la[0][u] = ldg128(Wrow + u * KST);
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) {
        const int s = cc & 1;
        __builtin_amdgcn_sched_barrier(0);
        if (cc + 1 < 8) {
#pragma unroll
            for (int u = 0; u < 4; ++u) la[s ^ 1][u] = ldg128(Wrow + (size_t)(cc + 1) * BLK + u * KST);
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const u32x4 ua = *reinterpret_cast<const u32x4*>(ub + cc * 128 + 16 * u);
            acc = mfma32(as_bf16x8(la[s][u]), as_bf16x8(ua), acc);
        }
        sink(cc, acc);
    }
}

// Column stage of the backward for half h, in place: wave w multiplies the four blocks c = 32h + 4w + cc of the packed
// factor W2 (both 32-row output tiles) with line (b, 4w + cc) of the exchange buffer and writes the 64 results over that
// same line: out[b][4w + cc][i], 128 bytes.  Every lane reads and writes its own row b = ln only and no other wave
// touches these four lines, so the order of one wave's LDS operations is all the synchronisation the overwrite needs;
// the results never wait in registers for the buffer to die (64 registers, which the kernel otherwise spills).
__device__ __forceinline__ void column_stage_inplace(const Lane& t_, const uint16_t* __restrict__ W2, unsigned char* ldsb, int h)
{
    unsigned char* line0 = ldsb + (size_t)t_.ln * SQ_ROWB + (4 * t_.wave) * 128;
    // fragment (block c, tile lt, K-step u) at ((c*2 + lt)*4 + u) * 512 elements, + lane * 8: the eight (block, tile)
    // steps of this wave are contiguous, n = 2*cc + lt
    const uint16_t* Wrow = W2 + ((size_t)(32 * h + 4 * t_.wave) * 2 * 4 * 64 + t_.lane) * 8;
    u32x4 la[2][4], ua[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) la[0][u] = ldg128(Wrow + (size_t)u * 512);
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        const int cc = n >> 1, lt = n & 1, s = n & 1;
        unsigned char* line = line0 + cc * 128;
        __builtin_amdgcn_sched_barrier(0);
        if (n + 1 < 8) {
#pragma unroll
            for (int u = 0; u < 4; ++u) la[s ^ 1][u] = ldg128(Wrow + (size_t)((n + 1) * 4 + u) * 512);
        }
        if (lt == 0) {  // the operand line is read once, before either tile's results are written over it
#pragma unroll
            for (int u = 0; u < 4; ++u) ua[u] = *reinterpret_cast<const u32x4*>(line + 64 * t_.g + 16 * u);
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = mfma32(as_bf16x8(la[s][u]), as_bf16x8(ua[u]), acc);
        // acc[i] = D[out = 32*lt + 8*(i/4) + 4*g + i%4][b = ln]
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
            *reinterpret_cast<u32x2*>(line + (32 * lt + 8 * i4 + 4 * t_.g) * 2) =
                u32x2{pack_bf16x2(acc[4 * i4], acc[4 * i4 + 1]), pack_bf16x2(acc[4 * i4 + 2], acc[4 * i4 + 3])};
    }
}

// Copies a 32 x 32-line LDS tile to global memory in full lines: wave w takes rows b = 4w..4w+3,
// 128 lines, eight per instruction (1 KiB contiguous).  Line (b, jl) goes to
// dst[(b0 + b) * 4096 + (col0 + jl) * 64 ..].  SWZ: tile rows are 4096 bytes and the 16-byte piece
// index is XOR-ed with b % 8; otherwise rows are SQ_ROWB bytes, pieces in order.
// BIAS: `add`, 64 values a line (line_bias), is added to the bf16 results.
template <bool SWZ, bool NT = SWZ, bool BIAS = false>
__device__ __forceinline__ void copy_out(const Lane& t_, const unsigned char* ldsb, uint16_t* __restrict__ dst,
                                         int64_t b0, int64_t B, int col0, const u32x4* add = nullptr)
{
#pragma unroll
    for (int k2 = 0; k2 < 16; ++k2) {
        const int line = 8 * k2 + (t_.lane >> 3), pc = t_.lane & 7;
        const int b = 4 * t_.wave + (line >> 5), jl = line & 31;
        const unsigned char* src = SWZ ? ldsb + (size_t)b * 4096 + jl * 128 + ((pc ^ (b & 7)) * 16)
                                       : ldsb + (size_t)b * SQ_ROWB + jl * 128 + pc * 16;
        u32x4 v = *reinterpret_cast<const u32x4*>(src);
        if constexpr (BIAS) {
#pragma unroll
            for (int w = 0; w < 4; ++w)
                v[w] = pack_bf16x2(__uint_as_float(v[w] << 16) + __uint_as_float(add[k2 & 3][w] << 16),
                                   __uint_as_float(v[w] & 0xffff0000u) + __uint_as_float(add[k2 & 3][w] & 0xffff0000u));
        }
        if (b0 + b < B) {
            uint16_t* p = dst + (b0 + b) * N64 + (size_t)(col0 + jl) * M64 + 8 * pc;
            if (NT) stg128_nt(p, v);  // final outputs: streamed; workspace copies stay cacheable for the next kernel
            else *reinterpret_cast<u32x4*>(p) = v;
        }
    }
}
// what a lane of copy_out adds to its lines: 8 of them apart, the same for every row
__device__ __forceinline__ void line_bias(const Lane& t_, const uint16_t* __restrict__ bias, int col0, u32x4 (&add)[4])
{
#pragma unroll
    for (int n = 0; n < 4; ++n) add[n] = ldg128(bias + (size_t)(col0 + 8 * n + (t_.lane >> 3)) * M64 + 8 * (t_.lane & 7));
}

__device__ __forceinline__ Lane make_lane()
{
    const int tid = threadIdx.x;
    Lane t;
    t.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    t.lane = tid & 63;
    t.ln = t.lane & 31;
    t.g = t.lane >> 5;
    return t;
}

// ------------------------------------------------------------------------ forward ----

// KEEP: the vector between the factors also goes to U, in the exchange layout, which is the one the backward reads.
// BIAS and KEEP are variants of their own: with tests of the pointers instead the plain forward took 0.6 to 2.4 us
// longer (packed, one row 16.6 us and 14.6, 16384 rows 68.2 and 66.3), and with a bias every line waited for its own.
template <bool PACKED, bool BIAS, bool KEEP>
__global__ void __launch_bounds__(512)
fwd_sq64_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ R, const uint16_t* __restrict__ L,
                const uint16_t* __restrict__ bias, uint16_t* __restrict__ y, uint16_t* __restrict__ U, int64_t B)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char ldsb[];
    const Lane t = make_lane();
    const int ln = t.ln, g = t.g;
    const int64_t b0 = (int64_t)blockIdx.x * SQ_BM;
    int64_t row = b0 + ln;
    row = row < B ? row : B - 1;  // rows past the end are computed from a valid row and dropped

    // step 1: Y1[b][kk][j] -> exchange layout T[b][j][kk]
    u32x4 pk1[16];  // pk1[i][t]: one 16-byte exchange piece per i, filled component by component
    block_stage<PACKED>(t, x + row * N64 + 32 * g, R, ldsb, pk1);

    // step 2 for the 32 blocks c = j of each half.
    // po[h][c2][i]: bf16 pair (c0 + 2*c2, c0 + 2*c2 + 1) of W[b = ln][c][l], c0 = 32h + 8cg,
    // l = 32*lt + 8*(i/4) + 4*g + i%4
    const int cg = t.wave & 3, lt = t.wave >> 2;
    uint32_t po[2][4][16];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h) {
            __syncthreads();  // step 2 of the first half has read everything it needs
            exchange_write(t, ldsb, pk1);
        }
        __syncthreads();
        if constexpr (KEEP) copy_out<false>(t, ldsb, U, b0, B, 32 * h);
        f32x16 ev;
        column_stage<PACKED>(t, L, ldsb, h, [&](int cc, const f32x16& acc) {
            if ((cc & 1) == 0) {
                ev = acc;
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) po[h][cc >> 1][i] = pack_bf16x2(ev[i], acc[i]);
            }
        });
    }

    // step 3: y[b][l*64 + c], transposed through LDS one 32-row tile of l per round.
    // LDS tile: [b][l][8 pieces of 16 B], piece index XOR-ed with b % 8 so that the writes of 8
    // adjacent lanes hit 8 different slots.
#pragma unroll
    for (int rnd = 0; rnd < 2; ++rnd) {
        u32x4 add[4];
        if constexpr (BIAS) line_bias(t, bias, 32 * rnd, add);
        __syncthreads();  // the exchange buffer (or the previous round's tile) is dead
        if (lt == rnd) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int l = 8 * (i >> 2) + 4 * g + (i & 3);
                    const int piece = (4 * h + cg) ^ (ln & 7);
                    *reinterpret_cast<u32x4*>(ldsb + (size_t)ln * 4096 + l * 128 + piece * 16) =
                        u32x4{po[h][0][i], po[h][1][i], po[h][2][i], po[h][3][i]};
                }
        }
        __syncthreads();
        copy_out<true, true, BIAS>(t, ldsb, y, b0, B, 32 * rnd, add);
    }
}

// ------------------------------------------------------------------------ pack ----

// A 64-block factor W[blk][out][in] (64 x 64 each) in MFMA fragment order, for one or two factors in
// one launch:  dst[blk][t2][u][lane][e] = W'[blk][32*t2 + lane%32][32*(lane/32) + 8*u + e], where W' = W,
// or W' = W^T per block (tr: the transposed multiply takes the transposed factors).  One thread = one
// 16-byte piece; 32768 pieces per factor.
struct Pack64Job { const uint16_t* src; uint16_t* dst; int tr; };
__global__ void __launch_bounds__(256)
pack64_kernel(Pack64Job j0, Pack64Job j1)
{
    const Pack64Job& j = blockIdx.x >> 7 ? j1 : j0;  // 128 workgroups of 256 pieces per factor
    const int pc = (blockIdx.x & 127) * 256 + threadIdx.x;
    const int lane = pc & 63, ln = lane & 31, g = lane >> 5;
    const int rest = pc >> 6, u = rest & 3, t2 = (rest >> 2) & 1, blk = rest >> 3;
    u32x4 o;
    if (!j.tr) {
        o = ldg128(j.src + ((size_t)blk * M64 + 32 * t2 + ln) * M64 + 32 * g + 8 * u);
    } else {
        const uint16_t* p = j.src + ((size_t)blk * M64 + 32 * g + 8 * u) * M64 + 32 * t2 + ln;
        uint16_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = p[(size_t)e * M64];
#pragma unroll
        for (int w = 0; w < 4; ++w) o[w] = (uint32_t)v[2 * w] | ((uint32_t)v[2 * w + 1] << 16);
    }
    *reinterpret_cast<u32x4*>(j.dst + (size_t)pc * 8) = o;
}

// ------------------------------------------------------------------------ backward ----

// dst[blk][c][r] = src[blk][r][c] for 64 x 64 bf16 blocks; one workgroup (256 threads) per block.
__global__ void __launch_bounds__(256)
transpose64_kernel(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst)
{
    __shared__ __attribute__((aligned(16))) uint16_t tile[64][72];  // row stride 144 B
    const int tid = threadIdx.x;
    const uint16_t* s = src + (size_t)blockIdx.x * 4096;
    uint16_t* d = dst + (size_t)blockIdx.x * 4096;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int e = tid + 256 * it;  // 16-byte piece: row e / 8, columns 8 * (e % 8) ..
        *reinterpret_cast<u32x4*>(&tile[e >> 3][8 * (e & 7)]) = ldg128(s + (size_t)e * 8);
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int e = tid + 256 * it;  // output piece: row c = e / 8, columns r0 = 8 * (e % 8) ..
        const int c = e >> 3, r0 = 8 * (e & 7);
        uint32_t v[4];
#pragma unroll
        for (int w = 0; w < 4; ++w)
            v[w] = (uint32_t)tile[r0 + 2 * w][c] | ((uint32_t)tile[r0 + 2 * w + 1][c] << 16);
        *reinterpret_cast<u32x4*>(d + (size_t)e * 8) = u32x4{v[0], v[1], v[2], v[3]};
    }
}

// The transposed multiply y = x M on its own: both adjoint steps in one kernel (no copies of the vector between them).
__global__ void __launch_bounds__(512)
fwd_t_sq64_kernel(const uint16_t* __restrict__ dW, const uint16_t* __restrict__ LT /* packed L^T */,
                  const uint16_t* __restrict__ RT /* packed R^T */, uint16_t* __restrict__ dx, int64_t B)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char ldsb[];
    const Lane t = make_lane();
    const int64_t b0 = (int64_t)blockIdx.x * SQ_BM;
    int64_t row = b0 + t.ln;
    row = row < B ? row : B - 1;
    u32x4 pk1[16];  // pk1[i][t]: one 16-byte exchange piece per i, filled component by component

    // ---- adjoint of step 2: dU[b][c][r] = sum_l LT[c][r][l] dW[b][c][l]; as dY1[b][kk = r][j = c]
    // the exchange layout T[b][r][c] is dY1[b][kk][j]: operand order of the next stage
    block_stage<true>(t, dW + row * N64 + 32 * t.g, LT, ldsb, pk1);

    // ---- adjoint of step 1: dx[b][kk*64 + i] = sum_j RT[kk][i][j] dY1[b][kk][j], written over the dY1 lines (see
    // column_stage_inplace): line (b, kk) of the buffer becomes dx[b][kk*64 ..], which is also the layout of dx itself
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h) exchange_write(t, ldsb, pk1);
        __syncthreads();
        column_stage_inplace(t, RT, ldsb, h);
        __syncthreads();
        copy_out<false, true>(t, ldsb, dx, b0, B, 32 * h);
        __syncthreads();  // the lines are read before the second half overwrites them
    }
}

// The vector between the factors for the backward: U[b][c][r] = Y1[b][kk = r][j = c], the exchange layout as it is.
__global__ void __launch_bounds__(512)
u_sq64_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ R /* packed */, uint16_t* __restrict__ U, int64_t B)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char ldsb[];
    const Lane t = make_lane();
    const int64_t b0 = (int64_t)blockIdx.x * SQ_BM;
    int64_t row = b0 + t.ln;
    row = row < B ? row : B - 1;
    u32x4 pk1[16];
    block_stage<true>(t, x + row * N64 + 32 * t.g, R, ldsb, pk1);
    __syncthreads();
    copy_out<false>(t, ldsb, U, b0, B, 0);
    __syncthreads();
    exchange_write(t, ldsb, pk1);
    __syncthreads();
    copy_out<false>(t, ldsb, U, b0, B, 32);
}

// One factor of the backward, the gradients of its input and of its weights together: with its 64 blocks W[c] (64 x 64),
//     out[b][64 c + r] = sum_l in[b][64 l + c] W[c][l][r],     dW[c][l][r] = sum_b in[b][64 l + c] other[b][64 c + r].
//   L:  in = dy, other = U (as u_sq64_kernel leaves it), out = dU
//   R:  in = dU, other = x, out = dx  (dU[b][64 j + kk] is dY1[b][kk][j]: the permutation between the factors is again a
//       column of every block, so that both launches are the same kernel on what the one before wrote)
// Workgroup = eight blocks c0 .. c0+7 and every nz-th 32 rows of the batch, wave = one block: W[c] in registers as the
// operand of the first product, dW[c] in registers as the sum of the second.  A step is 32 rows.  `in` comes in pieces
// of eight c (16 bytes of every 128-byte line; the workgroups of the other c read the rest of the lines at about the
// same time on the same XCD), is turned to [c][row][l] in registers and LDS and read twice, as rows for `out` and
// transposed for dW; the wave's columns of `other` travel straight into an LDS ring of its own.  One barrier per step,
// rows requested two (in) and three (other) steps ahead.
// At 16384 rows 95 us, 402 MB at 4.2 TB/s; the pieces of `in` cost eight times their bytes between L2 and L1, which is
// why eight blocks share a workgroup and not fewer.  All workgroups walk the batch together, the first launch from its
// end, so that each finds in the memory-side cache what the launch before wrote last (both stages with chunks of
// consecutive rows: 334 us against 325 for the training step).
constexpr int ST_ROWS = 32;
constexpr int ST_IN = 8 * ST_ROWS * 128;     // bytes of a step's `in`: two buffers
constexpr int ST_RING = 3 * ST_ROWS * 128;   // a wave's ring of `other`
constexpr size_t ST_LDS = 2 * ST_IN + 8 * ST_RING;
static_assert(ST_LDS <= kMaxLdsBytes, "LDS");
struct Stage64 {
    const uint16_t *in, *W, *other;
    uint16_t* out;
    void* P;  // partial dW[chunk][c][l][r], fp32 or bf16
    float* colsum;  // SUMS: row zi receives the column sums of `in` over the chunk
    int p_bf16, nz, steps, down;
    int64_t B;
};
// SUMS: and the sums of the columns of `in` (the bias gradient), by adding up the fragments that dW is multiplied from.
template <bool SUMS>
__device__ __forceinline__ void bwd_sq64_stage(const Stage64& a, unsigned char* ldsb)
{
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ln = lane & 31, h = lane >> 5;
    // a chunk's eight workgroups on one XCD (workgroups go to the eight XCDs in turn)
    const int nwg = gridDim.x, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, per = nwg >> 3;  // (a multiple of eight)
    const int v = xcd * per + slot, zi = v >> 3, cg = v & 7, c = cg * 8 + wave;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)ldsb;
    const uint32_t ring = lds0 + 2 * ST_IN + wave * ST_RING;

    // the rows of a step: reads past the last one give zeros, writes are dropped (their offsets, all in the lane's
    // own, which is what the range check looks at, lie past the buffer's end)
    auto rows_at = [&](const uint16_t* p, int s) {
        const int64_t row = ((int64_t)(a.down ? a.steps - 1 - s : s) * a.nz + zi) * ST_ROWS;
        const int n = s >= a.steps || row >= a.B ? 0 : a.B - row < ST_ROWS ? (int)(a.B - row) : ST_ROWS;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p) + row * N64, 0, n * N64 * 2, 0x00020000);
    };
    // `in`: thread = (row, l = 4 quad ..), four pieces of eight c
    const int irow = tid >> 4, quad = tid & 15;
    const uint32_t in_at = (uint32_t)(irow * N64 * 2 + quad * 512 + cg * 16);
    const uint32_t in_put = lds0 + irow * 128 + ((quad >> 3) ^ run_key<64>(irow)) * 64 + (quad & 7) * 8;
    u32x4 stage[2][4];
    auto load_in = [&](int s, int stg) {
        const auto buf = rows_at(a.in, s);
#pragma unroll
        for (int e = 0; e < 4; ++e) stage[stg][e] = __builtin_amdgcn_raw_buffer_load_b128(buf, in_at + e * 128, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto store_in = [&](auto par) {
        constexpr int K = decltype(par)::value;
        const u32x4(&p)[4] = stage[K];
        each<8>([&](auto cc) {
            constexpr int C = decltype(cc)::value, w = C >> 1;
            u32x2 d;
            if constexpr (C & 1) d = u32x2{pick_hi16(p[0][w], p[1][w]), pick_hi16(p[2][w], p[3][w])};
            else d = u32x2{pick_lo16(p[0][w], p[1][w]), pick_lo16(p[2][w], p[3][w])};
            lds_put64<K * ST_IN + C * ST_ROWS * 128>(in_put, d);
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    // rows of 64 features: eight lanes a row; what a lane's place holds of the row (8 rows further: the same)
    const int prow = lane >> 3, piece = (((lane & 7) >> 2) ^ run_key<64>(prow)) * 4 + (lane & 3);
    const uint32_t other_at = (uint32_t)(prow * N64 * 2 + c * 128 + piece * 16);
    auto load_other = [&](int s, int rsel) {
        const auto buf = rows_at(a.other, s);
        auto to = (__attribute__((address_space(3))) unsigned char*)ldsb + 2 * ST_IN + wave * ST_RING + rsel * (ST_ROWS * 128);
#pragma unroll
        for (int n = 0; n < 4; ++n)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (__attribute__((address_space(3))) void*)(to + n * 1024), 16,
                                                     other_at + n * 8 * N64 * 2, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // transposed operands: lane's address of run t of a row (see monarch_lds_tr.h)
    const int G = lane >> 4, j = lane & 15;
    const uint32_t tr = (8 * (G >> 1) + (j >> 2)) * 128 + 32 * (G & 1) + 8 * (j & 3);
    const uint32_t tr_at[2] = {tr + run_key<64>(j >> 2) * 64, tr + (1 ^ run_key<64>(j >> 2)) * 64};
    const uint32_t in_line = lds0 + wave * (ST_ROWS * 128) + ln * 128;
    const uint32_t in_rd[2] = {in_line + run_key<64>(ln) * 64 + h * 16, in_line + (1 ^ run_key<64>(ln)) * 64 + h * 16};

    load_other(0, 0);
    load_in(0, 0);
    load_other(1, 1);
    load_in(1, 1);
    load_other(2, 2);
    // W[c], turned by way of the wave's eighth of the `in` buffers: operand [r][l], r = 32 t + lane % 32, K-step u
    Frag wf[8];
    {
        const uint32_t at = lds0 + wave * 8192;
        u32x4 g[8];
#pragma unroll
        for (int n = 0; n < 8; ++n) g[n] = ldg128(a.W + (size_t)c * 4096 + (n * 8 + prow) * 64 + piece * 8);
        each<8>([&](auto n) { lds_put128<decltype(n)::value * 1024>(at + lane * 16, g[decltype(n)::value]); });
        each<16>([&](auto o) {
            constexpr int O = decltype(o)::value, T = O >> 3, U = (O >> 1) & 3, H = O & 1;
            const u32x2 d = lds_tr16<U * 2048 + H * 512>(at + tr_at[T]);
            (H ? wf[T * 4 + U].hi : wf[T * 4 + U].lo) = d;
        });
        lgkm_wait(wf);
    }
    lds_barrier();

    f32x16 dw[2][2];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) dw[t >> 1][t & 1][i] = 0.f;
    float sums[2] = {0.f, 0.f};  // column l = 32 t + lane % 32 of block c, half of the rows
    int rsel = 0;  // ring place of the step's `other`
    auto step = [&](int s, auto par) {
        constexpr int K = decltype(par)::value;
        store_in(par);
        load_in(s + 2, K);
        // the step's `other` was requested before its `in`, which is in the registers stored above
        wait_vmcnt<24>();
        lds_barrier();
        const uint32_t oat = ring + rsel * (ST_ROWS * 128);
        u32x4 rows[4];
        Frag it[4], ot[4];  // [tile of 32 features][K-step]
        each<4>([&](auto u) {
            constexpr int U = decltype(u)::value;
            rows[U] = lds_get128<K * ST_IN + (U & 1) * 32>(in_rd[U >> 1]);
        });
        each<8>([&](auto o) {
            constexpr int O = decltype(o)::value, T = O >> 2, U = (O >> 1) & 1, H = O & 1;
            const u32x2 d = lds_tr16<K * ST_IN + U * 2048 + H * 512>(lds0 + wave * (ST_ROWS * 128) + tr_at[T]);
            const u32x2 e = lds_tr16<U * 2048 + H * 512>(oat + tr_at[T]);
            (H ? it[T * 2 + U].hi : it[T * 2 + U].lo) = d;
            (H ? ot[T * 2 + U].hi : ot[T * 2 + U].lo) = e;
        });
        lgkm_wait(rows);
        lgkm_wait(it);
        lgkm_wait(ot);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (SUMS) {
            auto add_pair = [](uint32_t pair, float sum) {
                return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), bf16x2{(__bf16)1.f, (__bf16)1.f}, sum, false);
            };
#pragma unroll
            for (int o = 0; o < 4; ++o)
                sums[o >> 1] += add_pair(it[o].lo[0], add_pair(it[o].lo[1], add_pair(it[o].hi[0], add_pair(it[o].hi[1], 0.f))));
        }
        f32x16 o2[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int i = 0; i < 16; ++i) o2[t][i] = 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) o2[t] = mfma32(wf[t * 4 + u].operand(), as_bf16x8(rows[u]), o2[t]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                dw[t >> 1][t & 1] = mfma32(ot[(t & 1) * 2 + u].operand(), it[(t >> 1) * 2 + u].operand(), dw[t >> 1][t & 1]);
        // out: lane = row, runs of four r; turned to whole lines in the ring place that was just read
        each<8>([&](auto o) {
            constexpr int T = decltype(o)::value >> 2, Q = decltype(o)::value & 3;
            lds_put64<0>(oat + ln * 128 + (((4 * T + Q) ^ (ln & 7)) * 16) + h * 8,
                         u32x2{pack_bf16x2(o2[T][4 * Q], o2[T][4 * Q + 1]), pack_bf16x2(o2[T][4 * Q + 2], o2[T][4 * Q + 3])});
        });
        u32x4 line[4];
        each<4>([&](auto n) {
            constexpr int N = decltype(n)::value;
            line[N] = lds_get128<N * 1024>(oat + prow * 128 + (((lane & 7) ^ prow) * 16));
        });
        lgkm_wait(line);
        const auto buf = rows_at(a.out, s);
#pragma unroll
        for (int n = 0; n < 4; ++n)
            __builtin_amdgcn_raw_buffer_store_b128(line[n], buf, (uint32_t)((prow + 8 * n) * N64 * 2 + c * 128 + (lane & 7) * 16), 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_other(s + 3, rsel);
        rsel = rsel == 2 ? 0 : rsel + 1;
    };
    for (int s = 0; s < a.steps; s += 2) {
        step(s, std::integral_constant<int, 0>{});
        step(s + 1, std::integral_constant<int, 1>{});
    }
    wait_vmcnt<0>();  // nothing is on its way into LDS any more
    if constexpr (SUMS) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const float v = sums[t] + __shfl_xor(sums[t], 32);
            if (h == 0) a.colsum[(size_t)zi * N64 + (32 * t + ln) * 64 + c] = v;
        }
    }

    // partial dW: lane = l, runs of four r; the wave turns its 32 x 32 tiles in its ring
    const size_t base = ((size_t)zi * 64 + c) * 4096;
    each<4>([&](auto t4) {
        constexpr int T = decltype(t4)::value;
        const f32x16& d = dw[T >> 1][T & 1];
        const uint32_t at = ring + (T & 1) * 4096;
        const size_t tile = base + (T >> 1) * 32 * 64 + (T & 1) * 32;
        if (a.p_bf16) {
            u32x4 line[2];
            each<4>([&](auto q) {
                constexpr int Q = decltype(q)::value;
                lds_put64<Q * 16>(at + ln * 80 + h * 8, u32x2{pack_bf16x2(d[4 * Q], d[4 * Q + 1]), pack_bf16x2(d[4 * Q + 2], d[4 * Q + 3])});
            });
            each<2>([&](auto n) { line[decltype(n)::value] = lds_get128<decltype(n)::value * 16 * 80>(at + (lane >> 2) * 80 + (lane & 3) * 16); });
            lgkm_wait(line);
            uint16_t* to = (uint16_t*)a.P + tile + (lane >> 2) * 64 + (lane & 3) * 8;
#pragma unroll
            for (int n = 0; n < 2; ++n) *reinterpret_cast<u32x4*>(to + n * 16 * 64) = line[n];
        } else {
            u32x4 line[4];
            each<4>([&](auto q) {
                constexpr int Q = decltype(q)::value;
                lds_put128<0>(at + ln * 128 + ((2 * Q + h) ^ (ln & 7)) * 16,
                              __builtin_bit_cast(u32x4, f32x4{d[4 * Q], d[4 * Q + 1], d[4 * Q + 2], d[4 * Q + 3]}));
            });
            each<4>([&](auto n) { line[decltype(n)::value] = lds_get128<decltype(n)::value * 1024>(at + prow * 128 + (((lane & 7) ^ prow) * 16)); });
            lgkm_wait(line);
            float* to = (float*)a.P + tile + prow * 64 + (lane & 7) * 4;
#pragma unroll
            for (int n = 0; n < 4; ++n) *reinterpret_cast<u32x4*>(to + n * 8 * 64) = line[n];
        }
    });
}

template <bool SUMS>
__global__ void __launch_bounds__(512)
bwd_sq64_stage_kernel(const Stage64 a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char ldsb[];
    bwd_sq64_stage<SUMS>(a, ldsb);
}

// Batch chunks of the two stages: with the eight workgroups of a chunk about one per CU, at least two steps of 32 rows
// each, and no more than fit the workspace (`room`; one chunk is the least).  bf16 gradients have bf16 partial sums,
// but beyond 256 rows only: up to there the chunks of 64 rows would add a rounding.
struct Plan64 {
    size_t off_u, off_du, off_rp, off_partL, off_partR, total;
    int nz, steps, p_bf16;
};

Plan64 make_plan64(const Problem& pb, size_t room = SIZE_MAX)
{
    Plan64 pl{};
    const int64_t steps = (pb.B + ST_ROWS - 1) / ST_ROWS;
    pl.p_bf16 = pb.wgrad_f32() || pb.B <= 256 ? 0 : 1;
    size_t off = 0;
    const size_t act = align_up((size_t)(pb.B > 0 ? pb.B : 1) * N64 * 2, 256);
    pl.off_u = off;  off += pb.saved ? 0 : act;
    pl.off_du = off; off += act;
    pl.off_rp = off; off += align_up(pb.n_R() * 2, 256);
    const size_t chunk = (size_t)M64 * M64 * M64 * (pl.p_bf16 ? 2 : 4), fit = room > off ? (room - off) / (2 * chunk) : 0;
    pl.nz = (int)(steps > 64 ? 32 : steps > 2 ? steps / 2 : 1);
    if ((size_t)pl.nz > fit) pl.nz = fit > 1 ? (int)fit : 1;
    pl.steps = (int)((steps + pl.nz - 1) / pl.nz);
    pl.off_partL = off; off += pl.nz * chunk;
    pl.off_partR = off; off += pl.nz * chunk;
    pl.total = off;
    return pl;
}

}  // namespace

bool sq64_supported(const Problem& pb)
{
    // both readings of the mid permutation coincide when k = q
    return pb.dtype == 1 && pb.k == 64 && pb.p == 64 && pb.q == 64 && pb.s == 64;
}

int fwd_sq64(const Problem& pb, const void* x, const void* R, const void* L, void* y, hipStream_t st)
{
    if (!sq64_supported(pb)) return -2;
    auto kern = fwd_sq64_kernel<false, false, false>;
    if (allow_dynamic_lds((const void*)kern, SQ_LDS) != hipSuccess)
        return -4;
    const int64_t grid = (pb.B + SQ_BM - 1) / SQ_BM;
    if (grid > 0x7fffffffLL) return -2;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), SQ_LDS, st, (const uint16_t*)x, (const uint16_t*)R,
                       (const uint16_t*)L, (const uint16_t*)nullptr, (uint16_t*)y, (uint16_t*)nullptr, pb.B);
    return hip_status(hipGetLastError());
}

// forward on packed factors: workspace = packed R, then packed L
size_t fwd_sq64_workspace(const Problem& pb) { return align_up(pb.n_R() * 2, 256) + align_up(pb.n_L() * 2, 256); }

int fwd_sq64_ws(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    if (!sq64_supported(pb)) return -2;
    uint16_t* Rp = (uint16_t*)ws;
    uint16_t* Lp = (uint16_t*)((char*)ws + align_up(pb.n_R() * 2, 256));
    if (!pb.ws_packed()) {
        const Pack64Job jr{(const uint16_t*)R, Rp, 0}, jl{(const uint16_t*)L, Lp, 0};
        hipLaunchKernelGGL(pack64_kernel, dim3(2 * 128), dim3(256), 0, st, jr, jl);
        if (hipGetLastError() != hipSuccess) return -4;
    }
    auto kern = pb.saved ? (pb.bias ? fwd_sq64_kernel<true, true, true> : fwd_sq64_kernel<true, false, true>)
                         : (pb.bias ? fwd_sq64_kernel<true, true, false> : fwd_sq64_kernel<true, false, false>);
    if (allow_dynamic_lds((const void*)kern, SQ_LDS) != hipSuccess)
        return -4;
    const int64_t grid = (pb.B + SQ_BM - 1) / SQ_BM;
    if (grid > 0x7fffffffLL) return -2;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), SQ_LDS, st, (const uint16_t*)x, Rp, Lp, (const uint16_t*)pb.bias,
                       (uint16_t*)y, (uint16_t*)pb.saved, pb.B);
    return hip_status(hipGetLastError());
}

// ... that keeps the vector between the factors for the backward, which then neither reads x nor multiplies for it: a
// write of U in place of a kernel that reads x and writes U.  kept = U, then the packed factors of this call.  Training
// step of the layer, 16384 rows: 329 -> 287 us (forward 70 -> 90, without 54 + 5 in the backward), 4096 rows 106 -> 89;
// with a bias, which took a pass over y and one over dy, 414 -> 290 and 137 -> 90.  The price is memory from the
// forward to the backward, 8 KB a row (134 MB at 16384 rows), which the workspace of that backward then does not need
// (monarch_bwd_kept_workspace_bytes).
size_t sq64_mid_bytes(const Problem& pb) { return align_up((size_t)(pb.B > 0 ? pb.B : 1) * N64 * 2, 256); }
size_t sq64_kept_bytes(const Problem& pb) { return sq64_mid_bytes(pb) + fwd_sq64_workspace(pb); }
int fwd_sq64_keep(Problem pb, const void* x, const void* R, const void* L, void* y, void* kept, hipStream_t st)
{
    pb.saved = kept;
    return fwd_sq64_ws(pb, x, R, L, y, (char*)kept + sq64_mid_bytes(pb), st);
}

bool bwd_sq64_supported(const Problem& pb) { return sq64_supported(pb); }

// Transposed multiply: input rows re-laid [c][l] (one pass), L^T and R^T packed, then the dx stages.
size_t fwd_t_sq64_workspace(const Problem& pb)
{
    return align_up((size_t)(pb.B > 0 ? pb.B : 1) * N64 * 2, 256) + 2 * align_up((size_t)M64 * M64 * M64 * 2, 256);
}

int fwd_t_sq64(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    if (!sq64_supported(pb)) return -2;
    const int64_t grid = (pb.B + SQ_BM - 1) / SQ_BM;
    if (grid > 0x7fffffffLL || pb.B > 0x7fffffffLL) return -2;
    char* w = (char*)ws;
    uint16_t* xT = (uint16_t*)w;
    uint16_t* LT = (uint16_t*)(w + align_up((size_t)pb.B * N64 * 2, 256));
    uint16_t* RT = LT + align_up((size_t)M64 * M64 * M64 * 2, 256) / 2;
    const Pack64Job jlt{(const uint16_t*)L, LT, 1}, jrt{(const uint16_t*)R, RT, 1};
    hipLaunchKernelGGL(pack64_kernel, dim3(2 * 128), dim3(256), 0, st, jlt, jrt);
    hipLaunchKernelGGL(transpose64_kernel, dim3((unsigned)pb.B), dim3(256), 0, st, (const uint16_t*)x, xT);
    if (hipGetLastError() != hipSuccess) return -4;
    if (allow_dynamic_lds((const void*)fwd_t_sq64_kernel, SQ_LDS) != hipSuccess)
        return -4;
    hipLaunchKernelGGL(fwd_t_sq64_kernel, dim3((unsigned)grid), dim3(512), SQ_LDS, st, xT, LT, RT, (uint16_t*)y, pb.B);
    return hip_status(hipGetLastError());
}

size_t bwd_sq64_workspace(const Problem& pb) { return make_plan64(pb).total; }
size_t bwd_sq64_least(const Problem& pb) { return make_plan64(pb, 0).total; }

int bwd_sq64(const Problem& pb, const void* dy, const void* x, const void* R, const void* L, void* dx,
             void* dR, void* dL, void* ws, hipStream_t st)
{
    if (!sq64_supported(pb)) return -2;
    const Plan64 pl = make_plan64(pb, pb.ws_bytes);
    const bool f32out = pb.wgrad_f32();
    if (pb.B == 0) {
        int rc = f32out ? launch_fill_zero_f32((float*)dR, pb.n_R(), st) : launch_fill_zero_u16((uint16_t*)dR, pb.n_R(), st);
        if (rc) return rc;
        return f32out ? launch_fill_zero_f32((float*)dL, pb.n_L(), st) : launch_fill_zero_u16((uint16_t*)dL, pb.n_L(), st);
    }
    const int64_t grid = (pb.B + SQ_BM - 1) / SQ_BM;
    if (grid > 0x7fffffffLL || pb.B > 0x7fffffffLL) return -2;
    char* w = (char*)ws;
    const uint16_t* U = pb.saved ? (const uint16_t*)pb.saved : (const uint16_t*)(w + pl.off_u);
    uint16_t* dU = (uint16_t*)(w + pl.off_du);
    uint16_t* Rp = (uint16_t*)(w + pl.off_rp);
    auto stage = bwd_sq64_stage_kernel<false>, stage_sums = bwd_sq64_stage_kernel<true>;
    if (allow_dynamic_lds((const void*)u_sq64_kernel, SQ_LDS) != hipSuccess ||
        allow_dynamic_lds((const void*)stage, ST_LDS) != hipSuccess || allow_dynamic_lds((const void*)stage_sums, ST_LDS) != hipSuccess)
        return -4;
    if (!pb.saved) {
        const Pack64Job jr{(const uint16_t*)R, Rp, 0};
        hipLaunchKernelGGL(pack64_kernel, dim3(128), dim3(256), 0, st, jr, jr);
        hipLaunchKernelGGL(u_sq64_kernel, dim3((unsigned)grid), dim3(512), SQ_LDS, st, (const uint16_t*)x, Rp, (uint16_t*)(w + pl.off_u), pb.B);
        if (hipGetLastError() != hipSuccess) return -4;
    }
    WgradDesc dl{}, dr{};
    dl.M = dl.N = dl.G = M64; dl.seg_w = M64;
    dl.p_bf16 = pl.p_bf16;
    dr = dl;
    dl.P = (float*)(w + pl.off_partL); dl.out = dL;
    dr.P = (float*)(w + pl.off_partR); dr.out = dR;
    ColsumJob cj{};
    if (pb.dbias) cj = wgrad_colsum_job(pb, pl.nz);
    const Stage64 sl{(const uint16_t*)dy, (const uint16_t*)L, U, dU, dl.P, cj.part, dl.p_bf16, pl.nz, pl.steps, 1, pb.B};
    const Stage64 sr{dU, (const uint16_t*)R, (const uint16_t*)x, (uint16_t*)dx, dr.P, nullptr, dr.p_bf16, pl.nz, pl.steps, 0, pb.B};
    hipLaunchKernelGGL(pb.dbias ? stage_sums : stage, dim3((unsigned)(8 * pl.nz)), dim3(512), ST_LDS, st, sl);
    hipLaunchKernelGGL(stage, dim3((unsigned)(8 * pl.nz)), dim3(512), ST_LDS, st, sr);
    if (hipGetLastError() != hipSuccess) return -4;
    return wgrad_reduce_pair(dl, dr, f32out, pl.nz, st, pb.dbias ? &cj : nullptr);
}

}  // namespace monarch
