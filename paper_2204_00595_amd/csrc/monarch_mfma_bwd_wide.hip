// bf16 backward for "wide block" Monarch layers (k = 4): the adjoints of steps 3, 2, P^T, 1 of
// Section 3.3 (the paper leaves them to automatic differentiation, Section 4).
//
//   prep      re-lays the weights once per call in MFMA fragment order (see prep_frag_kernel): every
//             weight operand below is then one contiguous, fully coalesced 1 KiB read per wave.
//             L is transposed with its rows picked in the order the mid permutation scatters them,
//             R is transposed with its K-slots in the order the chained accumulators of `data` hold dY1.
//   data      blocks of 192 and more, and short batches: two workgroups per 64 batch rows, two waves for an R block (bwd_pair_data,
//             which passes dY1 through LDS); else, and for the transposed multiply, one workgroup, wave w <-> R block kk = w:
//               X) recompute step 1, Y1[b][kk][j] (x through a DMA-filled LDS ring, packed R fragments
//                  straight into registers), and write it to the workspace (dL needs U);
//               A) dY1[b][kk][c*Q/4 + r1] = sum_l dy[b][4*l + c] * L[c][l][4*r1 + kk]
//                  (adjoint of steps 3 + 2 + P^T in one contraction; dy is de-interleaved into
//                  LDS once per workgroup, the result stays in accumulators);
//               B) dx[b][kk*P + i] = sum_j dY1[b][kk][j] * R[kk][j][i], fed straight from the
//                  accumulators of A (converted to bf16 in registers): dY1 never goes through LDS
//                  as an operand.  dY1 is also written to the workspace for dR.
//   wgrad     dL and dR as batch-contracted GEMMs over (dy, Y1) and (dY1, x)
//             (monarch_mfma_wgrad.hip), split over the batch, then one reduction pass.
#include <type_traits>
#include "monarch_internal.h"
#include "monarch_mfma_common.h"
#include "monarch_colsum.h"
#include "monarch_mfma_stage1.h"
#include "monarch_act.h"

namespace monarch {

namespace {

// ------------------------------------------------------------------------ prep ----

// The weights are re-laid once per call in MFMA *fragment order*: for every (tile, K-step) the 64
// lanes' 16-byte operand pieces are stored back to back, so that a fragment load in the data kernel
// is one contiguous, fully coalesced 1 KiB read (eight cache lines) instead of 32 or 64 lines.
// One thread builds one 16-byte piece (eight gathered elements).  Three arrays:
//   XF[kk][t][jt][lane][e]      = R[kk][32*jt + lane%32][16*t + 8*(lane/32) + e]
//       (step-1 recompute, 32x32x16: the layout stage1_block streams)
//   LF[kk][c][kt][jt][lane][e]   = L[c][32*kt + 8*(lane/16) + e][4*(16*jt + lane%16) + kk]
//       (dY1 stage, 16x16x32: L transposed, rows picked as the mid permutation scatters them)
//   RF[kk][ig][u][it][lane][e]   = R[kk][32*u + 16*(e/4) + 4*(lane/16) + e%4][16*(ig*IG + it) + lane%16]
//       (dx stage, 16x16x32: R transposed, K-slots in the order the chained accumulators hold dY1; for the kernel that reads dY1
//       from LDS in the natural order, R[kk][32*u + 8*(lane/16) + e][..])
__global__ void __launch_bounds__(256)
prep_frag_kernel(const uint16_t* __restrict__ L, const uint16_t* __restrict__ R, uint16_t* __restrict__ XF,
                 uint16_t* __restrict__ LF, uint16_t* __restrict__ RF, int P, int Q, int S, int IG, bool chained)
{
    const int nR = 4 * Q * P / 8, nL = 4 * S * Q / 8;  // pieces per array
    int pc = blockIdx.x * 256 + threadIdx.x;
    uint16_t v[8];
    uint16_t* dst;
    if (pc < nR) {
        const int lane = pc & 63;
        int rest = pc >> 6;
        const int QT = Q / 32, T = P / 16;
        const int jt = rest % QT; rest /= QT;
        const int t = rest % T, kk = rest / T;
        const uint16_t* src = R + ((size_t)kk * Q + 32 * jt + (lane & 31)) * P + 16 * t + 8 * (lane >> 5);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = src[e];
        dst = XF + (size_t)pc * 8;
    } else if (pc < nR + nL) {
        pc -= nR;
        const int lane = pc & 63;
        int rest = pc >> 6;
        const int JT = Q / 4 / 16;
        const int jt = rest % JT; rest /= JT;
        const int KT = S / 32;
        const int kt = rest % KT; rest /= KT;
        const int c = rest & 3, kk = rest >> 2;
        const uint16_t* src = L + ((size_t)c * S + 32 * kt + 8 * (lane >> 4)) * Q + 4 * (16 * jt + (lane & 15)) + kk;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = src[(size_t)e * Q];
        dst = LF + (size_t)pc * 8;
    } else if (pc < 2 * nR + nL) {
        pc -= nR + nL;
        const int lane = pc & 63;
        int rest = pc >> 6;
        const int it = rest % IG; rest /= IG;
        const int U = Q / 32;
        const int u = rest % U; rest /= U;
        const int nig = P / 16 / IG;
        const int ig = rest % nig, kk = rest / nig;
        const int step = chained ? 4 : 8, gap = chained ? 16 : 4;  // rows from lane / 16 to the next; from e to e + 4
        const uint16_t* src = R + ((size_t)kk * Q + 32 * u + step * (lane >> 4)) * P + 16 * (ig * IG + it) + (lane & 15);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = src[(size_t)(gap * (e >> 2) + (e & 3)) * P];
        dst = RF + (size_t)pc * 8;
    } else {
        return;
    }
    u32x4 o;
#pragma unroll
    for (int w = 0; w < 4; ++w) o[w] = (uint32_t)v[2 * w] | ((uint32_t)v[2 * w + 1] << 16);
    *reinterpret_cast<u32x4*>(dst) = o;
}

// ------------------------------------------------------------------------ data ----

template <int P_, int Q_, int S_, int LC_, int IG_>
struct BwdWide {
    static constexpr int K = 4, P = P_, Q = Q_, S = S_, LC = LC_, IG = IG_;
    static constexpr int BM = 64, NB = 2;   // stage X uses 32 x 32 tiles (2 row tiles)
    static constexpr int NBT = 4;           // stages A, B use 16 x 16 tiles (4 row tiles)
    static constexpr int QK = Q / K, QT = Q / 32, KQ = K * Q;
    static constexpr int N_IN = K * P, N_OUT = K * S;
    static constexpr int JT = QK / 16;      // 16-wide j tiles per (kk, c)
    static constexpr int Y1_STRIDE = KQ + 8;
    static constexpr int DW_STRIDE = LC + 8;
    static constexpr int DX_COLS = IG * 16;          // dx columns staged per wave at a time
    static constexpr int DX_STRIDE = DX_COLS + 8;
    static constexpr size_t LDS_Y1 = (size_t)BM * Y1_STRIDE * 2;
    static constexpr size_t LDS_DW = (size_t)K * BM * DW_STRIDE * 2;
    static constexpr size_t LDS_DX = (size_t)4 * BM * DX_STRIDE * 2;
    using S1 = Stage1<P_, Q_>;               // step-1 recompute (x through an LDS ring, packed R fragments)
    static constexpr size_t max2(size_t a, size_t b) { return a > b ? a : b; }
    static constexpr size_t LDS_BYTES = max2(max2(LDS_Y1, LDS_DW), max2(LDS_DX, S1::LDS_X));
    static_assert(P % 64 == 0 && Q % 32 == 0 && S % 32 == 0 && QK % 16 == 0, "tile shapes");
    static_assert(S % LC == 0 && LC % 32 == 0 && (P / 16) % IG == 0, "loop splits");
    static_assert(DX_COLS % 8 == 0 && (64 % (DX_COLS / 8) == 0), "dx staging copy-out");
    static_assert(LDS_BYTES <= kMaxLdsBytes, "LDS");
};

// cooperative copy of a [ROWS][COLS] bf16 LDS tile (row stride `stride`) to global rows b0.. (row pitch ld);
// eight LDS reads are in flight per thread before the first store.  NT: streaming (non-temporal) stores.
template <int COLS, int NTHREADS, bool NT, int ROWS = 64>
__device__ __forceinline__ void copy_out_tile(const uint16_t* src, int stride, uint16_t* dst, int64_t ld,
                                              int64_t b0, int64_t B, int tid)
{
    constexpr int PER_ROW = COLS / 8, TASKS = ROWS * PER_ROW, PER = (TASKS + NTHREADS - 1) / NTHREADS;
    // the rounds are not unrolled: unrolled, the compiler precomputes every round's addresses and, next
    // to the accumulators that are live around the copies, spills them
#pragma unroll 1
    for (int i0 = 0; i0 < PER; i0 += 8) {
        u32x4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t = tid + (i0 + i) * NTHREADS;
            if (i0 + i < PER && t < TASKS) v[i] = lds128(src + (size_t)(t / PER_ROW) * stride + 8 * (t % PER_ROW));
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t = tid + (i0 + i) * NTHREADS;
            const int r = t / PER_ROW, u = t % PER_ROW;
            if (i0 + i < PER && t < TASKS && b0 + r < B) {
                uint16_t* p = dst + (b0 + r) * ld + 8 * u;
                if (NT) stg128_nt(p, v[i]);
                else *reinterpret_cast<u32x4*>(p) = v[i];
            }
        }
    }
}

// orders the LDS traffic of one wave (what its lanes wrote is visible to its later reads)
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// MODE 0: everything.  MODE 1: the transposed multiply y = x M on its own (dy is then the input x of
// that product, dx its output): the recompute of step 1 and the workspace copies of both intermediates
// are left out.  MODE 2: the forward saved the vector between the factors, so step 1 is not recomputed;
// dY1 still goes to the workspace for the weight-gradient GEMM.
// ACT: dx leaves multiplied by gelu'(x_pre) (the layer's input was x = gelu(x_pre)).
template <typename C, int MODE, bool ACT>
__global__ void __launch_bounds__(256)
bwd_wide_data_kernel(const uint16_t* __restrict__ dy, const uint16_t* __restrict__ x,
                     const uint16_t* __restrict__ XF, const uint16_t* __restrict__ LF,
                     const uint16_t* __restrict__ RF, uint16_t* __restrict__ dx,
                     uint16_t* __restrict__ Y1ws, uint16_t* __restrict__ dY1ws, const uint16_t* __restrict__ x_pre,
                     int64_t B)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int64_t b0 = (int64_t)blockIdx.x * C::BM;
    const int kk = wave;

    // dy is consumed in chunks of LC features l; a chunk (64 rows x 4*LC columns) is fetched into
    // registers well before it is de-interleaved into LDS, so that its HBM latency is hidden
    constexpr int RUNS = C::LC / 8;                 // 64-byte runs per row and chunk
    constexpr int DYT = 64 * RUNS / 256;            // runs per thread
    static_assert(64 * RUNS % 256 == 0, "dy chunk split");
    u32x4 raw[DYT][4];
    auto load_dy = [&](int l0) {
#pragma unroll
        for (int i = 0; i < DYT; ++i) {
            const int t = tid + i * 256;
            const int r = t / RUNS, u = t - r * RUNS;
            int64_t row = b0 + r;
            row = row < B ? row : B - 1;
            const uint16_t* p = dy + row * C::N_OUT + (size_t)(l0 + 8 * u) * 4;
#pragma unroll
            for (int w = 0; w < 4; ++w) raw[i][w] = ldg128(p + 8 * w);  // cached: the weight-gradient GEMM re-reads dy
        }
    };

    // ------------------------------------------------- X: recompute step 1 -> workspace ----
    if constexpr (MODE != 0) {
        load_dy(0);
    } else {
        const int ln = lane & 31, g = lane >> 5;
        f32x16 acc[C::QT * C::NB];
        stage1_block<typename C::S1>(x, XF, b0, B, kk, lane, lds + (size_t)wave * C::S1::XR * 4096, acc);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();  // every wave is done with its x ring: the space becomes the Y1 tile
        // lane holds D^T[j][b] for b = nb*32 + ln and j = jt*32 + 8*(i/4) + 4*g + i%4
#pragma unroll
        for (int jt = 0; jt < C::QT; ++jt)
#pragma unroll
            for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const f32x16& a = acc[jt * C::NB + nb];
                    u32x2 v = {pack_bf16x2(a[4 * i4 + 0], a[4 * i4 + 1]), pack_bf16x2(a[4 * i4 + 2], a[4 * i4 + 3])};
                    const int j = jt * 32 + 8 * i4 + 4 * g;
                    *reinterpret_cast<u32x2*>(lds + (size_t)(nb * 32 + ln) * C::Y1_STRIDE + kk * C::Q + j) = v;
                }
        load_dy(0);  // in flight during the copy-out below
        __syncthreads();
        copy_out_tile<C::KQ, 256, false>(lds, C::Y1_STRIDE, Y1ws, C::KQ, b0, B, tid);
        __syncthreads();
    }

    // 16 x 16 tile coordinates for stages A and B
    const int l16 = lane & 15, h = lane >> 4;

    // ------------------------------------------------- A: dY1 (accumulators) ----
    // accA[(c*JT + jt)*NBT + bt][e] = dY1[b = bt*16 + l16][kk][j = c*QK + jt*16 + 4*h + e]
    f32x4 accA[C::K * C::JT * C::NBT];
#pragma unroll
    for (int t = 0; t < C::K * C::JT * C::NBT; ++t) accA[t] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int l0 = 0; l0 < C::S; l0 += C::LC) {
        // A operand: fragment (c, kt, jt) of LF (rows kk*QK + jt*16 + l16 of L^T), streamed through a
        // ring of NSA K-steps over the flattened (c, t) loop; the first loads are issued before the
        // de-interleave below so that they overlap it.
        constexpr int T = C::LC / 32, NSA = 4, NSTEP = C::K * T;
        const uint16_t* Lk = LF + (((size_t)kk * 4 * (C::S / 32) + l0 / 32) * C::JT * 64 + lane) * 8;
        u32x4 af[NSA][C::JT];
        auto issue = [&](int n, int slot) {
            const int c = n / T, t = n % T;
#pragma unroll
            for (int jt = 0; jt < C::JT; ++jt)
                af[slot][jt] = ldg128(Lk + ((size_t)(c * (C::S / 32) + t) * C::JT + jt) * 512);
        };
#pragma unroll
        for (int d = 0; d < NSA - 1; ++d)
            if (d < NSTEP) issue(d, d);
        __builtin_amdgcn_sched_barrier(0);
        // de-interleave the chunk (loaded earlier, see load_dy) into LDS dWs[c][b][l - l0]
#pragma unroll
        for (int i = 0; i < DYT; ++i) {
            const int t = tid + i * 256;
            const int r = t / RUNS, u = t - r * RUNS;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                u32x4 v;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const uint32_t lo = raw[i][w][c >> 1], hi = raw[i][w][2 + (c >> 1)];
                    v[w] = (c & 1) ? pick_hi16(lo, hi) : pick_lo16(lo, hi);
                }
                *reinterpret_cast<u32x4*>(lds + ((size_t)c * 64 + r) * C::DW_STRIDE + 8 * u) = v;
            }
        }
        __syncthreads();
        if (l0 + C::LC < C::S) load_dy(l0 + C::LC);  // the next chunk is in flight during the MFMA loop
#pragma unroll
        for (int n = 0; n < NSTEP; ++n) {
            const int c = n / T, t = n % T;
            __builtin_amdgcn_sched_barrier(0);
            if (n + NSA - 1 < NSTEP) issue(n + NSA - 1, (n + NSA - 1) % NSA);
            __builtin_amdgcn_sched_barrier(0);
            // B operand: dWs[c][bt*16 + l16][l]
            const uint16_t* Wc = lds + ((size_t)c * 64 + l16) * C::DW_STRIDE + 8 * h;
            bf16x8 bfr[C::NBT];
#pragma unroll
            for (int bt = 0; bt < C::NBT; ++bt)
                bfr[bt] = as_bf16x8(lds128(Wc + (size_t)bt * 16 * C::DW_STRIDE + t * 32));
#pragma unroll
            for (int jt = 0; jt < C::JT; ++jt)
#pragma unroll
                for (int bt = 0; bt < C::NBT; ++bt)
                    accA[(c * C::JT + jt) * C::NBT + bt] =
                        mfma16(as_bf16x8(af[n % NSA][jt]), bfr[bt], accA[(c * C::JT + jt) * C::NBT + bt]);
        }
        __syncthreads();
    }
    // bf16 fragments of dY1: dfr[J][bt] holds j = J*16 + 4*h + 0..3 (J = c*JT + jt) for row bt*16 + l16
    u32x2 dfr[C::K * C::JT][C::NBT];
#pragma unroll
    for (int J = 0; J < C::K * C::JT; ++J)
#pragma unroll
        for (int bt = 0; bt < C::NBT; ++bt) {
            const f32x4& a = accA[J * C::NBT + bt];
            dfr[J][bt] = u32x2{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3])};
        }
    // dY1 -> workspace through LDS (natural layout [b][kk*Q + j])
    if constexpr (MODE != 1) {
#pragma unroll
        for (int J = 0; J < C::K * C::JT; ++J)
#pragma unroll
            for (int bt = 0; bt < C::NBT; ++bt)
                *reinterpret_cast<u32x2*>(lds + (size_t)(bt * 16 + l16) * C::Y1_STRIDE + kk * C::Q + J * 16 + 4 * h) = dfr[J][bt];
        __syncthreads();
        copy_out_tile<C::KQ, 256, false>(lds, C::Y1_STRIDE, dY1ws, C::KQ, b0, B, tid);
        __syncthreads();
    }

    // ------------------------------------------------- B: dx from the chained fragments ----
    // K-step u covers j in [32u, 32u+32): lane slots 0..3 <- tile 2u, slots 4..7 <- tile 2u+1;
    // the RF fragments are laid out in exactly that order.
    uint16_t* stage = lds + (size_t)wave * 64 * C::DX_STRIDE;
    constexpr int U = C::Q / 32;
    const uint16_t* Rt = RF + ((size_t)kk * (C::P / 16 / C::IG) * U * C::IG * 64 + lane) * 8;
    // The fragments of all (ig, u) steps are contiguous in RF: step n = ig*U + u.  They run through a
    // ring of NSB steps that continues across the ig loop (U % NSB == 0 keeps the slot numbers static).
    constexpr int NIG = (C::P / 16) / C::IG;
    constexpr int NSB = (U % 4 == 0) ? 4 : ((U % 3 == 0) ? 3 : 2);
    static_assert(U % NSB == 0, "ring");
    u32x4 af[NSB][C::IG];
    auto issue = [&](int n, int slot) {
#pragma unroll
        for (int it = 0; it < C::IG; ++it) af[slot][it] = ldg128(Rt + ((size_t)n * C::IG + it) * 512);
    };
#pragma unroll
    for (int d = 0; d < NSB - 1; ++d) issue(d, d);
    // ACT: what leaves is multiplied by gelu'(x_pre), which costs the vector units two to three times what the tile
    // costs the matrix cores, and a wave is alone on its SIMD: so the pieces of tile ig - 1 leave between the MFMAs of
    // tile ig (measured where it mattered most, 1024 x 256 blocks, 16384 rows: 128 -> 117 us).  hp[i] holds the x_pre
    // piece that task i multiplies by; it is replaced by the one of the next tile as soon as it is used.
    constexpr int PIECES = C::DX_COLS / 8;
    const auto pre_at = [&](int ig, int i) {
        const int t = lane + i * 64;
        int64_t row = b0 + t / PIECES;
        row = row < B ? row : B - 1;  // rows past the end are read from a valid row and never stored
        return x_pre + row * C::N_IN + kk * C::P + ig * C::DX_COLS + 8 * (t % PIECES);
    };
    const auto piece = [&](int i) {
        const int t = lane + i * 64;
        return lds128(stage + (size_t)(t / PIECES) * C::DX_STRIDE + 8 * (t % PIECES));
    };
    const auto put = [&](int ig, int i, const u32x4& v, const u32x4& h) {
        const int t = lane + i * 64, r = t / PIECES;
        u32x4 o;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float g0 = __uint_as_float(v[w] << 16), g1 = __uint_as_float(v[w] & 0xffff0000u);
            const float h0 = __uint_as_float(h[w] << 16), h1 = __uint_as_float(h[w] & 0xffff0000u);
            o[w] = pack_bf16x2(g0 * gelu_grad_f(h0), g1 * gelu_grad_f(h1));
        }
        if (b0 + r < B) stg128_nt(dx + (b0 + r) * C::N_IN + kk * C::P + ig * C::DX_COLS + 8 * (t % PIECES), o);
    };
    u32x4 hp[ACT ? PIECES : 1];
    if constexpr (ACT) {
        static_assert(64 % PIECES == 0, "whole rows per round");
#pragma unroll
        for (int i = 0; i < PIECES; ++i) hp[i] = ldg128_nt(pre_at(0, i));
    }
    auto tile = [&](int ig, auto previous) {
        constexpr bool kPrevious = ACT && decltype(previous)::value;
        f32x4 acc[C::IG * C::NBT];
#pragma unroll
        for (int t = 0; t < C::IG * C::NBT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n = ig * U + u;
            __builtin_amdgcn_sched_barrier(0);
            if (n + NSB - 1 < NIG * U) issue(n + NSB - 1, (u + NSB - 1) % NSB);
            const int i0 = u * PIECES / U, i1 = (u + 1) * PIECES / U;  // tasks of this step
            u32x4 v[(PIECES + U - 1) / U];
            if constexpr (kPrevious) {
#pragma unroll
                for (int i = i0; i < i1; ++i) v[i - i0] = piece(i);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int bt = 0; bt < C::NBT; ++bt) {
                const u32x4 bv = {dfr[2 * u][bt][0], dfr[2 * u][bt][1], dfr[2 * u + 1][bt][0], dfr[2 * u + 1][bt][1]};
                const bf16x8 bfr = as_bf16x8(bv);
#pragma unroll
                for (int it = 0; it < C::IG; ++it)
                    acc[it * C::NBT + bt] = mfma16(as_bf16x8(af[u % NSB][it]), bfr, acc[it * C::NBT + bt]);
            }
            if constexpr (kPrevious) {
#pragma unroll
                for (int i = i0; i < i1; ++i) {
                    put(ig - 1, i, v[i - i0], hp[i]);
                    hp[i] = ldg128_nt(pre_at(ig, i));
                }
            }
        }
        if constexpr (kPrevious) wave_fence();  // the pieces of the previous tile have been read
        // D^T[i][b]: lane holds i = it*16 + 4*h + 0..3 for row b = bt*16 + l16
#pragma unroll
        for (int it = 0; it < C::IG; ++it)
#pragma unroll
            for (int bt = 0; bt < C::NBT; ++bt) {
                const f32x4& a = acc[it * C::NBT + bt];
                *reinterpret_cast<u32x2*>(stage + (size_t)(bt * 16 + l16) * C::DX_STRIDE + it * 16 + 4 * h) =
                    u32x2{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3])};
            }
        // the staging tile is private to the wave: no workgroup barrier
        wave_fence();
        if constexpr (!ACT) {
            copy_out_tile<C::DX_COLS, 64, true>(stage, C::DX_STRIDE, dx + kk * C::P + ig * C::DX_COLS, C::N_IN, b0, B, lane);
            wave_fence();
        }
    };
    if constexpr (ACT) tile(0, std::false_type{});
    for (int ig = ACT ? 1 : 0; ig < NIG; ++ig) tile(ig, std::bool_constant<ACT>{});
    if constexpr (ACT) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) put(NIG - 1, i, piece(i), hp[i]);
    }
}

// The same stages for two of the four blocks kk per workgroup, two waves per block: half of the accumulators per wave,
// two waves per SIMD and two workgroups per CU, and the two workgroups of a row tile on two CUs where the tiles alone
// would leave CUs idle.
//   X  half of the columns j per wave
//   A  two of the four c per wave; dy comes through a DMA-filled LDS ring as it is and is picked apart where it is read
//   B  from the dY1 tile in LDS (as bf16, which is also what goes to the workspace for dR), half of the columns i, or of the rows
//      where the column tiles do not come out even, per wave
// What bounds it: between L2 and L1 the weights pass once per 64 rows and dy twice, 8 to 16 TB/s in all.  Measured,
// this kernel against the one above: 768 -> 3072, 8192 rows, 30.8 and 36.9 us; blocks of 256 x 1024, 16384 rows, 106.8
// + 96.0 and 117.5 + 97.6.
// More chunks of dy or of fragments on the way change nothing; 128 rows per workgroup (43.5; 109.4 + 100.5) and all
// four blocks in eight waves (the whole training step 516 us against 518, but 300 against 287 at 192 x 768 and 40000
// rows) do not pay.  With q = 256 the form that recomputes step 1 has 10 to 18 registers too few for two workgroups
// and spills them; step 1 in a launch of its own instead (monarch_mfma_y1.hip) is no better up to 12000 rows (256 x
// 1024, whole backward: 8192 rows 96 and 99 us, 12000 rows 120 and 118, 16384 rows 149 and 143).
template <int P_, int Q_, int S_, int BM_ = 64>
struct BwdPair {
    static constexpr int K = 4, P = P_, Q = Q_, S = S_, IG = 4;
    static constexpr int BM = BM_, NBT = BM / 16;    // rows of a workgroup, in stages A and B as 16-row tiles
    static constexpr int QK = Q / K, KQ = K * Q;
    static constexpr int N_IN = K * P, N_OUT = K * S;
    static constexpr int JT = QK / 16;               // 16-wide j tiles per (kk, c)
    static constexpr int T_STRIDE = 2 * Q + 8;       // LDS tile [BM][two blocks of Q]
    static constexpr int DX_COLS = IG * 16;          // dx columns of a tile of stage B
    static constexpr int DX_STRIDE = DX_COLS + 8;
    // stage B: the two waves of a block take every other tile of columns, or half of the rows each where the tiles do
    // not come out even
    static constexpr bool BY_COLS = P / DX_COLS % 2 == 0;
    static constexpr int BT = BY_COLS ? NBT : NBT / 2, TILES = BY_COLS ? P / DX_COLS / 2 : P / DX_COLS;
    static constexpr size_t LDS_TILE = (size_t)BM * T_STRIDE * 2;
    static constexpr size_t LDS_DX = (size_t)4 * 16 * DX_STRIDE * 2;
    static constexpr int RING = 4;                   // stage A: chunks of 32 l of dy in LDS, 256 bytes a row
    static constexpr size_t LDS_DY = (size_t)RING * BM * 256;
    // step-1 recompute, half of a block's columns per wave (x through an LDS ring, packed R fragments)
    using S1 = Stage1<P_, Q_ / 2, Q_ / 32, 2, BM / 32>;
    static constexpr size_t max2(size_t a, size_t b) { return a > b ? a : b; }
    static constexpr size_t LDS_BYTES = max2(LDS_TILE + LDS_DX, max2(LDS_DY, S1::LDS_X));
    static_assert(P % DX_COLS == 0 && Q % 64 == 0 && S % 64 == 0, "tile shapes");
    static_assert(2 * LDS_BYTES <= kMaxLdsBytes, "two workgroups per CU");
};

// MODE and ACT as above (no mode 1).
template <typename C, int MODE, bool ACT>
__device__ __forceinline__ void
bwd_pair_data(const uint16_t* __restrict__ dy, const uint16_t* __restrict__ x, const uint16_t* __restrict__ XF,
              const uint16_t* __restrict__ LF, const uint16_t* __restrict__ RF, uint16_t* __restrict__ dx,
              uint16_t* __restrict__ Y1ws, uint16_t* __restrict__ dY1ws, const uint16_t* __restrict__ x_pre, int64_t B)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // the two workgroups of a row tile follow one another on one XCD (workgroups go to the eight XCDs in turn)
    const int slot = blockIdx.x >> 3, kp = slot & 1;
    const int64_t b0 = ((int64_t)(slot >> 1) * 8 + (blockIdx.x & 7)) * C::BM;
    if (b0 >= B) return;  // (uniform)
    const int kl = wave >> 1, half = wave & 1, kk = 2 * kp + kl;

    // ------------------------------------------------- X: recompute step 1 -> workspace ----
    if constexpr (MODE == 0) {
        using S1 = typename C::S1;
        const int ln = lane & 31, g = lane >> 5;
        f32x16 acc[S1::QT * S1::NB];
        stage1_block<S1>(x, XF, b0, B, kk, lane, lds + (size_t)wave * S1::XR * S1::X_SLOT, acc, half * S1::QT);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();  // every wave is done with its x ring: the space becomes the Y1 tile
        // lane holds D^T[j][b] for b = nb*32 + ln and j = half*Q/2 + jt*32 + 8*(i/4) + 4*g + i%4
#pragma unroll
        for (int jt = 0; jt < S1::QT; ++jt)
#pragma unroll
            for (int nb = 0; nb < S1::NB; ++nb)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const f32x16& a = acc[jt * S1::NB + nb];
                    u32x2 v = {pack_bf16x2(a[4 * i4 + 0], a[4 * i4 + 1]), pack_bf16x2(a[4 * i4 + 2], a[4 * i4 + 3])};
                    const int j = half * (C::Q / 2) + jt * 32 + 8 * i4 + 4 * g;
                    *reinterpret_cast<u32x2*>(lds + (size_t)(nb * 32 + ln) * C::T_STRIDE + kl * C::Q + j) = v;
                }
        __syncthreads();
        copy_out_tile<2 * C::Q, 256, false, C::BM>(lds, C::T_STRIDE, Y1ws + kp * 2 * C::Q, C::KQ, b0, B, tid);
        __syncthreads();
    }

    // 16 x 16 tile coordinates for stages A and B
    const int l16 = lane & 15, h = lane >> 4;

    // ------------------------------------------------- A: dY1 (accumulators) ----
    // accA[(ci*JT + jt)*NBT + bt][e] = dY1[b = bt*16 + l16][kk][j = c*QK + jt*16 + 4*h + e], c = 2*half + ci
    f32x4 accA[2 * C::JT * C::NBT];
#pragma unroll
    for (int t = 0; t < 2 * C::JT * C::NBT; ++t) accA[t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // dy arrives in chunks of 32 l, as it is, through an LDS ring filled in whole 256-byte pieces of its rows, three
    // chunks ahead. 16-byte piece u of a row (l = 2u, 2u + 1 of all four c) lies in place u ^ (row % 16): the reads of
    // 16 rows are conflict-free.
    constexpr int NC = C::S / 32, DPT = C::BM * 16 / 256;  // chunks; requests of a thread per chunk
    const int64_t rows = B - b0 < C::BM ? B - b0 : C::BM;  // rows past the end read as zeros
    const auto dyb = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(dy) + b0 * C::N_OUT, 0, (int)rows * C::N_OUT * 2, 0x00020000);
    const uint32_t dy_at = (uint32_t)((tid >> 4) * C::N_OUT * 2 + 16 * ((tid & 15) ^ ((tid >> 4) & 15)));
    auto issue_dy = [&](int n) {
        const int m = n < NC ? n : NC - 1;  // past the last chunk: again the last one, for the count of the requests
        auto to = (__attribute__((address_space(3))) unsigned char*)lds + (n % C::RING) * C::BM * 256 + wave * 1024;
#pragma unroll
        for (int i = 0; i < DPT; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(dyb, (__attribute__((address_space(3))) void*)(to + i * 256 * 16), 16,
                                                     dy_at + i * 16 * C::N_OUT * 2, m * 256, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // A operand: fragments (c, chunk, jt) of LF (rows kk*QK + jt*16 + l16 of L^T), c = 2 * half + ci, one chunk ahead
    const uint16_t* Lk = LF + (((size_t)kk * 4 + 2 * half) * NC * C::JT * 64 + lane) * 8;
    u32x4 lf[2][2][C::JT];
    auto issue_l = [&](int n, int at) {
        const int m = n < NC ? n : NC - 1;
#pragma unroll
        for (int ci = 0; ci < 2; ++ci)
#pragma unroll
            for (int jt = 0; jt < C::JT; ++jt) lf[at][ci][jt] = ldg128(Lk + ((size_t)(ci * NC + m) * C::JT + jt) * 512);
        __builtin_amdgcn_sched_barrier(0);
    };
    issue_dy(0);
    issue_dy(1);
    issue_l(0, 0);
    issue_dy(2);
    for (int n0 = 0; n0 < NC; n0 += 2) {
#pragma unroll
        for (int par = 0; par < 2; ++par) {
            const int n = n0 + par;
            __builtin_amdgcn_sched_barrier(0);
            // chunk n has landed once only what was requested after it is outstanding: the two chunks behind it, a
            // chunk's fragments
            wait_vmcnt<2 * DPT + 2 * C::JT>();
            lds_barrier();  // ... for every wave, and nobody reads chunk n-1 any more
            issue_l(n + 1, par ^ 1);
            issue_dy(n + 3);
            const uint16_t* chunk = lds + (size_t)(n % C::RING) * C::BM * 128 + (size_t)l16 * 128;
            uint32_t lo[2][4], hi[2][4];  // l = 8h + 2w and the next one, c = 2 * half (low 16 bits) and the next one
            auto read = [&](int bt, int at) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const uint32_t* piece = reinterpret_cast<const uint32_t*>(chunk + bt * 16 * 128 + 8 * ((4 * h + w) ^ l16)) + half;
                    lo[at][w] = piece[0];
                    hi[at][w] = piece[2];
                }
            };
            read(0, 0);
#pragma unroll
            for (int bt = 0; bt < C::NBT; ++bt) {
                __builtin_amdgcn_sched_barrier(0);
                if (bt + 1 < C::NBT) read(bt + 1, (bt + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ci = 0; ci < 2; ++ci) {
                    u32x4 v;
#pragma unroll
                    for (int w = 0; w < 4; ++w) v[w] = ci ? pick_hi16(lo[bt & 1][w], hi[bt & 1][w]) : pick_lo16(lo[bt & 1][w], hi[bt & 1][w]);
#pragma unroll
                    for (int jt = 0; jt < C::JT; ++jt)
                        accA[(ci * C::JT + jt) * C::NBT + bt] =
                            mfma16(as_bf16x8(lf[par][ci][jt]), as_bf16x8(v), accA[(ci * C::JT + jt) * C::NBT + bt]);
                }
            }
        }
    }
    wait_vmcnt<0>();  // nothing is on its way into LDS any more
    __syncthreads();
    // dY1 of the two blocks as bf16 in LDS: [b][kl*Q + j], the operand of stage B and the layout of the workspace copy
#pragma unroll
    for (int J = 0; J < 2 * C::JT; ++J)
#pragma unroll
        for (int bt = 0; bt < C::NBT; ++bt) {
            const f32x4& a = accA[J * C::NBT + bt];
            *reinterpret_cast<u32x2*>(lds + (size_t)(bt * 16 + l16) * C::T_STRIDE + kl * C::Q + (2 * half * C::JT + J) * 16 + 4 * h) =
                u32x2{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3])};
        }

    // ------------------------------------------------- B: dx ----
    constexpr int U = C::Q / 32;
    const uint16_t* Rt = RF + ((size_t)kk * (C::P / C::DX_COLS) * U * C::IG * 64 + lane) * 8;
    // The fragments run through a ring of NSB steps that continues across the tiles (U % NSB == 0 keeps the slot
    // numbers static).
    constexpr int NSB = (U % 4 == 0) ? 4 : ((U % 3 == 0) ? 3 : 2);
    static_assert(U % NSB == 0, "ring");
    const auto column_tile = [&](int n) { return C::BY_COLS ? 2 * n + half : n; };
    u32x4 af[NSB][C::IG];
    auto issue = [&](int n, int u, int at) {
#pragma unroll
        for (int it = 0; it < C::IG; ++it) af[at][it] = ldg128(Rt + ((size_t)(column_tile(n) * U + u) * C::IG + it) * 512);
    };
#pragma unroll
    for (int d = 0; d < NSB - 1; ++d) issue(0, d, d);
    // what a lane stores of a 16-row tile: two pieces of 16 bytes, eight lanes a row
    const int row0 = C::BY_COLS ? 0 : C::BM / 2 * half;
    uint16_t* stage = lds + C::LDS_TILE / 2 + (size_t)wave * 16 * C::DX_STRIDE;
    const auto row_at = [&](int bt, int i) { return b0 + row0 + bt * 16 + i * 8 + (lane >> 3); };
    u32x4 hp[ACT ? 2 * C::BT : 1];
    const auto load_pre = [&](int n, int bt, int i) {
        int64_t row = row_at(bt, i);
        row = row < B ? row : B - 1;  // rows past the end are read from a valid row and never stored
        hp[bt * 2 + i] = ldg128_nt(x_pre + row * C::N_IN + kk * C::P + column_tile(n) * C::DX_COLS + 8 * (lane & 7));
    };
    if constexpr (ACT) {
#pragma unroll
        for (int i = 0; i < 2 * C::BT; ++i) load_pre(0, i >> 1, i & 1);
    }
    __syncthreads();  // the tile is complete; nothing below writes it
    copy_out_tile<2 * C::Q, 256, false, C::BM>(lds, C::T_STRIDE, dY1ws + kp * 2 * C::Q, C::KQ, b0, B, tid);

    for (int n = 0; n < C::TILES; ++n) {
        f32x4 acc[C::IG * C::BT];
#pragma unroll
        for (int t = 0; t < C::IG * C::BT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            __builtin_amdgcn_sched_barrier(0);
            if (u + NSB - 1 < U) issue(n, u + NSB - 1, (u + NSB - 1) % NSB);
            else if (n + 1 < C::TILES) issue(n + 1, u + NSB - 1 - U, (u + NSB - 1) % NSB);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int bt = 0; bt < C::BT; ++bt) {
                const bf16x8 bfr = as_bf16x8(lds128(lds + (size_t)(row0 + bt * 16 + l16) * C::T_STRIDE + kl * C::Q + 32 * u + 8 * h));
#pragma unroll
                for (int it = 0; it < C::IG; ++it)
                    acc[it * C::BT + bt] = mfma16(as_bf16x8(af[u % NSB][it]), bfr, acc[it * C::BT + bt]);
            }
        }
        // D^T[i][b]: lane holds i = it*16 + 4*h + 0..3 for row b = bt*16 + l16; 16 rows at a time leave by way of the
        // wave's staging tile (private to the wave: no workgroup barrier)
#pragma unroll
        for (int bt = 0; bt < C::BT; ++bt) {
#pragma unroll
            for (int it = 0; it < C::IG; ++it) {
                const f32x4& a = acc[it * C::BT + bt];
                *reinterpret_cast<u32x2*>(stage + (size_t)l16 * C::DX_STRIDE + it * 16 + 4 * h) =
                    u32x2{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3])};
            }
            wave_fence();
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                u32x4 v = lds128(stage + (size_t)(i * 8 + (lane >> 3)) * C::DX_STRIDE + 8 * (lane & 7));
                if constexpr (ACT) {
                    const u32x4 hv = hp[bt * 2 + i];
                    if (n + 1 < C::TILES) load_pre(n + 1, bt, i);
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const float g0 = __uint_as_float(v[w] << 16), g1 = __uint_as_float(v[w] & 0xffff0000u);
                        const float h0 = __uint_as_float(hv[w] << 16), h1 = __uint_as_float(hv[w] & 0xffff0000u);
                        v[w] = pack_bf16x2(g0 * gelu_grad_f(h0), g1 * gelu_grad_f(h1));
                    }
                }
                const int64_t row = row_at(bt, i);
                if (row < B) stg128_nt(dx + row * C::N_IN + kk * C::P + column_tile(n) * C::DX_COLS + 8 * (lane & 7), v);
            }
            wave_fence();
        }
    }
}

template <typename C, int MODE, bool ACT>
__global__ void __launch_bounds__(256, 2)
bwd_pair_data_kernel(const uint16_t* dy, const uint16_t* x, const uint16_t* XF, const uint16_t* LF, const uint16_t* RF, uint16_t* dx,
                     uint16_t* Y1ws, uint16_t* dY1ws, const uint16_t* x_pre, int64_t B)
{
    bwd_pair_data<C, MODE, ACT>(dy, x, XF, LF, RF, dx, Y1ws, dY1ws, x_pre, B);
}

// Where two workgroups share a row tile (bwd_pair_data_kernel), whole backward at 6000, 12000 and 40000 rows, with it
// and without: blocks of 192 and more always (192 x 768: 65 and 73 us, 94 and 94, 286 and 300; 256 x 1024: 85 and 98,
// 126 and 126, 380 and 403; 1024 x 256: 100 and 111, 140 and 144, 442 and 462); smaller ones up to 128 tiles, which
// alone would leave CUs idle (128 x 512: 46 and 50 us, 65 and 62, 148 and 151; 512 x 128: 47 and 53, 65 and 65, 180 and
// 168).
bool pairs(const Problem& pb) { return pb.q > 128 || (pb.B + 63) / 64 <= 128; }

// In tiles of 32 rows instead of 64 while every workgroup then has a CU of its own: the weights that a workgroup streams
// are the same, but of the two chains of K-steps that bound it each step has half of the products (256 x 1024 blocks,
// 4000 rows, the kernel alone 34.5 and 24.4 us, 1024 x 256 26.6 and 20.6; training step at 4000 rows, 128: 46 and 44,
// 192: 58 and 56, 192 x 768: 75 and 68, 256 x 1024: 99 and 89, 768 x 192: 78 and 74, 512 x 128: 54 and 49; at 5000 rows
// 80 and 78, 105 and 106, 81 and 81, 56 and 55; with the nonlinearity's factor, feed-forward block of width 768, 4000
// rows 183 and 174, 5000 rows 209 and 218; 16384 rows, 192 x 768: 139 and 149).
bool short_tiles(const Problem& pb) { return pb.B <= 4096; }

template <typename K>
int launch_data_on(K kern, size_t lds, int64_t grid, const Problem& pb, const void* dy, const void* x, const uint16_t* XF,
                   const uint16_t* LF, const uint16_t* RF, void* dx, uint16_t* Y1ws, uint16_t* dY1ws, hipStream_t st)
{
    if (allow_dynamic_lds((const void*)kern, lds) != hipSuccess)
        return -4;
    if (grid > 0x7fffffffLL) return -2;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), lds, st, (const uint16_t*)dy, (const uint16_t*)x, XF, LF, RF,
                       (uint16_t*)dx, Y1ws, dY1ws, (const uint16_t*)pb.x_pre, pb.B);
    return hip_status(hipGetLastError());
}

// no workspace for dY1: dx only; dY1 but no Y1 workspace: the forward saved that vector, or it is made elsewhere
template <int P, int Q, int S, int LC, int IG>
int launch_data(const Problem& pb, const void* dy, const void* x, const uint16_t* XF, const uint16_t* LF,
                const uint16_t* RF, void* dx, uint16_t* Y1ws, uint16_t* dY1ws, hipStream_t st)
{
    using C = BwdWide<P, Q, S, LC, IG>;
    const int64_t tiles = (pb.B + 63) / 64;
    auto run = [&](auto kern) { return launch_data_on(kern, C::LDS_BYTES, tiles, pb, dy, x, XF, LF, RF, dx, Y1ws, dY1ws, st); };
    if (!dY1ws) return pb.x_pre ? -2 : run(bwd_wide_data_kernel<C, 1, false>);
    if (pairs(pb)) {
        auto pair = [&](auto shape) {
            using D = decltype(shape);
            auto run2 = [&](auto kern) {  // two workgroups for each row tile, whole sets of eight tiles
                return launch_data_on(kern, D::LDS_BYTES, ((pb.B + D::BM - 1) / D::BM + 7) / 8 * 16, pb, dy, x, XF, LF, RF, dx, Y1ws, dY1ws, st);
            };
            if (Y1ws) return pb.x_pre ? run2(bwd_pair_data_kernel<D, 0, true>) : run2(bwd_pair_data_kernel<D, 0, false>);
            return pb.x_pre ? run2(bwd_pair_data_kernel<D, 2, true>) : run2(bwd_pair_data_kernel<D, 2, false>);
        };
        return short_tiles(pb) ? pair(BwdPair<P, Q, S, 32>()) : pair(BwdPair<P, Q, S>());
    }
    if constexpr (Q <= 128) {
        if (Y1ws) return pb.x_pre ? run(bwd_wide_data_kernel<C, 0, true>) : run(bwd_wide_data_kernel<C, 0, false>);
        return pb.x_pre ? run(bwd_wide_data_kernel<C, 2, true>) : run(bwd_wide_data_kernel<C, 2, false>);
    }
    return -2;
}

struct Entry {
    int p, q, s, ig;  // ig: a loop split of the data kernels that fixes the fragment order of the weights
    int (*fn)(const Problem&, const void*, const void*, const uint16_t*, const uint16_t*, const uint16_t*, void*,
              uint16_t*, uint16_t*, hipStream_t);
};

//                                    P    Q    S   LC  IG
const Entry kTable[] = {
    {192, 192, 192, 4, launch_data<192, 192, 192, 192, 4>},
    {192, 192, 768, 4, launch_data<192, 192, 768, 192, 4>},
    {256, 256, 1024, 4, launch_data<256, 256, 1024, 128, 4>},
    {1024, 256, 256, 4, launch_data<1024, 256, 256, 128, 4>},
    {768, 192, 192, 4, launch_data<768, 192, 192, 192, 4>},
    {256, 256, 256, 4, launch_data<256, 256, 256, 128, 4>},
    {192, 192, 576, 4, launch_data<192, 192, 576, 192, 4>},
    {256, 256, 768, 4, launch_data<256, 256, 768, 128, 4>},
    {128, 128, 128, 4, launch_data<128, 128, 128, 128, 4>},
    {128, 128, 512, 4, launch_data<128, 128, 512, 128, 4>},
    {512, 128, 128, 4, launch_data<512, 128, 128, 128, 4>},
    {64, 64, 64, 4, launch_data<64, 64, 64, 64, 4>},
    {64, 64, 128, 4, launch_data<64, 64, 128, 64, 4>},
    {128, 64, 64, 4, launch_data<128, 64, 64, 64, 4>},
};

const Entry* find(const Problem& pb)
{
    if (pb.dtype != 1 || pb.k != 4 || pb.perm_b()) return nullptr;
    for (const Entry& e : kTable)
        if (e.p == pb.p && e.q == pb.q && e.s == pb.s) return &e;
    return nullptr;
}

// The two weight-gradient GEMMs share one split of the batch into nz chunks: about one
// workgroup per CU in total, chunks of at least 256 rows (multiples of the 32-row pipeline
// step) so that the fp32 partial tiles stay small next to the operands.
struct Plan {
    size_t off_y1, off_dy1, off_xf, off_lf, off_rf, off_partL, off_partR, total;
    int nz, rows_per_chunk;
    bool ok;
};

void fill_descs(const Problem& pb, WgradDesc& dl, WgradDesc& dr)
{
    // dL[c][l][4*r1 + kk] = sum_b dy[b][4*l + c] * Y1[b][kk][c*Q/4 + r1]
    dl = WgradDesc{};
    dl.lda = pb.n_out(); dl.a_g = 1; dl.deint = 1;
    dl.ldb = pb.kq(); dl.b_g = pb.q / 4; dl.b_seg = pb.q; dl.seg_w = pb.q / 4;
    dl.M = pb.s; dl.N = pb.q; dl.G = 4; dl.rows = pb.B;
    // dR[kk][j][i] = sum_b dY1[b][kk][j] * x[b][kk*P + i]
    dr = WgradDesc{};
    dr.lda = pb.kq(); dr.a_g = pb.q; dr.deint = 0;
    dr.ldb = pb.n_in; dr.b_g = pb.p; dr.b_seg = 0; dr.seg_w = pb.p;
    dr.M = pb.q; dr.N = pb.p; dr.G = 4; dr.rows = pb.B;
}

// `room`: bytes there are; a plan with one chunk may need more.  (Chunks are whole 64 rows, so that a batch just
// below a multiple can have more of them than a longer one.)
Plan make_plan(const Problem& pb, size_t room = SIZE_MAX)
{
    Plan pl{};
    WgradDesc dl, dr;
    fill_descs(pb, dl, dr);
    const int tiles = wgrad_tiles(dl) + wgrad_tiles(dr);
    pl.ok = wgrad_tiles(dl) > 0 && wgrad_tiles(dr) > 0;
    if (!pl.ok) return pl;
    int64_t z = 256 / tiles;  // one workgroup (eight waves) per CU: its two LDS buffers leave room for one only
    const int64_t maxz = (pb.B + 255) / 256;
    if (z > maxz) z = maxz;
    if (z < 1) z = 1;
    const size_t act = align_up((size_t)(pb.B > 0 ? pb.B : 1) * pb.kq() * 2, 256);
    for (;; z = pl.nz - 1) {
        const int64_t rpc = ((pb.B + z - 1) / z + 63) / 64 * 64;  // whole pipeline rounds (two 32-row steps)
        pl.rows_per_chunk = (int)(rpc > 0 ? rpc : 32);
        pl.nz = (int)((pb.B + pl.rows_per_chunk - 1) / pl.rows_per_chunk);
        if (pl.nz < 1) pl.nz = 1;
        size_t off = 0;
        pl.off_y1 = off;  off += act;
        pl.off_dy1 = off; off += act;
        pl.off_xf = off; off += align_up(pb.n_R() * 2, 256);
        pl.off_lf = off; off += align_up(pb.n_L() * 2, 256);
        pl.off_rf = off; off += align_up(pb.n_R() * 2, 256);
        pl.off_partL = off; off += align_up((size_t)pl.nz * pb.n_L() * 4, 256);
        pl.off_partR = off; off += align_up((size_t)pl.nz * pb.n_R() * 4, 256);
        pl.total = off;
        if (pl.total <= room || pl.nz == 1) return pl;
    }
}

}  // namespace

bool bwd_wide_supported(const Problem& pb) { return find(pb) != nullptr && make_plan(pb).ok; }
bool saved_supported(const Problem& pb) { return bwd_wide_supported(pb) && fwd_wide_supported(pb); }

// Transposed multiply through the same data kernel (the weights in fragment order, then the dx stages).
size_t fwd_t_wide_workspace(const Problem& pb) { return 2 * align_up(pb.n_R() * 2, 256) + align_up(pb.n_L() * 2, 256); }

int fwd_t_wide(const Problem& pb, const void* x, const void* R, const void* L, void* y, void* ws, hipStream_t st)
{
    const Entry* e = find(pb);
    if (!e) return -2;
    char* w = (char*)ws;
    uint16_t* XF = (uint16_t*)w;
    uint16_t* LF = (uint16_t*)(w + align_up(pb.n_R() * 2, 256));
    uint16_t* RF = (uint16_t*)(w + align_up(pb.n_R() * 2, 256) + align_up(pb.n_L() * 2, 256));
    const size_t pieces = (2 * pb.n_R() + pb.n_L()) / 8;
    const int nprep = (int)((pieces + 255) / 256);
    hipLaunchKernelGGL(prep_frag_kernel, dim3((unsigned)nprep), dim3(256), 0, st, (const uint16_t*)L, (const uint16_t*)R,
                       XF, LF, RF, pb.p, pb.q, pb.s, e->ig, true);
    if (hipGetLastError() != hipSuccess) return -4;
    return e->fn(pb, x, nullptr, XF, LF, RF, y, nullptr, nullptr, st);
}

size_t bwd_wide_workspace(const Problem& pb) { return make_plan(pb).total; }
size_t bwd_wide_least(const Problem& pb) { return make_plan(pb, 0).total; }

int bwd_wide(const Problem& pb, const void* dy, const void* x, const void* R, const void* L, void* dx,
             void* dR, void* dL, void* ws, hipStream_t st)
{
    const Entry* e = find(pb);
    const Plan pl = make_plan(pb, pb.ws_bytes);
    if (!e || !pl.ok) return -2;
    char* w = (char*)ws;
    uint16_t* Y1ws = (uint16_t*)(w + pl.off_y1);
    uint16_t* dY1ws = (uint16_t*)(w + pl.off_dy1);
    uint16_t* XF = (uint16_t*)(w + pl.off_xf);
    uint16_t* LF = (uint16_t*)(w + pl.off_lf);
    uint16_t* RF = (uint16_t*)(w + pl.off_rf);
    const bool f32out = pb.wgrad_f32();
    if (pb.B == 0) {
        int rc = f32out ? launch_fill_zero_f32((float*)dR, pb.n_R(), st) : launch_fill_zero_u16((uint16_t*)dR, pb.n_R(), st);
        if (rc) return rc;
        return f32out ? launch_fill_zero_f32((float*)dL, pb.n_L(), st) : launch_fill_zero_u16((uint16_t*)dL, pb.n_L(), st);
    }
    const size_t pieces = (2 * pb.n_R() + pb.n_L()) / 8;
    const int nprep = (int)((pieces + 255) / 256);
    hipLaunchKernelGGL(prep_frag_kernel, dim3((unsigned)nprep), dim3(256), 0, st, (const uint16_t*)L, (const uint16_t*)R,
                       XF, LF, RF, pb.p, pb.q, pb.s, e->ig, !pairs(pb));
    if (hipGetLastError() != hipSuccess) return -4;
    // Step 1 (Y1, for dL) is recomputed either by the data kernel itself or, for long batches of the shapes that have
    // it, by a GEMM of its own with four times the rows per workgroup (monarch_mfma_y1.hip); not at all when the
    // forward saved it.
    const bool y1_apart = !pb.saved && y1_gemm_supported(pb);
    int rc = 0;
    if (y1_apart) {
        rc = y1_gemm(pb, x, XF, Y1ws, st);
        if (rc) return rc;
    }
    rc = e->fn(pb, dy, x, XF, LF, RF, dx, (pb.saved || y1_apart) ? nullptr : Y1ws, dY1ws, st);
    if (rc) return rc;

    WgradDesc dl, dr;
    fill_descs(pb, dl, dr);
    dl.A = (const uint16_t*)dy; dl.Bm = Y1ws; dl.P = (float*)(w + pl.off_partL); dl.out = dL;
    if (pb.saved) {
        // the saved vector is in stage-2 order: group c owns the Q contiguous columns c*Q .. of every row
        dl.Bm = (const uint16_t*)pb.saved;
        dl.b_g = pb.q; dl.b_seg = 0; dl.seg_w = pb.q;
    }
    dr.A = dY1ws; dr.Bm = (const uint16_t*)x; dr.P = (float*)(w + pl.off_partR); dr.out = dR;
    dl.rows_per_chunk = dr.rows_per_chunk = pl.rows_per_chunk;
    dl.p_bf16 = dr.p_bf16 = f32out ? 0 : 1;  // bf16 gradients: bf16 partial tiles
    ColsumJob cj{};
    if (pb.dbias) {
        cj = wgrad_colsum_job(pb, pl.nz);
        dl.colsum = cj.part;
    }
    rc = wgrad_gemm_pair(dl, dr, pl.nz, st);
    if (rc) return rc;
    return wgrad_reduce_pair(dl, dr, f32out, pl.nz, st, pb.dbias ? &cj : nullptr);
}

}  // namespace monarch
