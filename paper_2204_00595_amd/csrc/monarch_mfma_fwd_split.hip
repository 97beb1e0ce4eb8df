// bf16 forward of the four-block layers on packed weights, for batches too short to fill the chip with 64-row tiles of the
// fused kernel (monarch_mfma_fwd_frag.hip): one launch per block-diagonal factor, so that the weights are spread over all CUs
// instead of passing through the few that have a row tile.  The vector between the factors goes through the workspace in the MFMA
// fragments of the second stage: K-step j/4 contracts the 16 elements (kk, j%4), and block c = (j/4) / (Q/16) is a run of them.
//
//   stage 1   workgroup = (row tile, block kk, NT column tiles of 32): the four waves share out the contraction, so that every
//             byte of x and R the workgroup needs is loaded once, and add up their tiles through LDS
//   stage 2   workgroup = (row tile, NT column tiles of 32): wave c computes block c (again nothing is loaded twice);
//             the four blocks of an output row are interleaved through LDS and leave in whole rows
//
// U and the weights come in 1 KiB fragments straight from memory to registers; the rows of x do too where there are few
// tiles, and else in whole lines that change places through LDS (RowPieces).
// What bounds it: latency for one row tile (two launches of about 3.5 us), above that the address path of the L1: 20
// cycles a fragment for MFMAs of 32 cycles on four SIMDs.  With U in rows, a fragment of it took 62 cycles, and so did
// one of x (1531 rows: the stages of 1024 -> 4096 5.8 + 16.4 -> 5.2 + 15.5 us, the second one now bound by the
// nonlinearity, of 4096 -> 1024 12.8 + 7.6 -> 10.4 + 5.2).
// Measured, 1024 -> 4096 -> 1024 with bias and GELU, against the fused kernel alone and against U in rows: 8 rows 54
// us and 16 for both, 256 rows 66, 19.9 and 18.6, 1531 rows 69, 40.1 and 32.7; 768 -> 3072 -> 768, 1531 rows: 33.0 and
// 25.6.
#include "../../include/monarch.h"
#include "monarch_internal.h"
#include "monarch_mfma_common.h"
#include "monarch_mfma_pack.h"
#include "monarch_mfma_split.h"
#include "monarch_act.h"

namespace monarch {
namespace {

struct SplitPack {
    const uint16_t *R, *L;
    uint16_t *RF1, *LF2;
    int S, pieces, blocks;  // workgroups that compute; those after them pack
};

// PACK: R is read as it is, and further workgroups of the launch build the packed copies of R and L, for the second stage and for
// later calls.
template <int NB, int NT, int NG, int AHEAD, bool PACK, bool TURN>
__global__ void __launch_bounds__(256)
split_stage1_kernel(const uint16_t* __restrict__ x, const SplitPack w, uint16_t* __restrict__ U, int64_t B, int P, int Q, SplitGrid gr)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char split_lds[];
    if constexpr (PACK) {
        if ((int)blockIdx.x >= w.blocks) {
            pack_fwd_piece(w.R, w.L, w.RF1, w.LF2, P, Q, w.S, ((int)blockIdx.x - w.blocks) * 256 + (int)threadIdx.x);
            return;
        }
    }
    split_stage1<NB, NT, NG, AHEAD, PACK, false, TURN>(x, PACK ? w.R : w.RF1, U, B, P, Q, gr, (int)blockIdx.x, reinterpret_cast<f32x4*>(split_lds));
}

template <int NB, int NT, int NG, int AHEAD, bool ACT>
__global__ void __launch_bounds__(256)
split_stage2_kernel(const uint16_t* __restrict__ U, const uint16_t* __restrict__ LF2, const uint16_t* __restrict__ bias,
                    uint16_t* __restrict__ y, uint16_t* __restrict__ y_pre, int64_t B, int Q, int S, SplitGrid gr)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char split_lds[];
    constexpr int kStride = NT * 128 + 8, kRows = 32 * NB;
    uint16_t* const out = reinterpret_cast<uint16_t*>(split_lds);
    uint16_t* const pre = out + kRows * kStride;
    int rt, in;
    if (!split_index(gr, (int)blockIdx.x, rt, in)) return;
    const int c = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, ln = lane & 31, g = lane >> 5;
    const int KS = Q / 16, LT = S / 32, lt0 = in * NT;
    const int64_t b0 = (int64_t)rt * kRows;
    const int rows = B - b0 < kRows ? (int)(B - b0) : kRows;

    f32x16 acc[NB][NT];
    uint32_t a_at[NB], w_at[NT];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int i = 0; i < NB; ++i) a_at[i] = ln < rows ? (uint32_t)((g * rows + ln) * 16) : kNowhere;
#pragma unroll
    for (int j = 0; j < NT; ++j) w_at[j] = lt0 + j < LT ? (uint32_t)((lt0 + j) * KS * 1024 + lane * 16) : kNowhere;
    static_assert(NB == 1, "a tile of U has the rows of the workgroup");
    tile_product<NB, NT, NG, AHEAD, false, false, false>(U + b0 * 4 * Q + c * KS * rows * 16, a_at, (uint32_t)rows * 32, LF2 + (size_t)c * LT * KS * 512, w_at,
                                                  1024u, KS, acc, 0u, 0, nullptr);

#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int l = (lt0 + j) * 32 + ln;
        const float bv = bias && lt0 + j < LT ? __uint_as_float((uint32_t)bias[l * 4 + c] << 16) : 0.f;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int at = (i * 32 + 8 * (r / 4) + 4 * g + r % 4) * kStride + (j * 32 + ln) * 4 + c;
                const float v = acc[i][j][r] + bv;
                if constexpr (ACT) {
                    if (y_pre) pre[at] = (uint16_t)pack_bf16x2(v, v);
                    const float a = gelu_f(v);
                    out[at] = (uint16_t)pack_bf16x2(a, a);
                } else {
                    out[at] = (uint16_t)pack_bf16x2(v, v);
                }
            }
    }
    lds_barrier();
    constexpr int kPieces = NT * 16;  // of 16 bytes per row
    const int limit = (4 * S - lt0 * 128) / 8;
    for (int idx = threadIdx.x; idx < kRows * kPieces; idx += 256) {
        const int row = idx / kPieces, pc = idx % kPieces;
        if (row >= rows || pc >= limit) continue;
        const size_t to = (size_t)(b0 + row) * 4 * S + lt0 * 128 + pc * 8;
        *reinterpret_cast<u32x4*>(y + to) = lds128(out + row * kStride + pc * 8);
        if constexpr (ACT)
            if (y_pre) *reinterpret_cast<u32x4*>(y_pre + to) = lds128(pre + row * kStride + pc * 8);
    }
}

// Both factors in one launch, for a few rows on packed weights.  A workgroup computes 32 columns of one output block c, and
// for them the vector that block c contracts by itself: those are the outputs c q/4 .. (c + 1) q/4 of every block of the
// first factor, so that the workgroups of a block read the same quarter of R (128 KiB at 256 x 256) and none waits for
// another.  Eight waves: wave = (block kk, one of the two 32-row tiles of R that the quarter touches; once_covers says
// where there are no more), the contraction in four parts that are added up as in split_stage1 (the same bits); then one
// wave multiplies with L, whose fragments it requested at the start.  A workgroup's block goes by its XCD, for the
// quarter of R to come through two L2s.
// Bound by latency: one of memory, the way of the quarter through the L1 (2500 clocks at 256 x 256) and two chains of
// products.  On the GPU alone, 256 x 1024 blocks: 8 rows 6.5 us in two launches, 5.7 in one, 32 rows 6.9 and 6.8, 64 rows
// 7.0 and 7.2; 192 x 768: 8 rows 6.3 and 5.0, 64 rows 6.9 and 6.2; 512 x 128 (the quarter of R as large, four times the
// rows): 8 rows 5.6 and 6.3.  Both layers of width 1024 with the host's part, 8 rows: 15.8 and 12.9.
// DIRECT: RF1 and LF2 are R and L as they are, for the shapes that no call packs for the next: R in whole lines that
// change places through LDS, L in both halves of the 16 values that a step contracts.
template <int T4, int K4, bool ACT, bool DIRECT>
__global__ void __launch_bounds__(512)
split_once_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ RF1, const uint16_t* __restrict__ LF2,
                  const uint16_t* __restrict__ bias, uint16_t* __restrict__ y, uint16_t* __restrict__ y_pre, int64_t B, int P, int Q, int S)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char split_lds[];
    uint16_t* const Uf = reinterpret_cast<uint16_t*>(split_lds);  // fragments of the block's vector: [step][h][row][8]
    uint16_t* const xs = Uf + 4 * K4 * 2 * 32 * 8;                // 16-byte pieces of x: [piece][row ^ piece % 32]
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, ln = lane & 31, h = lane >> 5;
    const int bid = (int)blockIdx.x, c = (bid & 7) >> 1, lt = (bid >> 3) * 2 + (bid & 1), QT = Q / 32, KS = Q / 16, LT = S / 32;
    if (lt >= LT) return;
    const int64_t b0 = (int64_t)blockIdx.y * 32;
    const int rows = B - b0 < 32 ? (int)(B - b0) : 32, j0 = c * (Q / 4);
    const int kk = wave & 3, jt = j0 / 32 + (wave >> 2);
    const bool work = jt * 32 < j0 + Q / 4;

    // x in whole lines (taken as operands, 32 rows to a load, the launch was 8.6 us for 32 rows of 256 x 1024 blocks)
    constexpr int XN = (T4 + 1) / 2;  // 64 pieces of each of a wave's four rows
    const int pieces = P / 2;         // of a row
    const auto rx = buffer_at(x + b0 * 4 * P);
    u32x4 xv[4][XN];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int n = 0; n < XN; ++n)
            xv[i][n] = __builtin_amdgcn_raw_buffer_load_b128(rx, wave * 4 + i < rows && n * 64 + lane < pieces ? (n * 64 + lane) * 16u : kNowhere,
                                                             (uint32_t)(wave * 4 + i) * (8u * P), 0);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 lf[4 * K4], lf2[DIRECT ? 4 * K4 : 1];
    const uint32_t l_at = DIRECT ? (uint32_t)(ln * Q) * 2u : lane * 16u, l_step = DIRECT ? 32u : 1024u;
    const auto rl = buffer_at(DIRECT ? LF2 + ((size_t)c * S + lt * 32) * Q : LF2 + (size_t)(c * LT + lt) * KS * 512);
    if (wave == 0) {
#pragma unroll
        for (int ks = 0; ks < 4 * K4; ++ks) {
            lf[ks] = __builtin_amdgcn_raw_buffer_load_b128(rl, ks < KS ? l_at : kNowhere, ks * l_step, 0);
            if constexpr (DIRECT) lf2[ks] = __builtin_amdgcn_raw_buffer_load_b128(rl, ks < KS ? l_at : kNowhere, ks * l_step + 16u, 0);
        }
    }
    auto put = [&] {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (wave * 4 + i >= rows) break;
#pragma unroll
            for (int n = 0; n < XN; ++n) {
                const int pc = n * 64 + lane;
                if (pc < pieces) *reinterpret_cast<u32x4*>(xs + (pc * 32 + ((wave * 4 + i) ^ (pc & 31))) * 8) = xv[i][n];
            }
        }
    };
    if (!work) {
        put();
        lds_barrier();
    } else {
        const int T = P / 16;
        const auto rw = buffer_at(RF1 + (size_t)kk * Q * P);
        const uint32_t w_at = (uint32_t)jt * 1024u + lane * 16u;
        static_assert(!DIRECT || T4 <= 4, "a quarter of R's row is one line");
        u32x4 wf[4][DIRECT ? 1 : T4];
        RowPieces wr[DIRECT ? 4 : 1];
#pragma unroll
        for (int part = 0; part < 4; ++part) {
            const int lo = T * part / 4, n = T * (part + 1) / 4 - lo;
            if constexpr (DIRECT) {
                wr[part].fetch(rw, (uint32_t)(jt * 32 * P + 16 * lo) * 2u, 2u * P, 32, 2 * n, lane);
            } else {
#pragma unroll
                for (int t = 0; t < T4; ++t)
                    wf[part][t] = __builtin_amdgcn_raw_buffer_load_b128(rw, t < n ? w_at : kNowhere, (uint32_t)((lo + t) * QT) * 1024u, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        put();
        lds_barrier();
        f32x16 acc[4];
#pragma unroll
        for (int part = 0; part < 4; ++part) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[part][r] = 0.f;
            const int lo = T * part / 4, n = T * (part + 1) / 4 - lo;
            if constexpr (DIRECT) wr[part].turn(xs + P * 128 + wave * (int)(kTurnBytes / 2), lane);
#pragma unroll
            for (int t = 0; t < T4; ++t) {
                if (t >= n) continue;
                const int pc = (kk * T + lo + t) * 2 + h;
                const u32x4 w = DIRECT ? wr[DIRECT ? part : 0].v[t] : wf[part][DIRECT ? 0 : t];
                acc[part] = mfma32(as_bf16x8(w), as_bf16x8(lds128(xs + (pc * 32 + (ln ^ (pc & 31))) * 8)), acc[part]);
            }
        }
        // element 8 (r/4) + 4 h + r%4 of the tile is the vector's (kk, j): four j are half of a step's 16 bytes
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const int step = (jt * 32 + 8 * q4 + 4 * h - j0) / 4;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[0][4 * q4 + e] + acc[1][4 * q4 + e] + acc[2][4 * q4 + e] + acc[3][4 * q4 + e];
            if (jt * 32 + 8 * q4 + 4 * h >= j0 && step < KS)
                *reinterpret_cast<u32x2*>(Uf + ((step * 2 + (kk >> 1)) * 32 + ln) * 8 + (kk & 1) * 4) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        }
    }
    lds_barrier();
    if (wave != 0) return;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4 * K4; ++ks) {
        if constexpr (DIRECT) {  // of pairs 0 .. 7 those that half h brings: first values, then second ones (pack_fwd_piece)
            const u32x4 a = lf[ks], b = lf2[ks];
            const uint32_t d0 = h ? a[1] : a[0], d1 = h ? a[3] : a[2], d2 = h ? b[1] : b[0], d3 = h ? b[3] : b[2];
            lf[ks] = u32x4{pick_lo16(d0, d1), pick_lo16(d2, d3), pick_hi16(d0, d1), pick_hi16(d2, d3)};
        }
        if (ks < KS) acc = mfma32(as_bf16x8(lds128(Uf + ((ks * 2 + h) * 32 + ln) * 8)), as_bf16x8(lf[ks]), acc);
    }
    const int col = (lt * 32 + ln) * 4 + c;
    const float bv = bias ? __uint_as_float((uint32_t)bias[col] << 16) : 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r / 4) + 4 * h + r % 4;
        if (row >= rows) continue;
        const size_t at = (size_t)(b0 + row) * 4 * S + col;
        const float v = acc[r] + bv;
        if constexpr (ACT) {
            if (y_pre) y_pre[at] = (uint16_t)pack_bf16x2(v, v);
            const float a = gelu_f(v);
            y[at] = (uint16_t)pack_bf16x2(a, a);
        } else {
            y[at] = (uint16_t)pack_bf16x2(v, v);
        }
    }
}

struct SplitArgs {
    const uint16_t* x;
    SplitPack w;
    uint16_t *y, *U;
};
template <int NB, int NT, int AHEAD, int NG>
int launch_stage(const Problem& pb, int stage, const SplitArgs& a, hipStream_t st)
{
    unsigned blocks;
    if (stage == 1) {
        const SplitGrid gr = split_grid(pb.B, 32 * NB, 4 * ((pb.q / 32 + NT - 1) / NT), &blocks);
        constexpr bool kTurn = NT > 1;  // many tiles: launch_factor
        const size_t lds = pb.ws_packed() ? split_stage1_lds<NB, NT, kTurn>() : split_stage1_lds<NB, NT, true>();
        auto kern = pb.ws_packed() ? split_stage1_kernel<NB, NT, NG, AHEAD, false, kTurn> : split_stage1_kernel<NB, NT, NG, AHEAD, true, kTurn>;
        SplitPack w = a.w;
        w.blocks = (int)blocks;
        if (!pb.ws_packed()) blocks += (unsigned)((w.pieces + 255) / 256);
        if (hipError_t e = allow_dynamic_lds((const void*)kern, lds)) return hip_status(e);
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, st, a.x, w, a.U, pb.B, pb.p, pb.q, gr);
    } else {
        const SplitGrid gr = split_grid(pb.B, 32 * NB, (pb.s / 32 + NT - 1) / NT, &blocks);
        const size_t lds = (size_t)32 * NB * (NT * 128 + 8) * 2 * (pb.act && pb.y_pre ? 2 : 1);
        auto kern = pb.act ? split_stage2_kernel<NB, NT, NG, AHEAD, true> : split_stage2_kernel<NB, NT, NG, AHEAD, false>;
        if (hipError_t e = allow_dynamic_lds((const void*)kern, lds)) return hip_status(e);
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, st, (const uint16_t*)a.U, (const uint16_t*)a.w.LF2, (const uint16_t*)pb.bias,
                           a.y, (uint16_t*)pb.y_pre, pb.B, pb.q, pb.s, gr);
    }
    return hip_status(hipGetLastError());
}
template <int NB, int NT, int AHEAD>
int launch_steps(const Problem& pb, int stage, const SplitArgs& a, hipStream_t st)
{
    // K-steps of a wave: the longest quarter of p, all of q
    const int steps = stage == 1 ? (pb.p / 16 + 3) / 4 : pb.q / 16;
    switch ((steps + 3) / 4) {
        case 1: return launch_stage<NB, NT, AHEAD, 1>(pb, stage, a, st);
        case 2: return launch_stage<NB, NT, AHEAD, 2>(pb, stage, a, st);
        case 3: return launch_stage<NB, NT, AHEAD, 3>(pb, stage, a, st);
        case 4: return launch_stage<NB, NT, AHEAD, 4>(pb, stage, a, st);
    }
    return -2;
}

// 32 x 32 tiles with all their loads in flight while they give every CU at most two workgroups, 32 x 64 beyond (1024 -> 4096 ->
// 1024, both layers: 256 rows 20 and 25 us, 512 rows 26 and 25, 1531 rows 49 and 39; 64 x 64 and 64 x 128 tiles 46 and 48).
int launch_factor(const Problem& pb, int stage, const SplitArgs& a, hipStream_t st)
{
    const int64_t tiles = (pb.B + 31) / 32 * (stage == 1 ? pb.kq() / 32 : pb.s / 32);
    return tiles <= 512 ? launch_steps<1, 1, 4>(pb, stage, a, st) : launch_steps<1, 2, 2>(pb, stage, a, st);
}

// split_once_kernel has waves for two 32-row tiles of R in a quarter c q/4 .. (c + 1) q/4.  Of the multiples of 32 up
// to 256 only q = 224 has quarters that touch three (56 .. 111 and 112 .. 167).
constexpr bool once_covers(int q)
{
    for (int c = 0; c < 4; ++c)
        if (((c + 1) * q / 4 - 1) / 32 - c * q / 4 / 32 > 1) return false;
    return true;
}
static_assert(once_covers(32) && once_covers(64) && once_covers(96) && once_covers(128) && once_covers(160) && once_covers(192) && !once_covers(224) &&
              once_covers(256));

// Where one launch does for both factors (split_once_kernel): packed weights, p up to 256, one row tile, two where the
// quarter of R is small.  Weights as they are where no call packs them for the next, with q up to 128 and p up to 256,
// two row tiles; two launches and one, host included, us: blocks of 96 x 96 and 384 x 96 (width 384 -> 1536), 8 rows 8.7
// and 5.2, 64 rows 8.7 and 6.2; 96 x 96 twice, 64 rows 7.0 and 5.3; 128 x 272 and 160 x 128, 64 rows 7.3 and 7.2; 96 x 384
// and 96 x 96, 8 rows 7.4 and 8.0, 64 rows 7.3 and 8.7.
bool once_direct(const Problem& pb) { return !fwd_frag_supported(pb) && pb.q <= 128 && pb.p <= 256 && pb.B <= 64; }
bool once_preferred(const Problem& pb)
{
    return once_covers(pb.q) && (once_direct(pb) || (pb.ws_packed() && pb.p <= 256 && pb.B <= (pb.p * pb.q <= 192 * 192 ? 64 : 32)));
}
// T4, 4 K4: K-steps of a quarter of the first contraction and of the second
template <int T4, int K4, bool DIRECT>
int launch_once(const Problem& pb, const SplitArgs& a, hipStream_t st)
{
    auto kern = pb.act ? split_once_kernel<T4, K4, true, DIRECT> : split_once_kernel<T4, K4, false, DIRECT>;
    const dim3 grid((unsigned)((pb.s / 32 + 1) / 2 * 8), (unsigned)((pb.B + 31) / 32));
    const size_t lds = (size_t)K4 * 4096 + (size_t)pb.p * 256 + (DIRECT ? 8 * kTurnBytes : 0);
    if (hipError_t e = allow_dynamic_lds((const void*)kern, lds)) return hip_status(e);
    hipLaunchKernelGGL(kern, grid, dim3(512), lds, st, a.x, DIRECT ? a.w.R : (const uint16_t*)a.w.RF1, DIRECT ? a.w.L : (const uint16_t*)a.w.LF2,
                       (const uint16_t*)pb.bias, a.y, (uint16_t*)pb.y_pre, pb.B, pb.p, pb.q, pb.s);
    return hip_status(hipGetLastError());
}
template <int T4>
int launch_once_steps(const Problem& pb, const SplitArgs& a, hipStream_t st)
{
    if (pb.q <= 128) return launch_once<T4, 2, false>(pb, a, st);
    return pb.q <= 192 ? launch_once<T4, 3, false>(pb, a, st) : launch_once<T4, 4, false>(pb, a, st);
}
int launch_once_any(const Problem& pb, const SplitArgs& a, hipStream_t st)
{
    if (once_direct(pb))
        return pb.p <= 128 ? launch_once<2, 2, true>(pb, a, st) : launch_once<4, 2, true>(pb, a, st);
    return pb.p <= 128 ? launch_once_steps<2>(pb, a, st) : pb.p <= 192 ? launch_once_steps<3>(pb, a, st) : launch_once_steps<4>(pb, a, st);
}

// Rows whose vector between the factors fits the static workspace behind the packed weights, so that monarch_fwd_static
// runs the same kernels as monarch_fwd_ws: what a call asks room for, no less for a longer batch than for a shorter
// one. A row takes q / 32 times 256 bytes.
int64_t fit_rows(const Problem& pb)
{
    const size_t packed = fwd_frag_packed(pb), row = (size_t)pb.kq() * 2, room = MONARCH_STATIC_WORKSPACE_BYTES;
    const int64_t fit = packed < room ? (int64_t)((room - packed) / row) : 0;
    return pb.B < fit ? pb.B : fit;
}
// Longer batches go in slices of about the same length: `n`, each but the last of `rows`, whole tiles.
struct Slices {
    int64_t n, rows;
};
Slices slices(const Problem& pb)
{
    const int64_t fit = fit_rows(pb), most = fit / 32 * 32;
    if (fit == pb.B) return Slices{1, pb.B};
    if (most == 0) return Slices{0, 0};
    const int64_t n = (pb.B + most - 1) / most;
    return Slices{n, ((pb.B + n - 1) / n + 31) / 32 * 32};
}
// Where they pay: every slice reads the weights again, in launches of its own, while the shape-generic kernels, which
// run otherwise, take the same time for any batch until their output is long.  Up to seven slices and 80 Mi output
// values; shape-generic kernels and slices, us: blocks of 256 x 256 and 256 x 512, 3360 rows (two slices) 64 and 26,
// 8192 rows (three) 66 and 49; 1024 x 256 and 256 x 2048, 4096 rows (four) 236 and 105; 256 x 256 and 256 x 3072, 3840
// rows (five) 214 and 140, 4608 rows (six) 213 and 166, 6144 rows (eight) 214 and 219 to 235, 8192 rows (eleven) 214
// and 311; 1024 x 256 and 256 x 2880, 768 rows (four of 192) 286 and 68, 8192 rows (43) 287 and 675; longer outputs,
// 256 x 192 and 192 x 4096, 5120 rows (five, 80 Mi) 211 and 190, 6528 rows (six) 211 and 258; 128 x 128 and 128 x 4096,
// 5120 rows (two, 80 Mi) 141 and 114, 7936 rows (two) 161 and 175.  The shapes with a fused kernel never have more than
// two.
bool slices_pay(const Problem& pb)
{
    const int64_t n = slices(pb).n;
    return n == 1 || (n > 0 && n <= 7 && pb.B * pb.n_out() <= (80 << 20));
}

}  // namespace

bool fwd_split_supported(const Problem& pb)  // a wave holds 16 K-steps at most
{
    return pb.dtype == 1 && pb.k == 4 && !pb.perm_b() && pb.p % 16 == 0 && pb.q % 32 == 0 && pb.s % 32 == 0 && pb.p <= 1024 &&
           pb.q <= 256;
}

// Where there is a fused kernel, which takes the same time for any number of row tiles that leaves CUs idle: up to 3072
// rows, 4352 where the output is narrower than the input, 2048 for wider outputs of more than 128 columns a block.  us,
// the fused kernel first, without packed weights and with them: 768 -> 3072 with the nonlinearity, 2000 rows 22.8 and
// 18.4, 16.0 and 14.6, 2500 rows 23.1 and 22.6, 16.2 and 18.7; 1024 -> 4096, 1500 rows 26.7 and 22.2, 20.5 and 16.5,
// 2500 rows 27.9 and 29.4, 21.6 and 22.9; 512 -> 2048, 3000 rows 21.8 and 17.3, 17.1 and 14.2, 4000 rows 22.2 and 21.2,
// 17.1 and 18.0; 4096 -> 1024, 2500 rows 43.1 and 22.7, 37.1 and 20.5, 4000 rows (two slices) 43.2 and 37.1, 37.8 and
// 35.2, 5000 rows 43.6 and 43.6, 38.5 and 40.9; 3072 -> 768, 4000 rows 30.5 and 21.5, 25.1 and 19.2, 5000 rows (two
// slices) 30.7 and 31.3, 25.3 and 28.0; 2048 -> 512, 4000 rows 19.3 and 13.1, 12.9 and 12.7, 5000 rows 19.4 and 15.8,
// 12.9 and 15.0; 768 -> 768, 3000 rows 17.6 and 12.9, 12.9 and 12.2; 1024 -> 1024 21.9 and 16.1, 16.5 and 14.2; 512 ->
// 512 11.9 and 9.5, 7.9 and 9.1.  Where the other choice is the shape-generic kernel (width 384: 47 us for 300 rows, 60
// for 8000), up to 8192.
bool fwd_split_preferred(const Problem& pb)
{
    const int64_t most = !fwd_frag_supported(pb) ? 8192 : pb.s < pb.p ? 4352 : pb.s > pb.p && pb.q > 128 ? 2048 : 3072;
    return fwd_split_supported(pb) && pb.B > 0 && pb.B <= most && slices_pay(pb);
}

size_t fwd_split_mid_bytes(const Problem& pb) { return align_up((size_t)fit_rows(pb) * pb.kq() * 2, 256); }

int fwd_split(const Problem& given, const void* x, const void* R, const void* L, uint16_t* RF1, uint16_t* LF2, void* y, void* U,
              hipStream_t st)
{
    Problem pb = given;
    const int64_t rows = slices(given).rows;
    for (int64_t b = 0; b < given.B; b += rows) {
        pb.B = given.B - b < rows ? given.B - b : rows;
        const size_t to = (size_t)b * pb.n_out();
        if (given.y_pre) pb.y_pre = (uint16_t*)given.y_pre + to;
        const SplitArgs a{(const uint16_t*)x + (size_t)b * pb.n_in,
                          SplitPack{(const uint16_t*)R, (const uint16_t*)L, RF1, LF2, pb.s, (int)((pb.n_R() + pb.n_L()) / 8), 0}, (uint16_t*)y + to,
                          (uint16_t*)U};
        int rc;
        if (once_preferred(pb)) {
            rc = launch_once_any(pb, a, st);
        } else {
            rc = launch_factor(pb, 1, a, st);
            if (!rc) rc = launch_factor(pb, 2, a, st);
        }
        if (rc) return rc;
        pb.flags |= MONARCH_FLAG_WS_PACKED;  // the first slice has packed the weights
    }
    return 0;
}

}  // namespace monarch
