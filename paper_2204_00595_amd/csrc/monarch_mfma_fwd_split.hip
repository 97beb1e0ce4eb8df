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
    tile_product<NB, NT, NG, AHEAD, false, false>(U + b0 * 4 * Q + c * KS * rows * 16, a_at, (uint32_t)rows * 32, LF2 + (size_t)c * LT * KS * 512, w_at,
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
        constexpr size_t lds = split_stage1_lds<NB, NT, kTurn>();
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

}  // namespace

bool fwd_split_supported(const Problem& pb)  // a wave holds 16 K-steps at most
{
    return pb.dtype == 1 && pb.k == 4 && !pb.perm_b() && pb.p % 16 == 0 && pb.q % 32 == 0 && pb.s % 32 == 0 && pb.p <= 1024 &&
           pb.q <= 256;
}

// Where there is a fused kernel, up to 3072 rows (48 of its row tiles; it takes the same time for any number of them):
// 1024 -> 4096 -> 1024, both layers with the nonlinearity, 2600 rows 70 and 46 us; 768 -> 3072 alone 3500 rows 17.4 and
// 21.3, 3072 -> 768 28.0 and 27.0; 512 -> 2048 alone 13.2 and 15.3, 2048 -> 512 17.1 and 15.2.  Where the other choice
// is the shape-generic kernel (width 384: 47 us for 300 rows, 60 for 8000), up to 8192.  And only where it all fits the
// static workspace, so that monarch_fwd_static runs the same kernels as monarch_fwd_ws.
bool fwd_split_preferred(const Problem& pb)
{
    return fwd_split_supported(pb) && pb.B > 0 && pb.B <= (fwd_frag_supported(pb) ? 3072 : 8192) &&
           fwd_frag_packed(pb) + fwd_split_mid_bytes(pb) <= MONARCH_STATIC_WORKSPACE_BYTES;
}

size_t fwd_split_mid_bytes(const Problem& pb) { return align_up((size_t)pb.B * pb.kq() * 2, 256); }

int fwd_split(const Problem& pb, const void* x, const void* R, const void* L, uint16_t* RF1, uint16_t* LF2, void* y, void* U,
              hipStream_t st)
{
    const SplitArgs a{(const uint16_t*)x, SplitPack{(const uint16_t*)R, (const uint16_t*)L, RF1, LF2, pb.s, (int)((pb.n_R() + pb.n_L()) / 8), 0},
                      (uint16_t*)y, (uint16_t*)U};
    const int rc = launch_factor(pb, 1, a, st);
    return rc ? rc : launch_factor(pb, 2, a, st);
}

}  // namespace monarch
