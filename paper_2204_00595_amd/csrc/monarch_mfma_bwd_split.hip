// bf16 backward of the four-block layers on batches too short to fill the chip with 64-row tiles of the data kernel of
// monarch_mfma_bwd_wide.hip: one launch per adjoint factor, so that the weights are spread over all CUs.
//
// With the vector between the factors kept in its permuted order, dU[b][4j + kk] = dY1[b][kk][j], both adjoint steps
// are one operation: the input has its four blocks interleaved, the output has them one after the other,
//     out[b][g*N + n] = sum_m in[b][4m + g] W[g][m][n]
//   dU from dy:  W = L (m = l, n = r; g*N + n = c*q + r is the permuted position)
//   dx from dU:  W = R (m = j, n = i)
//
//   prep     transposed fragments of L and R (below), the recomputed Y1 (split_stage1, which reads R as it is), as workgroups
//            of one launch
//   adjoint  workgroup = (32 rows, NT column tiles of 32 of all four blocks): the waves share out the contraction, a K-step of
//            16 m is one whole 128-byte line per row, picked apart in registers; the waves' tiles are added up through LDS,
//            wave g keeps block g
//   wgrad    as in the wide backward (monarch_mfma_wgrad.hip), with dU as the interleaved operand of dR
//
// Fragments: WT[g][nt][t][lane][e] = W[g][16t + 4*(e/2) + 2*(lane/32) + e%2][32*nt + lane%32]: lane half h holds, of
// the 16 m of a step, the pairs that its 16-byte pieces 2i + h of the line bring.
//
// What bounds it: latency for a few row tiles (three launches of about 5 us), the address path of the L1 above; the
// rows come in whole lines that change places through LDS (RowPieces; training step of the feed-forward block of width
// 1024, 2000 rows: 224 -> 196 us, of width 768 169 -> 150, 200 rows 106 -> 99).  Measured, GPU time of a training step,
// before there were these kernels, with them, and with R in whole lines and two or three workgroups of `adjoint` to a
// CU: the feed-forward block of width 1024, 1000 rows 262, 153 and 122 us, 2000 rows 189 (with them) and 165; of width
// 384, 1500 rows 98 and 91.
#include "monarch_internal.h"
#include "monarch_mfma_common.h"
#include "monarch_mfma_split.h"
#include "monarch_colsum.h"
#include "monarch_act.h"

namespace monarch {
namespace {

struct BwdPrep {
    const uint16_t *x, *R, *L;
    uint16_t *Y1, *LT, *RT;
    int P, Q, S;
    int y1_blocks;  // workgroups of the recompute (none where the forward saved the vector), then those of the packing
};

// one 16-byte piece of the transposed fragments of W (4 blocks of M x N)
__device__ __forceinline__ void pack_adjoint_piece(const uint16_t* __restrict__ W, uint16_t* __restrict__ WT, int M, int N, int pc)
{
    const int lane = pc & 63;
    int rest = pc >> 6;
    const int T = M / 16, NTT = N / 32;
    const int t = rest % T; rest /= T;
    const int nt = rest % NTT, g = rest / NTT;
    const uint16_t* src = W + ((size_t)g * M + 16 * t + 2 * (lane >> 5)) * N + 32 * nt + (lane & 31);
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = (uint32_t)src[(size_t)(4 * i) * N] | ((uint32_t)src[(size_t)(4 * i + 1) * N] << 16);
    *reinterpret_cast<u32x4*>(WT + (size_t)pc * 8) = o;
}

template <int NT, int NG>
__global__ void __launch_bounds__(256)
bwd_split_prep_kernel(const BwdPrep w, int64_t B, SplitGrid gr)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char split_lds[];
    int bid = (int)blockIdx.x;
    if (bid < w.y1_blocks) {
        split_stage1<1, NT, NG, 4 / NT, true, true, (NT > 1)>(w.x, w.R, w.Y1, B, w.P, w.Q, gr, bid, reinterpret_cast<f32x4*>(split_lds));
        return;
    }
    bid -= w.y1_blocks;
    const int nL = 4 * w.S * w.Q / 8, nR = 4 * w.Q * w.P / 8, pc = bid * 256 + (int)threadIdx.x;
    if (pc < nL) pack_adjoint_piece(w.L, w.LT, w.S, w.Q, pc);
    else if (pc < nL + nR) pack_adjoint_piece(w.R, w.RT, w.Q, w.P, pc - nL);
}

// NS: K-steps of a wave, at most (see tile_product).  ACT: the result is multiplied by gelu'(x_pre).
// The bounds on the registers keep two workgroups to a CU, three where the loads are few: left alone, the compiler kept
// copies of the sums and took 290, for one (256 rows of dU x 1024 columns, 2000 rows: 27.4 us, now 17.0; with the
// nonlinearity's factor, 700 rows 17.2, now 13.0).
template <int NT, int NS, bool ACT>
__global__ void __launch_bounds__(256, NT == 1 && NS <= 4 ? 3 : 2)
adjoint_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ WT, uint16_t* __restrict__ out,
               const uint16_t* __restrict__ x_pre, int64_t B, int M, int N, SplitGrid gr)
{
    constexpr int AHEAD = NT == 1 ? 3 : 2, BUF = AHEAD < NS ? AHEAD : NS;
    extern __shared__ __attribute__((aligned(16))) unsigned char split_lds[];
    f32x4* const part = reinterpret_cast<f32x4*>(split_lds);
    int rt, ng;
    if (!split_index(gr, (int)blockIdx.x, rt, ng)) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, ln = lane & 31, h = lane >> 5;
    const int NTT = N / 32, nt0 = ng * NT, T = M / 16;
    const int lo = T * wave / 4, steps = T * (wave + 1) / 4 - lo;
    const int64_t b0 = (int64_t)rt * 32;
    const int rows = B - b0 < 32 ? (int)(B - b0) : 32;

    const auto ra = buffer_at(in + b0 * 4 * M), rw = buffer_at(WT);
    uint16_t* const turn = reinterpret_cast<uint16_t*>(split_lds) + wave * (int)(kTurnBytes / 2);
    uint32_t w_at[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) w_at[j] = nt0 + j < NTT ? (uint32_t)(((nt0 + j) * T + lo) * 1024 + lane * 16) : kNowhere;
    const uint32_t w_block = (uint32_t)NTT * T * 1024;

    f32x16 acc[4][NT];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[g][j][r] = 0.f;

    RowPieces af[BUF];
    u32x4 wf[BUF][4][NT];
    auto load = [&](int t, int buf) {
        af[buf].fetch(ra, (uint32_t)((lo + t) * 128), (uint32_t)(8 * M), rows, t < steps ? 8 : 0, lane);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const uint32_t w = t < steps ? w_at[j] : kNowhere;
#pragma unroll
            for (int g = 0; g < 4; ++g) wf[buf][g][j] = __builtin_amdgcn_raw_buffer_load_b128(rw, w, g * w_block + t * 1024, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int t = 0; t < BUF; ++t) load(t, t);
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        af[t % BUF].turn(turn, lane);
        const u32x4(&a)[4] = af[t % BUF].v;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            // a piece holds m0: c0 c1 | c2 c3, m1: c0 c1 | c2 c3
            u32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (g & 1) ? pick_hi16(a[i][g >> 1], a[i][2 + (g >> 1)]) : pick_lo16(a[i][g >> 1], a[i][2 + (g >> 1)]);
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[g][j] = mfma32(as_bf16x8(wf[t % BUF][g][j]), as_bf16x8(v), acc[g][j]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (t + BUF < NS) load(t + BUF, t % BUF);
    }

    auto at = [&](int j, int q4) { return (size_t)(b0 + ln) * 4 * N + wave * N + (nt0 + j) * 32 + 8 * q4 + 4 * h; };
    u32x2 pre[ACT ? NT : 1][4];  // what the results of block `wave` are multiplied with
    lds_barrier();  // the sums take the place of the rows
    // the waves' sums: wave w hands two blocks to wave w ^ 2, then one to wave w ^ 1, and keeps block w
    auto slot = [&](int owner, int g, int j, int q4) { return (((owner * 2 + g) * NT + j) * 4 + q4) * 64 + lane; };
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        const int bit = 2 >> round;
        if (ACT && round) {  // on its way during the second round: before the first there are no registers for it
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    pre[j][q4] = ln < rows && nt0 + j < NTT ? *reinterpret_cast<const u32x2*>(x_pre + at(j, q4)) : u32x2{0, 0};
        }
        if (round) lds_barrier();  // the first round's values have been read
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if ((round == 0 ? ((g ^ wave) & 2) == 2 : (g ^ wave) == 1))
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4)
                        part[slot(wave ^ bit, g & (bit - 1), j, q4)] = f32x4{acc[g][j][4 * q4], acc[g][j][4 * q4 + 1], acc[g][j][4 * q4 + 2], acc[g][j][4 * q4 + 3]};
        }
        lds_barrier();
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if ((round == 0 ? ((g ^ wave) & 2) == 0 : g == wave))
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const f32x4 v = part[slot(wave, g & (bit - 1), j, q4)];
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[g][j][4 * q4 + e] += v[e];
                    }
        }
    }
    if (ln >= rows) return;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (g != wave) continue;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if (nt0 + j >= NTT) continue;
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                float v[4] = {acc[g][j][4 * q4], acc[g][j][4 * q4 + 1], acc[g][j][4 * q4 + 2], acc[g][j][4 * q4 + 3]};
                if constexpr (ACT) {
                    const u32x2 u = pre[j][q4];
                    v[0] *= gelu_grad_f(__uint_as_float(u[0] << 16));
                    v[1] *= gelu_grad_f(__uint_as_float(u[0] & 0xffff0000u));
                    v[2] *= gelu_grad_f(__uint_as_float(u[1] << 16));
                    v[3] *= gelu_grad_f(__uint_as_float(u[1] & 0xffff0000u));
                }
                *reinterpret_cast<u32x2*>(out + at(j, q4)) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            }
        }
    }
}

template <int NT, int NS>
int launch_adjoint(const uint16_t* in, const uint16_t* WT, uint16_t* out, const uint16_t* x_pre, int64_t B, int M, int N, hipStream_t st)
{
    unsigned blocks;
    const SplitGrid gr = split_grid(B, 32, (N / 32 + NT - 1) / NT, &blocks);
    constexpr size_t lds = (size_t)NT * 8 * 4096;
    auto kern = x_pre ? adjoint_kernel<NT, NS, true> : adjoint_kernel<NT, NS, false>;
    if (hipError_t e = allow_dynamic_lds((const void*)kern, lds)) return hip_status(e);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, st, in, WT, out, x_pre, B, M, N, gr);
    return hip_status(hipGetLastError());
}
template <int NT>
int adjoint_steps(const uint16_t* in, const uint16_t* WT, uint16_t* out, const uint16_t* x_pre, int64_t B, int M, int N, hipStream_t st)
{
    const int steps = (M / 16 + 3) / 4;
#define MONARCH_STEPS(NS) \
    if (steps <= NS) return launch_adjoint<NT, NS>(in, WT, out, x_pre, B, M, N, st);
    MONARCH_STEPS(1)
    MONARCH_STEPS(2)
    MONARCH_STEPS(3)
    MONARCH_STEPS(4)
    MONARCH_STEPS(6)
    MONARCH_STEPS(8)
    MONARCH_STEPS(12)
    MONARCH_STEPS(16)
#undef MONARCH_STEPS
    return -2;
}
int adjoint(const uint16_t* in, const uint16_t* WT, uint16_t* out, const void* x_pre, int64_t B, int M, int N, hipStream_t st)
{
    const int64_t tiles = (B + 31) / 32 * (N / 32);
    return tiles <= 512 ? adjoint_steps<1>(in, WT, out, (const uint16_t*)x_pre, B, M, N, st)
                        : adjoint_steps<2>(in, WT, out, (const uint16_t*)x_pre, B, M, N, st);
}

template <int NT>
int launch_prep(const BwdPrep& w, int64_t B, const SplitGrid& gr, unsigned blocks, hipStream_t st)
{
    constexpr size_t lds = split_stage1_lds<1, NT, true>();
    const int ng = ((w.P / 16 + 3) / 4 + 3) / 4;
    auto kern = ng == 1 ? bwd_split_prep_kernel<NT, 1> : ng == 2 ? bwd_split_prep_kernel<NT, 2>
              : ng == 3 ? bwd_split_prep_kernel<NT, 3> : bwd_split_prep_kernel<NT, 4>;
    if (hipError_t e = allow_dynamic_lds((const void*)kern, lds)) return hip_status(e);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, st, w, B, gr);
    return hip_status(hipGetLastError());
}

struct Plan {
    size_t y1, du, lt, rt, partL, partR, total;
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
    // dR[kk][j][i] = sum_b dU[b][4*j + kk] * x[b][kk*P + i]
    dr = WgradDesc{};
    dr.lda = pb.kq(); dr.a_g = 1; dr.deint = 1;
    dr.ldb = pb.n_in; dr.b_g = pb.p; dr.b_seg = 0; dr.seg_w = pb.p;
    dr.M = pb.q; dr.N = pb.p; dr.G = 4; dr.rows = pb.B;
}
// `room`: bytes there are; a plan with one chunk may need more
Plan make_plan(const Problem& pb, size_t room = SIZE_MAX)
{
    Plan pl{};
    WgradDesc dl, dr;
    fill_descs(pb, dl, dr);
    pl.ok = wgrad_tiles(dl) > 0 && wgrad_tiles(dr) > 0;
    if (!pl.ok) return pl;
    // batch chunks: as many as keep one workgroup per CU, of at least 64 rows (two pipeline steps of 32)
    int64_t z = 256 / (wgrad_tiles(dl) + wgrad_tiles(dr));
    const int64_t most = (pb.B + 63) / 64;
    z = z > most ? most : z;
    z = z < 1 ? 1 : z;
    const size_t act = align_up((size_t)pb.B * pb.kq() * 2, 256);
    for (;; z = pl.nz - 1) {
        pl.rows_per_chunk = (int)(((pb.B + z - 1) / z + 63) / 64 * 64);
        pl.nz = (int)((pb.B + pl.rows_per_chunk - 1) / pl.rows_per_chunk);
        size_t off = 0;
        pl.y1 = off; off += act;
        pl.du = off; off += act;
        pl.lt = off; off += align_up(pb.n_L() * 2, 256);
        pl.rt = off; off += align_up(pb.n_R() * 2, 256);
        pl.partL = off; off += align_up((size_t)pl.nz * pb.n_L() * 4, 256);
        pl.partR = off; off += align_up((size_t)pl.nz * pb.n_R() * 4, 256);
        pl.total = off;
        if (pl.total <= room || pl.nz == 1) return pl;
    }
}

}  // namespace

// Where there is a wide backward: up to 1536 rows for square layers, 1800 for others, and there further where the
// nonlinearity's factor comes with it (`act_split`), which costs the wide kernel the time of its products again.
// Training step on these kernels and on the wide one: blocks of 128, 1000 rows 36 and 38 us, 2000 rows 42 and 41; of
// 192, 1000 rows 43 and 44, 1600 rows 48 and 47; of 256, 1300 rows 50 and 51, 1600 rows 53 and 52; of 192 and 768, 1300
// rows 55 and 57, 2000 rows 62 and 60; of 256 and 1024, 1600 rows 71 and 74, 2500 rows 84 and 79; of 1024 and 256, 1600
// rows 75 and 76, 2000 rows 81 and 78; of 768 and 192, 1000 rows 52 and 55, 1600 rows 62 and 60; of the feed-forward
// block of width 1024, 2000 rows 164 and 173, 2500 rows 190 and 183; of 768, 2000 rows 134 and 135, 2500 rows 147 and
// 144; of 512, 2000 rows 100 and 105, 2500 rows 116 and 108.  Not for blocks of 64 alone (8 rows 19 and 18, 1000 rows
// 22 and 21).
// Where the other choice is the shape-generic bf16 kernel: up to 4096 rows for square layers (width 384, 6000 rows 61 and
// 65, 8000 rows 70 and 69).  For others as far as p + s goes, which that kernel's data path grows with while here every
// row tile costs its launches of workgroups: 16384 rows from p + s = 384 on (96 x 384 blocks, 6000 rows 69 and 76, 12000
// rows 90 and 117; 384 x 96 75 and 78, 112 and 124; 96 x 288 67 and 69, 88 and 100; the worst of 103 shapes, blocks of 320
// x 32 and 32 x 96, 8000 rows 41 and 36), 6144 from 128 on with q up to 128 (backward of 96 x 96 and 96 x 192, 6000 rows 43
// and 48, 14000 rows 64 and 54; of 160 x 96 and 96 x 32 40 and 40, 57 and 43), else 4096 (64 x 160 and 160 x 32, 6000 rows
// 43 and 41, 16384 rows 70 and 46).  Not where it is the shape-generic contractions (q = 256 with p or s = 1024), which
// hold the vectors between the factors in fp32.
bool bwd_split_preferred(const Problem& pb)
{
    const bool wide = bwd_wide_supported(pb);
    if ((!wide && !tiled_bwd_supported(pb)) || (wide && pb.p == 64 && pb.s == 64)) return false;
    const int both = pb.p + pb.s;
    const int64_t most = !wide ? (pb.p == pb.s ? 4096 : both >= 384 ? 16384 : both >= 128 && pb.q <= 128 ? 6144 : 4096)
                       : pb.p == pb.s ? 1536 : !pb.act_split ? 1800 : pb.s < pb.p ? 2200 : 2560;
    return pb.dtype == 1 && pb.k == 4 && !pb.perm_b() && pb.p % 32 == 0 && pb.q % 32 == 0 && pb.s % 32 == 0 && pb.p <= 1024 &&
           pb.s <= 1024 && pb.q <= 256 && pb.B > 0 && pb.B <= most && make_plan(pb).ok;
}

size_t bwd_split_workspace(const Problem& pb) { return make_plan(pb).total; }
size_t bwd_split_least(const Problem& pb) { return make_plan(pb, 0).total; }

int bwd_split(const Problem& pb, const void* dy, const void* x, const void* R, const void* L, void* dx, void* dR, void* dL, void* ws,
              hipStream_t st)
{
    const Plan pl = make_plan(pb, pb.ws_bytes);
    if (!pl.ok) return -2;
    char* w = (char*)ws;
    uint16_t *Y1 = (uint16_t*)(w + pl.y1), *dU = (uint16_t*)(w + pl.du), *LT = (uint16_t*)(w + pl.lt), *RT = (uint16_t*)(w + pl.rt);
    const int nt = (pb.B + 31) / 32 * (pb.kq() / 32) <= 512 ? 1 : 2;
    unsigned blocks = 0;
    SplitGrid gr{};
    if (!pb.saved) gr = split_grid(pb.B, 32, 4 * ((pb.q / 32 + nt - 1) / nt), &blocks);
    BwdPrep pr{(const uint16_t*)x, (const uint16_t*)R, (const uint16_t*)L, Y1, LT, RT, pb.p, pb.q, pb.s, (int)blocks};
    blocks += (unsigned)(((pb.n_R() + pb.n_L()) / 8 + 255) / 256);
    int rc = nt == 1 ? launch_prep<1>(pr, pb.B, gr, blocks, st) : launch_prep<2>(pr, pb.B, gr, blocks, st);
    if (!rc) rc = adjoint((const uint16_t*)dy, LT, dU, nullptr, pb.B, pb.s, pb.q, st);
    if (!rc) rc = adjoint(dU, RT, (uint16_t*)dx, pb.x_pre, pb.B, pb.q, pb.p, st);
    if (rc) return rc;

    WgradDesc dl, dr;
    fill_descs(pb, dl, dr);
    dl.A = (const uint16_t*)dy; dl.Bm = Y1; dl.P = (float*)(w + pl.partL); dl.out = dL;
    if (pb.saved) {  // in stage-2 order: group c owns the columns c*Q ..
        dl.Bm = (const uint16_t*)pb.saved;
        dl.b_g = pb.q; dl.b_seg = 0; dl.seg_w = pb.q;
    }
    dr.A = dU; dr.Bm = (const uint16_t*)x; dr.P = (float*)(w + pl.partR); dr.out = dR;
    dl.rows_per_chunk = dr.rows_per_chunk = pl.rows_per_chunk;
    // bf16 partial sums only where the kernels of long batches have several too, beyond 256 rows: up to there the
    // chunks of 64 rows would add a rounding (200 rows: dR and dL 2.34e-3 off float64 with fp32 sums, 2.88e-3 without;
    // from 257 rows on 2.88e-3 against 2.94e-3 in the chunks of 256)
    dl.p_bf16 = dr.p_bf16 = pb.wgrad_f32() || pb.B <= 256 ? 0 : 1;
    ColsumJob cj{};
    if (pb.dbias) {
        cj = wgrad_colsum_job(pb, pl.nz);
        dl.colsum = cj.part;
    }
    rc = wgrad_gemm_pair(dl, dr, pl.nz, st);
    return rc ? rc : wgrad_reduce_pair(dl, dr, pb.wgrad_f32(), pl.nz, st, pb.dbias ? &cj : nullptr);
}

}  // namespace monarch
