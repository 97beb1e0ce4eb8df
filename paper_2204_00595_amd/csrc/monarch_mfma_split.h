// Shared by the forward and backward of the four-block layers on short batches (monarch_mfma_fwd_split.hip,
// monarch_mfma_bwd_split.hip): tile products straight from memory, the dealing of row tiles, the first factor.
#pragma once
#include "monarch_internal.h"
#include "monarch_mfma_common.h"

namespace monarch {
namespace {

constexpr uint32_t kNowhere = 0xffffffffu;  // a load there reads zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void* p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7fffffffu, 0x00020000);
}

// 32 rows x 128 bytes of a matrix in memory -> a lane's four 16-byte pieces 2 i + lane / 32 of row lane % 32, which is
// how the MFMAs want them.  Loaded like that a load touches 32 rows and takes the L1 62 cycles (rows of 1024, 2048 or
// 3072 bytes); with eight lanes on the 128 bytes of a row it takes 20, and the pieces change places through LDS that
// the wave owns.
constexpr int kTurnRow = 72;                            // bf16 values of a row there: an odd number of 16-byte units
constexpr size_t kTurnBytes = 32 * kTurnRow * 2;        // per wave
struct RowPieces {
    u32x4 v[4];
    // at: byte offset of the first row's 128 bytes; ld: bytes of a row; rows: rows there are; pieces: 16-byte pieces
    // there are (even)
    __device__ __forceinline__ void fetch(__amdgpu_buffer_rsrc_t rs, uint32_t at, uint32_t ld, int rows, int pieces, int lane)
    {
        const uint32_t mine = at + (uint32_t)(lane >> 3) * ld + (lane & 7) * 16;
        const bool in = (lane & 7) < pieces;
#pragma unroll
        for (int n = 0; n < 4; ++n)
            v[n] = __builtin_amdgcn_raw_buffer_load_b128(rs, in && (lane >> 3) + 8 * n < rows ? mine : kNowhere, (uint32_t)(8 * n) * ld, 0);
    }
    __device__ __forceinline__ void turn(uint16_t* lds, int lane)
    {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int n = 0; n < 4; ++n) *reinterpret_cast<u32x4*>(lds + ((lane >> 3) + 8 * n) * kTurnRow + (lane & 7) * 8) = v[n];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = lds128(lds + (lane & 31) * kTurnRow + (2 * i + (lane >> 5)) * 8);
        __builtin_amdgcn_wave_barrier();
    }
};

// acc[nb][nt] += (32 rows nb) x (32 columns nt) over `steps` K-steps, at most 4 * NG.  a_at / w_at: byte offsets of
// this lane's first piece (kNowhere: a row or tile that does not exist), a_step / w_step: from one K-step to the next;
// W_FIRST: the weights are the first MFMA operand (the result is transposed).  Loads are issued four K-steps at a time,
// `AHEAD` such groups ahead; the trip count is a template parameter because loads past the end, even of nothing, cost
// as much as real ones.
// TURN (NB = 1): the rows, of a_ld bytes, are read in whole lines (RowPieces); a_at is the uniform offset of the first.
// W_TURN: so are the weights, whose rows have w_step bytes; w_at is the uniform offset of each tile's first row.
template <int NB, int NT, int NG, int AHEAD, bool W_FIRST, bool TURN, bool W_TURN>
__device__ __forceinline__ void tile_product(const void* a, const uint32_t (&a_at)[NB], uint32_t a_step, const void* w, const uint32_t (&w_at)[NT],
                                             uint32_t w_step, int steps, f32x16 (&acc)[NB][NT], uint32_t a_ld, int rows, uint16_t* lds)
{
    static_assert(!TURN || NB == 1, "one row tile");
    constexpr int G = 4, BUF = AHEAD < NG ? AHEAD : NG;
    const int lane = threadIdx.x & 63;
    const auto ra = buffer_at(a), rw = buffer_at(w);
    RowPieces af[BUF][NB], wf[BUF][NT];
    auto load = [&](int gr, int buf) {
        if constexpr (TURN) {
            af[buf][0].fetch(ra, a_at[0] + gr * (G * 32), a_ld, rows, 2 * (steps - gr * G), lane);
        } else {
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int d = 0; d < G; ++d)
                    af[buf][n].v[d] = __builtin_amdgcn_raw_buffer_load_b128(ra, gr * G + d < steps ? a_at[n] : kNowhere, (gr * G + d) * a_step, 0);
        }
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            if constexpr (W_TURN) {
                wf[buf][n].fetch(rw, w_at[n] + gr * (G * 32), w_step, w_at[n] == kNowhere ? 0 : 32, 2 * (steps - gr * G), lane);
            } else {
#pragma unroll
                for (int d = 0; d < G; ++d)
                    wf[buf][n].v[d] = __builtin_amdgcn_raw_buffer_load_b128(rw, gr * G + d < steps ? w_at[n] : kNowhere, (gr * G + d) * w_step, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int gr = 0; gr < BUF; ++gr) load(gr, gr);
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
        if constexpr (TURN) af[gr % BUF][0].turn(lds, lane);
        if constexpr (W_TURN) {
#pragma unroll
            for (int n = 0; n < NT; ++n) wf[gr % BUF][n].turn(lds, lane);
        }
#pragma unroll
        for (int d = 0; d < G; ++d)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = W_FIRST ? mfma32(as_bf16x8(wf[gr % BUF][j].v[d]), as_bf16x8(af[gr % BUF][i].v[d]), acc[i][j])
                                        : mfma32(as_bf16x8(af[gr % BUF][i].v[d]), as_bf16x8(wf[gr % BUF][j].v[d]), acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        if (gr + BUF < NG) load(gr + BUF, gr % BUF);
    }
}

struct SplitGrid {
    int row_tiles, inner, deal;  // deal: row tiles belong to XCDs (their x, U and y meet in one L2)
};
__device__ __forceinline__ bool split_index(const SplitGrid& gr, int bid, int& rt, int& in)
{
    const int seq = gr.deal ? bid >> 3 : bid;
    rt = gr.deal ? (seq / gr.inner) * 8 + (bid & 7) : seq / gr.inner;
    in = seq % gr.inner;
    return rt < gr.row_tiles;
}

// Step 1 for one workgroup: Y1 of 32 * NB rows, block kk, NT column tiles of 32.  The four waves share out the
// contraction, so that every byte of x and R the workgroup needs is loaded once, and add up their tiles through LDS
// (split_stage1_lds bytes).
// DIRECT: W is R as it is, read in whole lines, else the packed copy RF1.  TURN: so is x.  NATURAL: out[b][kk*Q + j],
// else the order the packed L contracts, (j/4, kk, j%4), in MFMA fragments: out[b/32][j/4][h][row][e] = element 8 h + e
// of the 16 (kk, j%4) of row b % 32, with no more rows in the last tile than there are.
// R as it is in 16-byte pieces of 32 of its rows held the address path of the L1 up three times as long as the packed
// copy: blocks of 256 x 1024, 2000 rows 21.5 us, in whole lines 14.2, 300 rows 11.0 and 7.4; of 256 x 256, 2000 rows 9.3
// and 8.2.
template <int NB, int NT, bool LINES>
constexpr size_t split_stage1_lds() { return (size_t)4 * NB * NT * 4096 + (LINES ? 4 * kTurnBytes : 0); }
template <int NB, int NT, int NG, int AHEAD, bool DIRECT, bool NATURAL, bool TURN>
__device__ __forceinline__ void split_stage1(const uint16_t* __restrict__ x, const uint16_t* __restrict__ W, uint16_t* __restrict__ U,
                                             int64_t B, int P, int Q, const SplitGrid& gr, int bid, f32x4* part)
{
    int rt, in;
    if (!split_index(gr, bid, rt, in)) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, ln = lane & 31, g = lane >> 5;
    const int QT = Q / 32, groups = gr.inner / 4;
    const int kk = in / groups, jt0 = (in % groups) * NT;
    const int64_t b0 = (int64_t)rt * 32 * NB;
    const int rows = B - b0 < 32 * NB ? (int)(B - b0) : 32 * NB;
    const int T = P / 16, lo = T * wave / 4, hi = T * (wave + 1) / 4;

    f32x16 acc[NB][NT];
    uint32_t a_at[NB], w_at[NT];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int i = 0; i < NB; ++i)
        a_at[i] = TURN ? (uint32_t)(32 * lo) : i * 32 + ln < rows ? (uint32_t)(((i * 32 + ln) * 4 * P + 16 * lo + 8 * g) * 2) : kNowhere;
#pragma unroll
    for (int j = 0; j < NT; ++j)
        w_at[j] = jt0 + j >= QT ? kNowhere
                : DIRECT ? (uint32_t)(((jt0 + j) * 32 * P + 16 * lo) * 2)
                           : (uint32_t)((lo * QT + jt0 + j) * 1024 + lane * 16);
    tile_product<NB, NT, NG, AHEAD, true, TURN, DIRECT>(
        x + b0 * 4 * P + kk * P, a_at, 32u, W + (size_t)kk * Q * P, w_at, DIRECT ? (uint32_t)(2 * P) : (uint32_t)QT * 1024, hi - lo, acc,
        (uint32_t)(8 * P), rows, reinterpret_cast<uint16_t*>(part + 4 * NB * NT * 256) + wave * (int)(kTurnBytes / 2));

    // wave w keeps the four columns j = 8 * w + 4 * g .. of every tile
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                part[(((wave * NB + i) * NT + j) * 4 + q4) * 64 + lane] =
                    f32x4{acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]};
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            f32x4 v = part[((i * NT + j) * 4 + wave) * 64 + lane];
#pragma unroll
            for (int o = 1; o < 4; ++o) {
                const f32x4 t = part[(((o * NB + i) * NT + j) * 4 + wave) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += t[e];
            }
            const int row = i * 32 + ln, col = (jt0 + j) * 32 + 8 * wave + 4 * g;
            const u32x2 o = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            if constexpr (NATURAL) {
                if (row < rows && jt0 + j < QT) *reinterpret_cast<u32x2*>(U + (b0 + row) * 4 * Q + kk * Q + col) = o;
            } else if (row < rows && jt0 + j < QT) {
                const int tall = rows - i * 32 < 32 ? rows - i * 32 : 32;  // rows of the tile
                *reinterpret_cast<u32x2*>(U + (b0 + i * 32) * 4 * Q + (((col >> 2) * 2 + (kk >> 1)) * tall + ln) * 8 + (kk & 1) * 4) = o;
            }
        }
}

inline SplitGrid split_grid(int64_t B, int rows, int inner, unsigned* blocks)
{
    const int tiles = (int)((B + rows - 1) / rows), even = (tiles + 7) / 8 * 8;
    SplitGrid gr{tiles, inner, 5 * even <= 6 * tiles};
    *blocks = (unsigned)((gr.deal ? even : tiles) * inner);
    return gr;
}

}  // namespace
}  // namespace monarch
