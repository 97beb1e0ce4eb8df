// Weight gradients of the Monarch multiply as batched "TN" GEMMs on bf16 MFMA:
//
//     out[g][m][n] = sum_b  A[b][g, m] * Bm[b][g, n]            (contraction over the batch)
//
//   dL[c][l][r]  = sum_b dW[b][c][l] * U[b][c*q + r]     A = dy (column l*k + c),  Bm = U
//   dR[kk][j][i] = sum_b dY1[b][kk][j] * x[b][kk*p + i]  A = dY1,                  Bm = x
//
// (the adjoints of steps 2 and 1 of Section 3.3).  Both operands are stored batch-major, i.e.
// the contraction index is the slow one, so they are staged row-major in LDS and read back with
// the transposing LDS load of gfx950 (ds_read_b64_tr_b16), which hands every lane four consecutive
// batch rows of one feature: exactly the MFMA operand layout.
//
// One workgroup = four groups g, two waves per group (each takes every other 16-row K-step on its own
// accumulators: two waves per SIMD hide each other's staging and LDS latencies), a TM x TN tile of
// each group's output; the batch is split into chunks whose fp32 partial tiles are summed by
// `wgrad_reduce_kernel`, which also undoes the column order used for dL and converts to the
// output type.
//
// What bounds it: memory.  A further step of 32 rows costs what its rows take at 4 to 5 TB/s (768 -> 768: 1.1 us; from 50000 rows
// on the launch reads at 4.7 TB/s), and 9 us are the launch, the first rows' latency and the partial tiles, which all workgroups
// write at the same time.  To get there the work of a step is dealt out between its MFMAs (`multiply`), B goes into LDS without
// passing through registers, and the rows of the interleaved operand are read in whole lines (each wave load of its runs of 64
// bytes held the L1 up three times as long): rows staged by way of registers before the products, with fragments read in between,
// took 31.2 us where this takes 29.7 (768 -> 3072, 8192 rows; whole training step 101.4 -> 99.2), 80.4 + 76.3 where this takes
// 77.8 + 72.8 (feed-forward block of width 1024, 16384 rows; 551 -> 546).
//
// The bias gradient, the column sums of dy, comes with dL: a wave adds up the fragments of dy it multiplies (v_dot2
// against ones, five instructions for eight rows), in the tiles of the first columns n alone.  A pass of its own over
// dy cost more than the products slow down (GPU time of the training step of the feed-forward block of width 1024,
// 16384 rows: 583 -> 565 us; the launch that did it beside the weights' re-layout 26.9 + 11.6 -> 6.0 + 5.6, the two
// launches of products 153 -> 160; 768 -> 768, 12608 rows: 6.3 -> 3.0 against 24.2 -> 24.8).  The sums are off float64
// by 2.8e-8 (12608 rows), those of that pass were by 6.3e-8.
#include <type_traits>
#include "monarch_internal.h"
#include "monarch_mfma_common.h"
#include "monarch_mfma_stage1.h"
#include "monarch_lds_tr.h"
#include "monarch_colsum.h"

namespace monarch {

namespace {

constexpr int KB = 32;    // batch rows per pipeline step (two 16-row K-steps)
constexpr int NTHR = 512;  // eight waves per workgroup

// A load at this offset (past the end of the buffer, whatever is added to it) reads zeros; make_problem keeps KB rows of any
// operand below it.
constexpr uint32_t kNowhere = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void* p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7fffffffu, 0x00020000);
}

// MSPLIT = false: the two waves of a group split the K-steps (each keeps the whole TM x TN tile, summed at the end);
// MSPLIT = true (large tiles): they split the tile's rows m instead, each taking both K-steps of a pipeline step on
// its own half of the accumulators -- 128 x 128 per group in 2 x 128 accumulator registers, which halves the operand
// bytes fetched per flop against the 64 x 128 tile.
template <int TM, int TN, bool DEINT, bool SUMS, bool MSPLIT>
__device__ __forceinline__ void wgrad_gemm_body(const WgradDesc& d, const int tile, const int zi)
{
    constexpr int MT = TM / 32, NT = TN / 32;
    constexpr int MTW = MSPLIT ? MT / 2 : MT;  // m tiles of one wave
    static_assert(!MSPLIT || MT % 2 == 0, "row split");
    constexpr int ABUF = 4 * KB * TM * 2, BBUF = 4 * KB * TN * 2;  // bytes of a step's rows [4][KB][T]: two buffers of A, then three of B
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];

    // eight waves: wave = (group g, half kh); the two waves of a group each take one 16-row K-step of every
    // 32-row pipeline step on their own accumulators, which are summed through LDS at the end (MSPLIT: each
    // takes half of the tile's rows m over both K-steps, and nothing is summed)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int grp = wave & 3, kh = wave >> 2;
    const int tiles_n = d.N / TN;
    const int tiles_mn = (d.M / TM) * tiles_n;
    const int g0 = (tile / tiles_mn) * 4, tmn = tile % tiles_mn;
    const int m0 = (tmn / tiles_n) * TM, n0 = (tmn % tiles_n) * TN;
    const int64_t row_lo = (int64_t)zi * d.rows_per_chunk;
    int64_t row_hi = row_lo + d.rows_per_chunk;
    if (row_hi > d.rows) row_hi = d.rows;
    const int64_t nrows = row_hi > row_lo ? row_hi - row_lo : 0;

    // ---- per-thread load tasks (pieces of 16 bytes, side by side in a row) ----
    // Addresses are fixed for the whole chunk: byte offsets from the (uniform) first row of a step, LDS offsets inside a
    // buffer, and the row of the task inside a step.  B goes straight into LDS, 64 pieces side by side per wave; A by way of
    // registers, where a piece of the interleaved operand (two m of four groups) is picked apart.
    constexpr int A_PER = 4 * KB * TM / 8 / NTHR, B_PER = 4 * KB * TN / 8 / NTHR;
    static_assert(A_PER * NTHR * 8 == 4 * KB * TM && B_PER * NTHR * 8 == 4 * KB * TN, "every thread has the same tasks");
    u32x4 areg[2][A_PER];
    uint32_t pa[A_PER], pb[B_PER], la[A_PER];
    int ra[A_PER], rb[B_PER];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
#pragma unroll
    for (int t = 0; t < A_PER; ++t) {
        const int task = tid + t * NTHR;
        if (DEINT) {
            const int r = task / (TM / 2), u = task % (TM / 2);  // m = 2u, 2u + 1
            ra[t] = r;
            pa[t] = (uint32_t)(r * d.lda + m0 * 4 + g0 + 8 * u) * 2;
            la[t] = lds0 + r * TM * 2 + ((u >> 4) ^ run_key<TM>(r)) * 64 + (u & 15) * 4;
        } else {
            const int g = task / (KB * TM / 8), rem = task % (KB * TM / 8);
            const int r = rem / (TM / 8), u = rem % (TM / 8);
            ra[t] = g0 + g < d.G ? r : (1 << 30);  // a group past the last one: zeros
            pa[t] = (uint32_t)(r * d.lda + (g0 + g) * d.a_g + m0 + 8 * u) * 2;
            la[t] = lds0 + (g * KB + r) * TM * 2 + ((u >> 2) ^ run_key<TM>(r)) * 64 + (u & 3) * 16;
        }
    }
#pragma unroll
    for (int t = 0; t < B_PER; ++t) {
        const int task = tid + t * NTHR;  // its place in LDS; the piece that belongs there:
        const int g = task / (KB * TN / 8), rem = task % (KB * TN / 8);
        const int r = rem / (TN / 8), u = ((rem % (TN / 8) >> 2) ^ run_key<TN>(r)) * 4 + (rem & 3);
        const int n = n0 + 8 * u;
        rb[t] = g0 + g < d.G ? r : (1 << 30);
        pb[t] = (uint32_t)(r * d.ldb + (g0 + g) * d.b_g + (n / d.seg_w) * d.b_seg + (n % d.seg_w)) * 2;
    }

    // Rows r0 .. r0+KB-1 of the chunk; rows past its end load nothing and read as zeros: a buffer load at an offset
    // past the buffer's end.  A branch around each load instead makes the compiler lose count of the loads in flight
    // and wait for all of them.
    auto rows_left = [&](int64_t r0) { return nrows - r0 < KB ? (int)(nrows - r0) : KB; };
    auto load_a = [&](int64_t r0, int stg, int t) {
        const auto buf = buffer_at(d.A + (row_lo + r0) * d.lda);
        areg[stg][t] = __builtin_amdgcn_raw_buffer_load_b128(buf, ra[t] < rows_left(r0) ? pa[t] : kNowhere, 0, 0);
    };
    auto load_b = [&](int64_t r0, int bsel, int t) {
        const auto buf = buffer_at(d.Bm + (row_lo + r0) * d.ldb);
        auto to = (__attribute__((address_space(3))) unsigned char*)lds + 2 * ABUF + bsel * BBUF + (t * NTHR + wave * 64) * 16;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (__attribute__((address_space(3))) void*)to, 16,
                                                 rb[t] < rows_left(r0) ? pb[t] : kNowhere, 0, 0, 0);
    };
    // register stage -> buffer BUF of A; of an interleaved piece the two m of group c, side by side with the other lanes'
    auto store_a = [&](auto buf, int stg, int t, auto c) {
        constexpr int C = decltype(c)::value, OFF = decltype(buf)::value * ABUF;
        const u32x4& v = areg[stg][t];
        if constexpr (DEINT) {
            const uint32_t lo = v[C >> 1], hi = v[2 + (C >> 1)];
            lds_put32<OFF + C * KB * TM * 2>(la[t], (C & 1) ? pick_hi16(lo, hi) : pick_lo16(lo, hi));
        } else {
            lds_put128<OFF>(la[t], v);
        }
    };

    // ---- fragments ----
    // lane's address of run t of a row: the first row of a K-step is a multiple of 8, so the key depends on the lane alone
    uint32_t aat[MTW], bat[NT];
    {
        const int G = lane >> 4, j = lane & 15, row = (MSPLIT ? 0 : 16 * kh) + 8 * (G >> 1) + (j >> 2);
        const int in_run = 32 * (G & 1) + 8 * (j & 3);
#pragma unroll
        for (int t = 0; t < MTW; ++t)
            aat[t] = lds0 + (grp * KB + row) * TM * 2 + (((MSPLIT ? kh * MTW : 0) + t) ^ run_key<TM>(j >> 2)) * 64 + in_run;
#pragma unroll
        for (int t = 0; t < NT; ++t) bat[t] = lds0 + 2 * ABUF + (grp * KB + row) * TN * 2 + (t ^ run_key<TN>(j >> 2)) * 64 + in_run;
    }
    Frag fr[2][MTW + NT];
    // half H of fragment I (MTW of A, then NT of B) of K-step K from buffer BUF of A and buffer `bsel` of B
    auto read_half = [&](Frag (&f)[MTW + NT], auto buf, int bsel, auto kstep, auto i, auto half) {
        constexpr int I = decltype(i)::value, H = decltype(half)::value, ROW = 16 * decltype(kstep)::value + 4 * H;
        u32x2 v;
        if constexpr (I < MTW) v = lds_tr16<decltype(buf)::value * ABUF + ROW * TM * 2>(aat[I]);
        else v = lds_tr16<ROW * TN * 2>(bat[I - MTW] + bsel * BBUF);
        (H ? f[I].hi : f[I].lo) = v;
    };
    constexpr int READS = 2 * (MTW + NT);
    auto read = [&](Frag (&f)[MTW + NT], auto buf, int bsel, auto kstep, auto o) {
        constexpr int O = decltype(o)::value;
        read_half(f, buf, bsel, kstep, std::integral_constant<int, O / 2>{}, std::integral_constant<int, O % 2>{});
    };

    // column sums of A from the fragments of the products: eight rows of a feature per lane, a chain for each parity of the step
    float cs[2][MTW] = {};
    auto add_rows = [&](float& s, const bf16x8& f) {
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        const u32x4 v = __builtin_bit_cast(u32x4, f);
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t pair = v[w];  // (a bit cast of the element itself takes element 0)
            t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), bf16x2{(__bf16)1.f, (__bf16)1.f}, t, false);
        }
        s += t;
    };

    f32x16 acc[MTW * NT];
#pragma unroll
    for (int t = 0; t < MTW * NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;

    // products of one K-step, with `count` other operations dealt out between them: an MFMA takes 32 cycles, in which the wave
    // requests what comes next
    auto multiply = [&](const Frag (&f)[MTW + NT], int k, auto count, auto op) {
        constexpr int OPS = decltype(count)::value, TILES = MTW * NT;
        each<TILES>([&](auto tile_no) {
            constexpr int T = decltype(tile_no)::value;
            acc[T] = mfma32(f[MTW + T % NT].operand(), f[T / NT].operand(), acc[T]);  // (transposed: a lane holds runs of n of one m)
            if constexpr (SUMS && T % NT == 0) add_rows(cs[k][T / NT], f[T / NT].operand());
            each<(T + 1) * OPS / TILES - T * OPS / TILES>([&](auto o) { op(std::integral_constant<int, decltype(o)::value + T * OPS / TILES>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // Pipeline, one workgroup barrier per 32-row step s: past it the rows of step s+1 are in LDS for all waves and nobody reads
    // those of step s any more.  While the products of step s run, the fragments of step s+1 are read, its A buffer's
    // predecessor takes the rows of step s+2 from the registers, the B rows of step s+3 are requested into the buffer that B(s)
    // left, and the A rows of step s+4 into the registers just freed: two steps for memory to answer.  (MSPLIT: a step is two
    // K-steps, the fragments of the second are read during the products of the first, before the barrier.)  The loop body has
    // no branches (a step past the end of the chunk works on zeros): control flow here makes the compiler shuffle the
    // accumulators between blocks.
    constexpr int AN = A_PER, BN = B_PER;  // load instructions of a step
    constexpr int AW = DEINT ? 4 : 1;      // stores of a piece
    using Zero = std::integral_constant<int, 0>;
    using One = std::integral_constant<int, 1>;
    if (nrows > 0) {  // (uniform) an empty chunk touches no memory and yields a zero partial tile
    auto load_a_all = [&](int64_t r0, int stg) {
#pragma unroll
        for (int t = 0; t < A_PER; ++t) load_a(r0, stg, t);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto load_b_all = [&](int64_t r0, int bsel) {
#pragma unroll
        for (int t = 0; t < B_PER; ++t) load_b(r0, bsel, t);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto store_a_all = [&](auto buf, int stg) {
        each<AN * AW>([&](auto o) { store_a(buf, stg, decltype(o)::value / AW, std::integral_constant<int, decltype(o)::value % AW>{}); });
        __builtin_amdgcn_sched_barrier(0);
    };
    load_a_all(0, 0);
    load_b_all(0, 0);
    load_a_all(KB, 1);
    load_b_all(KB, 1);
    store_a_all(Zero{}, 0);
    load_a_all(2 * KB, 0);
    load_b_all(2 * KB, 2);  // in the order of the loop, or the compiler waits there for too much
    store_a_all(One{}, 1);
    load_a_all(3 * KB, 1);
    wait_vmcnt<3 * AN + 2 * BN>();  // B rows of step 0
    lds_barrier();
    each<READS>([&](auto o) { read(fr[0], Zero{}, 0, Zero{}, o); });
    lgkm_wait(fr[0]);
    int bsel = 0;  // buffer of the B rows of the step
    auto step = [&](int64_t r0, auto par) {
        constexpr int K = decltype(par)::value;
        using Next = std::integral_constant<int, K ^ 1>;
        const int bnext = bsel == 2 ? 0 : bsel + 1;
        Frag (&now)[MTW + NT] = fr[MSPLIT ? 1 : K];        // multiplied past the barrier
        Frag (&then)[MTW + NT] = fr[MSPLIT ? 0 : K ^ 1];   // read there
        if constexpr (MSPLIT) {
            multiply(then, K, std::integral_constant<int, READS>{}, [&](auto o) { read(now, par, bsel, One{}, o); });
            lgkm_wait(now);
        }
        // what was requested after the B rows of step s+1
        wait_vmcnt<2 * AN + BN>();
        lds_barrier();
        multiply(now, K, std::integral_constant<int, READS + AN * AW + AN + BN>{}, [&](auto o) {
            constexpr int O = decltype(o)::value, S = O - READS, L = S - AN * AW - BN;
            if constexpr (S < 0) read(then, Next{}, bnext, Zero{}, o);
            else if constexpr (S < AN * AW) store_a(par, K, S / AW, std::integral_constant<int, S % AW>{});
            else if constexpr (L < 0) load_b(r0 + 3 * KB, bsel, S - AN * AW);
            else load_a(r0 + 4 * KB, K, L);
            __builtin_amdgcn_sched_barrier(0);
        });
        lgkm_wait(then);
        bsel = bnext;
    };
    for (int64_t r0 = 0; r0 < nrows; r0 += 2 * KB) {
        step(r0, Zero{});
        step(r0 + KB, One{});
    }
    wait_vmcnt<0>();  // nothing is on its way into LDS any more
    }
    auto store_sums = [&](int mt, float v) {
        if (lane < 32) d.colsum[(size_t)zi * d.lda + 4 * (m0 + (MSPLIT ? kh * MTW * 32 : 0) + mt * 32 + lane) + grp] = v;
    };
    if constexpr (SUMS) {
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
            cs[0][mt] += cs[1][mt];
            cs[0][mt] += __shfl_xor(cs[0][mt], 32);  // the other eight rows of the K-steps
            if constexpr (MSPLIT) store_sums(mt, cs[0][mt]);
        }
    }

    // Partial tiles P[z][g][m][n].  A lane holds, of each 32 x 32 tile, the m = lane % 32 and four n of every eight:
    // the wave turns the tile through its own piece of LDS (4 KB) into rows of whole 16-byte stores.  (A 2-byte store
    // per element instead: 0.8 us more at 768 -> 768, 12608 rows.)
    const bool live = g0 + grp < d.G;  // (the group count need not be a multiple of four)
    const int ln = lane & 31, h = lane >> 5;
    const size_t pbase = (((size_t)zi * d.G + g0 + grp) * d.M) * d.N;
    auto store_tile = [&](int mt, int nt, const f32x16& a, unsigned char* turn) {
        const size_t at = pbase + (size_t)(m0 + (MSPLIT ? kh * MTW * 32 : 0) + mt * 32) * d.N + n0 + nt * 32;
        if (d.p_bf16) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<u32x2*>(turn + ln * 80 + q * 16 + h * 8) =
                    u32x2{pack_bf16x2(a[4 * q], a[4 * q + 1]), pack_bf16x2(a[4 * q + 2], a[4 * q + 3])};
            __builtin_amdgcn_wave_barrier();
            uint16_t* to = reinterpret_cast<uint16_t*>(d.P) + at + (size_t)(lane >> 2) * d.N + (lane & 3) * 8;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(turn + ((lane >> 2) + 16 * u) * 80 + (lane & 3) * 16);
                if (live) *reinterpret_cast<u32x4*>(to + (size_t)16 * u * d.N) = v;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4*>(turn + ln * 128 + ((2 * q + h) ^ (ln & 7)) * 16) =
                    f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
            __builtin_amdgcn_wave_barrier();
            float* to = d.P + at + (size_t)(lane >> 3) * d.N + (lane & 7) * 4;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(turn + ((lane >> 3) + 8 * u) * 128 + ((lane & 7) ^ (lane >> 3)) * 16);
                if (live) *reinterpret_cast<f32x4*>(to + (size_t)8 * u * d.N) = v;
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    __syncthreads();  // the buffers are no longer read
    if constexpr (MSPLIT) {
#pragma unroll
        for (int t = 0; t < MTW * NT; ++t)
            store_tile(t / NT, t % NT, acc[t], reinterpret_cast<unsigned char*>(lds) + (wave * 2 + t % 2) * 4096);
    } else {
        // the two waves of a group hand each other half of their tiles (fp32), add and store the other half
        constexpr int NTILE = MT * NT, R1 = (NTILE + 1) / 2;
        float* red = reinterpret_cast<float*>(lds) + (size_t)grp * NTILE * 1024;
        float* redc = reinterpret_cast<float*>(lds) + (size_t)4 * NTILE * 1024 + grp * MT * 32 + ln;
        auto hand = [&](int t) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4*>(red + t * 1024 + q * 256 + lane * 4) =
                    f32x4{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
        };
        auto finish = [&](int t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(red + t * 1024 + q * 256 + lane * 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[t][4 * q + i] += v[i];
            }
            __builtin_amdgcn_wave_barrier();
            store_tile(t / NT, t % NT, acc[t], reinterpret_cast<unsigned char*>(red + t * 1024));
        };
        if (kh == 1) {
            if constexpr (SUMS)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) redc[mt * 32] = cs[0][mt];
#pragma unroll
            for (int t = 0; t < R1; ++t) hand(t);
        } else {
#pragma unroll
            for (int t = R1; t < NTILE; ++t) hand(t);
        }
        __syncthreads();
        if (kh == 0) {
            if constexpr (SUMS)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) store_sums(mt, cs[0][mt] + redc[mt * 32]);
#pragma unroll
            for (int t = 0; t < R1; ++t) finish(t);
        } else {
#pragma unroll
            for (int t = R1; t < NTILE; ++t) finish(t);
        }
    }
}

// more accumulators than one wave of a pair can hold
constexpr bool msplit(int tm, int tn) { return (tm / 32) * (tn / 32) > 9; }

// One launch for up to two GEMMs over the same batch chunks.  Workgroups are handed to the
// eight XCDs round-robin by linear id; the id is remapped so that each XCD owns a contiguous
// range of (chunk, tile) pairs with the tile index fastest: the tiles that re-read the same
// operand rows then run on one XCD at about the same time and share its L2.
template <int TM, int TN>
__global__ void __launch_bounds__(NTHR)
wgrad_gemm_kernel(WgradDesc d0, WgradDesc d1, int tiles0, int tiles)
{
    const int nwg = gridDim.x, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int per = nwg >> 3, rem = nwg & 7;
    const int v = xcd * per + (xcd < rem ? xcd : rem) + slot;
    const int t = v % tiles, zi = v / tiles;
    constexpr bool MSPLIT = msplit(TM, TN);
    if (t < tiles0) {
        if (d0.colsum && t % (d0.N / TN) == 0) wgrad_gemm_body<TM, TN, true, true, MSPLIT>(d0, t, zi);
        else if (d0.deint) wgrad_gemm_body<TM, TN, true, false, MSPLIT>(d0, t, zi);
        else wgrad_gemm_body<TM, TN, false, false, MSPLIT>(d0, t, zi);
    } else {
        if (d1.deint) wgrad_gemm_body<TM, TN, true, false, MSPLIT>(d1, t - tiles0, zi);
        else wgrad_gemm_body<TM, TN, false, false, MSPLIT>(d1, t - tiles0, zi);
    }
}

// add(z, count) over 0 .. nz-1, eight at a time, then four, then one
template <typename F>
__device__ __forceinline__ void for_chunks(int nz, F add)
{
    int z = 0;
    for (; z + 8 <= nz; z += 8) add(z, std::integral_constant<int, 8>{});
    if (z + 4 <= nz) {
        add(z, std::integral_constant<int, 4>{});
        z += 4;
    }
    for (; z < nz; ++z) add(z, std::integral_constant<int, 1>{});
}

// out[g][m][col(n)] = sum_z P[z][g][m][n];  col(n) = (n % seg_w) * (N / seg_w) + n / seg_w
// (identity when seg_w == N).  Blocks [0, blocks0) reduce d0, the rest d1; eight consecutive elements per
// thread (16-byte loads of bf16 partial tiles, two 16-byte loads of fp32 ones), eight chunks in flight.
// Blocks from `blocks01` on (when cj.part is set) run the second pass of the bias gradient instead.
template <bool OUT_F32>
__global__ void __launch_bounds__(256)
wgrad_reduce_kernel(WgradDesc d0, WgradDesc d1, int blocks0, int nz, ColsumJob cj, int blocks01)
{
    if ((int)blockIdx.x >= blocks01) {
        if (OUT_F32) colsum_final_body<float, 256>(cj, (int)blockIdx.x - blocks01);
        else colsum_final_body<bf16_t, 256>(cj, (int)blockIdx.x - blocks01);
        return;
    }
    const bool first = (int)blockIdx.x < blocks0;
    const WgradDesc& d = first ? d0 : d1;
    const size_t total = (size_t)d.G * d.M * d.N;  // a multiple of 8: N is a multiple of 32
    const size_t e = ((size_t)(blockIdx.x - (first ? 0 : blocks0)) * 256 + threadIdx.x) * 8;
    if (e >= total) return;
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (d.p_bf16) {
        const uint16_t* P = reinterpret_cast<const uint16_t*>(d.P) + e;
        auto add = [&](int z, auto count) {
            u32x4 v[decltype(count)::value];
#pragma unroll
            for (int u = 0; u < decltype(count)::value; ++u) v[u] = ldg128(P + (size_t)(z + u) * total);
#pragma unroll
            for (int u = 0; u < decltype(count)::value; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    s[2 * w] += __uint_as_float(v[u][w] << 16);
                    s[2 * w + 1] += __uint_as_float(v[u][w] & 0xffff0000u);
                }
        };
        for_chunks(nz, add);
    } else {
        const float* P = d.P + e;
        auto add = [&](int z, auto count) {
            f32x4 v[decltype(count)::value][2];
#pragma unroll
            for (int u = 0; u < decltype(count)::value; ++u) {
                v[u][0] = *reinterpret_cast<const f32x4*>(P + (size_t)(z + u) * total);
                v[u][1] = *reinterpret_cast<const f32x4*>(P + (size_t)(z + u) * total + 4);
            }
#pragma unroll
            for (int u = 0; u < decltype(count)::value; ++u)
#pragma unroll
                for (int w = 0; w < 8; ++w) s[w] += v[u][w >> 2][w & 3];
        };
        for_chunks(nz, add);
    }
    // the eight elements share a row and (seg_w being a multiple of 8) a segment: their outputs are nseg apart
    const int nseg = d.N / d.seg_w;
    const size_t rowbase = e / d.N * d.N;
    const int n = (int)(e - rowbase);
    const size_t o = rowbase + (size_t)(n % d.seg_w) * nseg + n / d.seg_w;
    if (OUT_F32) {
        float* out = (float*)d.out + o;
        if (nseg == 1) {
            *reinterpret_cast<f32x4*>(out) = f32x4{s[0], s[1], s[2], s[3]};
            *reinterpret_cast<f32x4*>(out + 4) = f32x4{s[4], s[5], s[6], s[7]};
        } else {
#pragma unroll
            for (int w = 0; w < 8; ++w) out[(size_t)w * nseg] = s[w];
        }
    } else {
        uint16_t* out = (uint16_t*)d.out + o;
        if (nseg == 1) {
            *reinterpret_cast<u32x4*>(out) =
                u32x4{pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3]), pack_bf16x2(s[4], s[5]), pack_bf16x2(s[6], s[7])};
        } else {
#pragma unroll
            for (int w = 0; w < 8; ++w) out[(size_t)w * nseg] = (uint16_t)(pack_bf16x2(s[w], 0.f) & 0xffffu);
        }
    }
}

int tiles_of(const WgradDesc& d, int tm, int tn) { return (d.M / tm) * (d.N / tn) * ((d.G + 3) / 4); }

template <int TM, int TN>
int launch_gemm(const WgradDesc& d0, const WgradDesc* d1, int nz, hipStream_t st)
{
    // two buffers of A, three of B; in their place at the end the tiles that two waves add up, and the column sums
    constexpr size_t pipeline = (size_t)4 * KB * (2 * TM + 3 * TN) * 2;
    constexpr size_t sums = msplit(TM, TN) ? 0 : (size_t)4 * ((TM / 32) * (TN / 32) * 4096 + TM * 4);
    constexpr size_t lds = pipeline > sums ? pipeline : sums;
    static_assert(lds <= kMaxLdsBytes, "LDS");
    auto kern = wgrad_gemm_kernel<TM, TN>;
    if (allow_dynamic_lds((const void*)kern, lds) != hipSuccess)
        return -4;
    const int t0 = tiles_of(d0, TM, TN), t1 = d1 ? tiles_of(*d1, TM, TN) : 0;
    hipLaunchKernelGGL(kern, dim3((t0 + t1) * nz), dim3(NTHR), lds, st, d0, d1 ? *d1 : d0, t0, t0 + t1);
    return hip_status(hipGetLastError());
}

int launch_gemm_tile(int tm, int tn, const WgradDesc& d0, const WgradDesc* d1, int nz, hipStream_t st)
{
#define MONARCH_WG_CASE(TM_, TN_) \
    if (tm == TM_ && tn == TN_) return launch_gemm<TM_, TN_>(d0, d1, nz, st);
    MONARCH_WG_CASE(128, 128)
    MONARCH_WG_CASE(96, 96)
    MONARCH_WG_CASE(64, 128)
    MONARCH_WG_CASE(128, 64)
    MONARCH_WG_CASE(64, 64)
    MONARCH_WG_CASE(32, 32)
#undef MONARCH_WG_CASE
    return -2;
}

}  // namespace

bool wgrad_tile_ok(int M, int N, int seg_w, int* tm, int* tn)
{
    // tile shapes instantiated above; a tile's 8-column pieces must not straddle a segment
    if (seg_w % 8 != 0) return false;
    const int cand[][2] = {{128, 128}, {96, 96}, {64, 128}, {128, 64}, {64, 64}, {32, 32}};
    for (auto& c : cand)
        if (M % c[0] == 0 && N % c[1] == 0) {
            *tm = c[0];
            *tn = c[1];
            return true;
        }
    return false;
}

int wgrad_tiles(const WgradDesc& d)
{
    int tm, tn;
    if (!wgrad_tile_ok(d.M, d.N, d.seg_w, &tm, &tn) || (d.deint && d.G != 4)) return 0;
    return tiles_of(d, tm, tn);
}

int wgrad_gemm_pair(const WgradDesc& d0, const WgradDesc& d1, int nz, hipStream_t st)
{
    int tm0, tn0, tm1, tn1;
    if (!wgrad_tile_ok(d0.M, d0.N, d0.seg_w, &tm0, &tn0) || (d0.deint && d0.G != 4)) return -2;
    if (!wgrad_tile_ok(d1.M, d1.N, d1.seg_w, &tm1, &tn1) || (d1.deint && d1.G != 4)) return -2;
    if (tm0 == tm1 && tn0 == tn1) return launch_gemm_tile(tm0, tn0, d0, &d1, nz, st);
    const int rc = launch_gemm_tile(tm0, tn0, d0, nullptr, nz, st);
    return rc ? rc : launch_gemm_tile(tm1, tn1, d1, nullptr, nz, st);
}

ColsumJob wgrad_colsum_job(const Problem& pb, int nz)
{
    ColsumJob cj = make_colsum_job(pb, nullptr, pb.dbias, pb.colsum_ws);
    cj.chunks = nz;  // no more than it was: chunks of at least 64 rows against 16, and of 256 / tiles against 1024 / (s / 64)
    return cj;
}

int wgrad_reduce_pair(const WgradDesc& d0, const WgradDesc& d1, bool out_f32, int nz, hipStream_t st, const ColsumJob* cj)
{
    if (d0.seg_w % 8 != 0 || d1.seg_w % 8 != 0 || d0.N % 8 != 0 || d1.N % 8 != 0) return -2;  // eight elements per thread
    const size_t b0 = ((size_t)d0.G * d0.M * d0.N / 8 + 255) / 256, b1 = ((size_t)d1.G * d1.M * d1.N / 8 + 255) / 256;
    ColsumJob job{};
    if (cj) job = *cj;
    const size_t b2 = cj ? (size_t)colsum_final_blocks(job) : 0;
    if (b0 + b1 + b2 > 0x7fffffffULL) return -2;
    const dim3 grid((unsigned)(b0 + b1 + b2));
    if (out_f32)
        hipLaunchKernelGGL(wgrad_reduce_kernel<true>, grid, dim3(256), 0, st, d0, d1, (int)b0, nz, job, (int)(b0 + b1));
    else
        hipLaunchKernelGGL(wgrad_reduce_kernel<false>, grid, dim3(256), 0, st, d0, d1, (int)b0, nz, job, (int)(b0 + b1));
    return hip_status(hipGetLastError());
}

}  // namespace monarch
