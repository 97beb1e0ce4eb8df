// Batch-major bf16 rows in LDS and the transposing reads of them (ds_read_b64_tr_b16), for pipelines whose next rows are on their
// way into LDS (buffer_load ... lds) while these are read.
#pragma once
#include <type_traits>
#include <utility>
#include "monarch_mfma_common.h"

namespace monarch {

// A row of TW features of one group is TW / 32 runs of 64 bytes in LDS, unpadded.  Half a wave of a transposing read
// touches one run of four consecutive rows, which must fall on disjoint quarters of the 64 banks: the runs of a row
// change places by the row (strides of one or three runs do it by themselves).
template <int TW>
__device__ __forceinline__ constexpr int run_key(int row)
{
    return TW == 128 ? row & 3 : TW == 64 ? (row >> 1) & 1 : 0;
}
// The LDS accesses of the pipeline are written out, and the wave waits for them by itself (lgkm_wait): the compiler
// puts a wait for everything that is on its way into LDS (buffer_load ... lds) before a transposing read it knows of.
// It takes the registers of such a read as written at once, so what it makes must not touch them, nor pass a branch,
// before the wait: every read is handed to lgkm_wait within its basic block, none is left unused, and a test
// (test_lds_reads_in_flight.py) reads the assembly of the sources that include this file.
// Transposing read: within each 16 lanes, lane i receives element (i % 4) of lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4.
template <int OFF>
__device__ __forceinline__ u32x2 lds_tr16(uint32_t at)
{
    static_assert(OFF >= 0 && OFF < 65536, "offset field");
    u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(at), "n"(OFF));
    return v;
}
template <int OFF>
__device__ __forceinline__ u32x4 lds_get128(uint32_t at)
{
    static_assert(OFF >= 0 && OFF < 65536, "offset field");
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(at), "n"(OFF));
    return v;
}
template <int OFF>
__device__ __forceinline__ void lds_put32(uint32_t at, uint32_t v)
{
    static_assert(OFF >= 0 && OFF < 65536, "offset field");
    asm volatile("ds_write_b32 %0, %1 offset:%2" : : "v"(at), "v"(v), "n"(OFF));
}
template <int OFF>
__device__ __forceinline__ void lds_put64(uint32_t at, const u32x2& v)
{
    static_assert(OFF >= 0 && OFF < 65536, "offset field");
    asm volatile("ds_write_b64 %0, %1 offset:%2" : : "v"(at), "v"(v), "n"(OFF));
}
template <int OFF>
__device__ __forceinline__ void lds_put128(uint32_t at, const u32x4& v)
{
    static_assert(OFF >= 0 && OFF < 65536, "offset field");
    asm volatile("ds_write_b128 %0, %1 offset:%2" : : "v"(at), "v"(v), "n"(OFF));
}
// An MFMA operand (32 features x 16 batch rows) on its way from LDS: lane (f = lane % 32, h = lane / 32) gets rows 8h .. 8h+7 of
// feature f, four of them in each half.
struct Frag {
    u32x2 lo, hi;
    __device__ __forceinline__ bf16x8 operand() const { return as_bf16x8(u32x4{lo[0], lo[1], hi[0], hi[1]}); }
};
template <int N>
__device__ __forceinline__ void lgkm_wait(Frag (&f)[N])
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(f[i].lo), "+v"(f[i].hi));
}
template <int N>
__device__ __forceinline__ void lgkm_wait(u32x4 (&v)[N])
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}
template <int... I, typename F>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
// f(0) .. f(N - 1), the numbers as constants
template <int N, typename F>
__device__ __forceinline__ void each(F f) { each_of(std::make_integer_sequence<int, N>{}, f); }

}  // namespace monarch
