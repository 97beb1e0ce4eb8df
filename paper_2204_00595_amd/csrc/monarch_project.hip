// Projection of a dense n x n matrix, n = m^2, onto the square Monarch matrices (Section 3.3,
// Theorem 1, Algorithm 1): with At[l][j][k][i] = A[l*m + j][k*m + i], the slice G = At[:, j, k, :] of the
// closest Monarch matrix is the best rank-1 approximation sigma_1 u_1 v_1^T of that slice of A, and
// L[j][:][k] = sqrt(sigma_1) u_1,  R[k][j][:] = sqrt(sigma_1) v_1.
//
// Only the leading triple is needed: v_1 is the leading eigenvector of S = G^T G, and u_1 = G v_1 / sigma_1.  (Forming S costs
// the leading pair no accuracy: the relative gap of sigma^2 is twice that of sigma.)  One wavefront per slice squares S
// (scaled to trace 1) until it is of rank one: after t squarings the second eigenvalue has shrunk to (sigma_2/sigma_1)^(2^(t+1)),
// so a gap of 1e-6 is resolved in about twenty squarings, and rounding in a later squaring meets a wider gap than in the first.
//
// A squaring of a symmetric matrix on the matrix cores needs next to no data movement: lane (c, h) of a 16 x 16
// accumulator tile holds S[4h + r][c] = S[c][4h + r], which is what the same lane has to bring as either operand of
// contraction step r.  Tiles below the diagonal are transposes of those above, by way of LDS.
//
// From 17 rows on the products are those of three bf16 planes of the entries (six v_mfma_f32_16x16x32_bf16 for the
// eight contraction indices of two tiles that a lane holds, 96 clocks for the 256 of v_mfma_f32_16x16x4_f32), which
// costs 5.5 vector instructions an entry and leaves less rounding: products off float64 by 2.0e-7 of them for 4.7e-7
// (root mean square over eight matrices, m = 32), 3.2e-7 for 5.6e-7 (m = 64).  Calls in a row, on the fp32 matrix cores
// and in planes, us: m = 24 10.3 to 11.3 and 8.9 to 9.3, 32 10.8 to 11.6 and 9.0 to 10.6, 40 35 and 27, 48 47 and 34,
// 64 135 and 84 (a profiler, which separates the launches, has 10.7 to 11.9 for m = 32).
// What bounds it: from 33 rows on the vector units and the matrix cores, by about the same (m = 64: 1900 clocks of
// products and 2000 of splitting, scaling and summing up for a squaring, two waves per SIMD), below the chain of
// squarings.  Sums over the lanes stay in the vector registers and run beside the products (m = 32, 1024 slices: 15.8
// us with shuffles between them, 13.3 without; the four lanes of a column meet by row swaps).  The one-sided Jacobi SVD
// that was here before (all m triples, three cross-lane shuffles per element and rotation) took 784 us for m = 32 and
// 5.8 ms for m = 64, and was less accurate (products 2e-5 off at m = 64).
#include <type_traits>
#include "monarch_internal.h"
#include "monarch_device.h"
#include "monarch_mfma_common.h"

namespace monarch {
namespace {

constexpr int kMaxSquarings = 32;     // relative gaps down to 1e-8, below fp32
constexpr float kRankOne = 1e-4f;     // 1 - |S|_F^2 at trace 1, about twice the second eigenvalue; one squaring more follows
constexpr int kWavesPerBlock = 4;     // slices of neighbouring k: their rows of A lie next to each other

// Reductions over the wave inside the vector registers: a shuffle goes through LDS, and six of them in a row took as long as the
// squaring beside them.
template <int CTRL>
__device__ __forceinline__ float lane_move(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
// over the four lanes of a column of a tile: 16 and 32 apart
template <typename Op>
__device__ __forceinline__ float column_reduce(float v, Op op)
{
    const uint32_t a = __float_as_uint(v);
    const auto p = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const uint32_t b = __float_as_uint(op(__uint_as_float(p[0]), __uint_as_float(p[1])));
    const auto q = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return op(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
template <typename Op>
__device__ __forceinline__ float wave_reduce(float v, Op op)
{
    v = op(v, lane_move<0xB1>(v));   // the neighbour, the pair next to it, the other four, the other eight of a row of 16
    v = op(v, lane_move<0x4E>(v));
    v = op(v, lane_move<0x141>(v));
    v = op(v, lane_move<0x140>(v));
    return column_reduce(v, op);
}
__device__ __forceinline__ float wave_sum(float v) { return wave_reduce(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float column_sum(float v) { return column_reduce(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); }); }

// Eight values as three bf16 planes that add up to them, the values first rounded, what that leaves rounded, and the
// rest: an operand of v_mfma_f32_16x16x32_bf16 each.  (Entries are at most one; what is below 2^-126 is lost.)
__device__ __forceinline__ void planes_of(const f32x4& lo, const f32x4& hi, bf16x8 (&out)[3])
{
    float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
            if (u < 2) {
                v[2 * i] -= __uint_as_float(w[i] << 16);
                v[2 * i + 1] -= __uint_as_float(w[i] & 0xffff0000u);
            }
        }
        out[u] = as_bf16x8(w);
    }
}
// the six largest products of planes; the others add up to 2^-24 of the product
__device__ __forceinline__ f32x4 plane_sums(const bf16x8 (&a)[3], const bf16x8 (&b)[3], f32x4 c)
{
#pragma unroll
    for (int w = 2; w >= 0; --w)
#pragma unroll
        for (int u = 0; u <= w; ++u) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[w - u], c, 0, 0, 0);
    return c;
}

// NT x NT tiles of 16 x 16
template <typename T, int NT>
__global__ void __launch_bounds__(64 * kWavesPerBlock, 2) project_kernel(const T* __restrict__ A, T* __restrict__ R, T* __restrict__ L, int m)
{
    constexpr int H = 4, TS = 16, NA = 4;             // lanes per column of a tile, its side, values per lane
    constexpr int GT = TS * NT / H;                   // steps of H rows of G
    constexpr int GP = NT == 3 ? 16 : GT;             // ... rounded up to a power of two
    constexpr int kStride = TS + 4, kUpper = NT * (NT - 1) / 2;
    constexpr bool kPlanes = NT > 1;                  // the squarings on the bf16 matrix cores
    __shared__ __align__(16) float shared[kWavesPerBlock][kUpper > 0 ? kUpper * TS * kStride : H * GP];
    const int slice = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (slice >= m * m) return;  // no barriers below
    float* const lds = shared[threadIdx.x >> 6];
    const int j = slice / m, k = slice - j * m;
    const int lane = threadIdx.x & 63, c = lane & 15, h = lane >> 4;
    const size_t n = (size_t)m * m;

    // g[a][t] = G[H*t + h][TS*a + c]
    float g[NT][GT];
    float big = 0.f;
#pragma unroll
    for (int t = 0; t < GT; ++t)
#pragma unroll
        for (int a = 0; a < NT; ++a) {
            const int l = H * t + h, i = TS * a + c;
            g[a][t] = (l < m && i < m) ? Elem<T>::load(A + ((size_t)l * m + j) * n + (size_t)k * m + i) : 0.f;
        }
#pragma unroll
    for (int t = 0; t < GT; ++t)
#pragma unroll
        for (int a = 0; a < NT; ++a) big = fmaxf(big, fabsf(g[a][t]));
    big = wave_max(big);
    // a power of two brings the largest entry near one: the squares neither overflow nor vanish
    int ex = 0;
    if (big > 0.f) (void)frexpf(big, &ex);
    float trace = 0.f;  // of S
#pragma unroll
    for (int t = 0; t < GT; ++t)
#pragma unroll
        for (int a = 0; a < NT; ++a) {
            g[a][t] = ldexpf(g[a][t], -ex);
            trace = fmaf(g[a][t], g[a][t], trace);
        }
    trace = wave_sum(trace);

    f32x4 S[NT][NT];  // S[a][b]: rows of tile a, columns of tile b
    // the tiles below the diagonal from those above, by way of LDS
    auto mirror = [&]() {
        int at = 0;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int b = a + 1; b < NT; ++b, at += TS * kStride)
#pragma unroll
                for (int r = 0; r < NA; ++r) lds[at + (4 * h + r) * kStride + c] = S[a][b][r];
        __builtin_amdgcn_wave_barrier();
        at = 0;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int b = a + 1; b < NT; ++b, at += TS * kStride)
                S[b][a] = *reinterpret_cast<const f32x4*>(lds + at + c * kStride + 4 * h);
        __builtin_amdgcn_wave_barrier();
    };
    // S = X^T X above the diagonal: tile column a of X is `steps` pieces of four contraction indices, x(a, step), which lane
    // (c, h) brings in the same places for both operands, so that their order does not matter
    auto gram = [&](auto steps, auto x) {
        constexpr int N = decltype(steps)::value;
        if constexpr (kPlanes) {
            bf16x8 p[(N + 1) / 2][NT][3];
#pragma unroll
            for (int t = 0; t < (N + 1) / 2; ++t)
#pragma unroll
                for (int a = 0; a < NT; ++a) planes_of(x(a, 2 * t), 2 * t + 1 < N ? x(a, 2 * t + 1) : f32x4{0.f, 0.f, 0.f, 0.f}, p[t][a]);
#pragma unroll
            for (int a = 0; a < NT; ++a)
#pragma unroll
                for (int b = a; b < NT; ++b) S[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < (N + 1) / 2; ++t)
#pragma unroll
                for (int a = 0; a < NT; ++a)
#pragma unroll
                    for (int b = a; b < NT; ++b) S[a][b] = plane_sums(p[t][a], p[t][b], S[a][b]);
        } else {
            f32x4 q[NT][NT];
#pragma unroll
            for (int a = 0; a < NT; ++a)
#pragma unroll
                for (int b = a; b < NT; ++b) q[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
                for (int r = 0; r < NA; ++r)
#pragma unroll
                    for (int a = 0; a < NT; ++a)
#pragma unroll
                        for (int b = a; b < NT; ++b) q[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x(a, t)[r], x(b, t)[r], q[a][b], 0, 0, 0);
#pragma unroll
            for (int a = 0; a < NT; ++a)
#pragma unroll
                for (int b = a; b < NT; ++b) S[a][b] = q[a][b];
        }
    };
    gram(std::integral_constant<int, NT>(), [&](int a, int t) { return f32x4{g[a][4 * t], g[a][4 * t + 1], g[a][4 * t + 2], g[a][4 * t + 3]}; });
    mirror();

    // S = S^2 at trace 1; returns the trace before, |S|_F^2, which is 1 exactly when S, at trace 1 itself, is of rank
    // one.  The sum over the lanes runs beside the products.
    auto square = [&]() {
        float norm2 = 0.f;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int b = 0; b < NT; ++b)
#pragma unroll
                for (int r = 0; r < NA; ++r) norm2 = fmaf(S[a][b][r], S[a][b][r], norm2);
        gram(std::integral_constant<int, NT>(), [&](int a, int t) { return S[t][a]; });
        norm2 = wave_sum(norm2);
        const float inv = norm2 > 0.f ? 1.f / norm2 : 0.f;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int b = a; b < NT; ++b)
#pragma unroll
                for (int r = 0; r < NA; ++r) S[a][b][r] *= inv;
        mirror();
        return norm2;
    };
    {
        const float inv = trace > 0.f ? 1.f / trace : 0.f;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int b = 0; b < NT; ++b)
#pragma unroll
                for (int r = 0; r < NA; ++r) S[a][b][r] *= inv;
    }
    for (int it = 0; it < kMaxSquarings; ++it)
        if (!(1.f - square() > kRankOne)) break;  // NaN ends it too

    // v_1 is every column of S up to scale: the row with the largest diagonal entry
    float best = -1.f;
    int who = 0;
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int r = 0; r < NA; ++r) {
            const int row = 4 * h + r;
            if (row == c && S[a][a][r] > best) {
                best = S[a][a][r];
                who = TS * a + c;
            }
        }
    {
        const float top = wave_max(best);
        who = -(int)wave_max(best == top ? -(float)who : -1e9f);  // the first of equal ones
    }
    float v[NT];
#pragma unroll
    for (int a = 0; a < NT; ++a) {
        v[a] = 0.f;
#pragma unroll
        for (int e = 0; e < NT; ++e)
#pragma unroll
            for (int r = 0; r < NA; ++r)
                if (TS * e + 4 * h + r == who) v[a] = S[e][a][r];
        v[a] = column_sum(v[a]);  // one of the H lanes of a column has it, the others zero
    }

    // Twice u = G v, with one step v = G^T u in between: what rounding left of the other vectors shrinks with their singular
    // values, and v is the image of u.
    float u = 0.f, sigma2 = 0.f;
    int l = 0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        float nv = 0.f;
#pragma unroll
        for (int a = 0; a < NT; ++a) nv = fmaf(v[a], v[a], nv);
        nv = wave_sum(nv) / H;
        const float unit = nv > 0.f ? 1.f / sqrtf(nv) : 0.f;
        float w[GP];
#pragma unroll
        for (int a = 0; a < NT; ++a) v[a] *= unit;
#pragma unroll
        for (int t = 0; t < GP; ++t) {
            w[t] = 0.f;
            if (t < GT)
#pragma unroll
                for (int a = 0; a < NT; ++a) w[t] = fmaf(g[a][t], v[a], w[t]);
        }
        // sum over the TS lanes of a row, each lane keeping half of its values at every step while it has more than
        // one; the partners are the lanes 15 - c, 7 - c of eight, c ^ 2 and c ^ 1, which differ in the bit d
        int t0 = 0;
        auto halve = [&](auto ctrl, auto count, int d) {
            constexpr int CTRL = decltype(ctrl)::value, left = decltype(count)::value / 2;
            if constexpr (left > 0) {
                const bool upper = (lane & d) != 0;
                t0 = 2 * t0 + (upper ? 1 : 0);
#pragma unroll
                for (int t = 0; t < left; ++t) {
                    const float give = upper ? w[t] : w[t + left];
                    const float keep = upper ? w[t + left] : w[t];
                    w[t] = keep + lane_move<CTRL>(give);
                }
            } else {
                w[0] += lane_move<CTRL>(w[0]);
            }
        };
        halve(std::integral_constant<int, 0x140>(), std::integral_constant<int, GP>(), 8);
        halve(std::integral_constant<int, 0x141>(), std::integral_constant<int, GP / 2>(), 4);
        halve(std::integral_constant<int, 0x4E>(), std::integral_constant<int, GP / 4>(), 2);
        halve(std::integral_constant<int, 0xB1>(), std::integral_constant<int, GP / 8>(), 1);
        u = w[0];
        l = H * t0 + h;
        constexpr int kHeld = TS / GP;  // lanes that hold the same element
        sigma2 = wave_sum(u * u) / kHeld;
        if (pass == 0) {
            __builtin_amdgcn_wave_barrier();
            lds[l] = u;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int a = 0; a < NT; ++a) v[a] = 0.f;
#pragma unroll
            for (int t = 0; t < GT; ++t) {
                const float ut = lds[H * t + h];
#pragma unroll
                for (int a = 0; a < NT; ++a) v[a] = fmaf(g[a][t], ut, v[a]);
            }
#pragma unroll
            for (int a = 0; a < NT; ++a) v[a] = column_sum(v[a]);
        }
    }
    const float sigma = sqrtf(sigma2);
    // sqrt(sigma_1) of the unscaled slice
    const float root = sqrtf((ex & 1) ? 2.f * sigma : sigma), scale = ldexpf(1.f, (ex - (ex & 1)) / 2);
    if (l < m) Elem<T>::store(L + ((size_t)j * m + l) * m + k, sigma > 0.f ? u / sigma * root * scale : 0.f);
#pragma unroll
    for (int a = 0; a < NT; ++a)
        if (h == 0 && TS * a + c < m) Elem<T>::store(R + ((size_t)k * m + j) * m + TS * a + c, v[a] * root * scale);
}

template <typename T>
void launch_t(const void* A, void* R, void* L, int m, hipStream_t st)
{
    const dim3 grid((unsigned)((m * m + kWavesPerBlock - 1) / kWavesPerBlock)), block(64 * kWavesPerBlock);
    if (m <= 16) hipLaunchKernelGGL((project_kernel<T, 1>), grid, block, 0, st, (const T*)A, (T*)R, (T*)L, m);
    else if (m <= 32) hipLaunchKernelGGL((project_kernel<T, 2>), grid, block, 0, st, (const T*)A, (T*)R, (T*)L, m);
    else if (m <= 48) hipLaunchKernelGGL((project_kernel<T, 3>), grid, block, 0, st, (const T*)A, (T*)R, (T*)L, m);
    else hipLaunchKernelGGL((project_kernel<T, 4>), grid, block, 0, st, (const T*)A, (T*)R, (T*)L, m);
}

}  // namespace

bool project_supported(int m) { return m >= 1 && m <= 64; }

int launch_project(const void* A, void* R, void* L, int m, int dtype, hipStream_t st)
{
    if (!project_supported(m)) return -2;
    if (dtype == 0) launch_t<float>(A, R, L, m, st);
    else launch_t<bf16_t>(A, R, L, m, st);
    return hip_status(hipGetLastError());
}

}  // namespace monarch
