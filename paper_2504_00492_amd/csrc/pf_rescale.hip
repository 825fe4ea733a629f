// beta -> beta_eff = (1 - exp(-beta |k|^2)) / |k|^2 for every (k, beta) pair: the step size with
// which a rank-1 delta step is the exact flow of its increment instead of its Euler step
// (Section 3.3 of ParallelFlow, arXiv 2504.00492: exp(a b^T) = Id + ((e^x - 1) / x) a b^T with
// x = <b, a>, here a = beta k, b = -k; the input increment picks up the same factor).
// One row of K per 16 lanes: 16-byte loads where the row length allows, partial sums combined
// with cross-lane shuffles (__shfl_xor) inside the 16-lane row, fp32 arithmetic.
#include "pf_internal.h"
#include "pf_common.h"

#include <type_traits>

namespace pf {

namespace {

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<uint16_t>(uint16_t v) { return bf16_bits_to_f32(v); }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ uint16_t from_f32<uint16_t>(float v)
{
    bf16 b = (bf16)v;
    return __builtin_bit_cast(uint16_t, b);
}

template <typename T>
__global__ __launch_bounds__(256) void beta_exponential_kernel(const T *__restrict__ K, const T *beta, T *beta_out,
                                                              long long rows, int dk)
{
    constexpr int VEC = 16 / sizeof(T);
    const int l16 = threadIdx.x & 15;
    const long long row0 = (long long)blockIdx.x * 16 + (threadIdx.x >> 4);
    for (long long row = row0; row < rows; row += (long long)gridDim.x * 16) {
        const T *k = K + row * dk;
        float s = 0.f;
        if (dk % VEC == 0) {
            for (int e = l16 * VEC; e < dk; e += 16 * VEC) {
                T v[VEC];
                *reinterpret_cast<u32x4 *>(v) = *reinterpret_cast<const u32x4 *>(k + e);
#pragma unroll
                for (int i = 0; i < VEC; ++i) s = fmaf(to_f32(v[i]), to_f32(v[i]), s);
            }
        } else {
            for (int e = l16; e < dk; e += 16) s = fmaf(to_f32(k[e]), to_f32(k[e]), s);
        }
#pragma unroll
        for (int m = 8; m >= 1; m >>= 1) s += __shfl_xor(s, m, 16);
        if (l16 == 0) {
            const float b = to_f32(beta[row]);
            const float be = s > 0.f ? -expm1f(-b * s) / s : b;
            beta_out[row] = from_f32<T>(be);
        }
    }
}

// Rows of G = 8 or 16 units of 16 bytes: a lane has its unit of N = 8 rows on their way at once, a wavefront 64 or 32 rows.
// The sums over the G lanes of a row meet as in the kernel above (same pairs, same order), but from 8 lanes on each step
// halves the sums a lane still holds, so that a lane ends with the sum of one row and takes one beta: one expm1f for all
// rows of the wavefront instead of one for every four.
// What bounds it: HBM, 5.9 TB/s (32 heads x 65536 tokens, r = 2, d_k = 128, bf16).  us, one row per 16 lanes / this:
//   bf16, d_k = 64     24 heads x 4096, r = 2    9.1 / 4.0
//   bf16, d_k = 128    32 x 4096, r = 2         16.3 / 11.9     32 x 65536, r = 2     229 / 182
// (64 rows of 16 units a wavefront, 16 loads and sums in registers: 19.5 and 212 at d_k = 128, and 6.6 against 3.9 for 128 rows)
template <typename T, int G>
__global__ __launch_bounds__(256) void beta_exponential_kernel(const T *__restrict__ K, const T *beta, T *beta_out,
                                                              long long rows, std::integral_constant<int, G>)
{
    constexpr int VEC = 16 / sizeof(T), N = 8, per = 64 / G;   // per: rows of a load
    const int lane = threadIdx.x & 63, p = lane % G;
    const long long first = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * (N * per);
    if (first >= rows) return;
    // load i brings rows first + per i .. + per - 1 (beyond the last: the last once more)
    u32x4 v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const long long row = first + per * i + lane / G;
        v[i] = *reinterpret_cast<const u32x4 *>(K + (row < rows ? row : rows - 1) * (G * VEC) + p * VEC);
    }
    // lane p of a row's lanes keeps load p % 8
    const long long row = first + per * (p % N) + lane / G;
    const bool own = row < rows && p < N;
    const float b = to_f32(beta[row < rows ? row : rows - 1]);
    float s[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        T e[VEC];
        *reinterpret_cast<u32x4 *>(e) = v[i];
        s[i] = 0.f;
#pragma unroll
        for (int q = 0; q < VEC; ++q) s[i] = fmaf(to_f32(e[q]), to_f32(e[q]), s[i]);
        if constexpr (G == 16) s[i] += __shfl_xor(s[i], 8, G);
    }
#pragma unroll
    for (int m = N / 2; m >= 1; m >>= 1) {
        const bool upper = p & m;
#pragma unroll
        for (int i = 0; i < m; ++i) {
            const float mine = upper ? s[i + m] : s[i], other = upper ? s[i] : s[i + m];
            s[i] = mine + __shfl_xor(other, m, G);
        }
    }
    if (own) beta_out[row] = from_f32<T>(s[0] > 0.f ? -expm1f(-b * s[0]) / s[0] : b);
}

}  // namespace

hipError_t launch_beta_exponential(const void *K, const void *beta, void *beta_out, long long rows, int dk,
                                   bool is_bf16, hipStream_t stream)
{
    if (rows == 0) return hipSuccess;
    auto launch = [&](auto one) {
        using T = decltype(one);
        const T *k = static_cast<const T *>(K), *b = static_cast<const T *>(beta);
        T *o = static_cast<T *>(beta_out);
        auto wide = [&](auto G) {
            constexpr int per = 4 * 8 * 64 / decltype(G)::value;   // rows of a workgroup
            void (*kern)(const T *, const T *, T *, long long, decltype(G)) = beta_exponential_kernel;
            hipLaunchKernelGGL(kern, dim3((unsigned)((rows + per - 1) / per)), dim3(256), 0, stream, k, b, o, rows, G);
        };
        const int bytes = dk * (int)sizeof(T);
        const long long want = (rows + 15) / 16;
        // Rows of 8 or 16 units, where 16 rows to a workgroup are more workgroups than the chip holds at once (8 a compute
        // unit): up to there a row per 16 lanes has all rows on their way as well, and sums less in each lane.  us, one row per
        // 16 lanes / eight loads a lane, inputs in the last-level cache and cold:
        //                        2048 rows                 32768                     36864                     65536
        //   bf16, d_k = 64    2.17 / 2.61, 2.99 / 3.81  2.89 / 2.75, 3.85 / 4.29  3.12 / 2.75, 4.86 / 4.34  4.04 / 2.82, 5.76 / 4.72
        //         d_k = 128   2.16 / 2.76, 3.01 / 4.06  2.88 / 2.96, 4.46 / 4.77  3.10 / 3.16, 5.38 / 5.29  4.15 / 3.47, 6.57 / 6.10
        //   fp32, d_k = 32    2.11 / 2.56, 2.81 / 3.68  2.78 / 2.69, 3.64 / 4.09  3.03 / 2.70, 4.67 / 4.16  3.82 / 2.82, 5.56 / 4.74
        //         d_k = 64    2.10 / 2.74, 2.88 / 4.43  2.78 / 2.99, 4.25 / 5.17  3.02 / 3.15, 5.18 / 5.47  3.95 / 3.46, 6.33 / 6.23
        // Other widths: one row per 16 lanes.
        if (want > 8LL * device_cu_count()) {
            if (bytes == 128) return wide(std::integral_constant<int, 8>{});
            if (bytes == 256) return wide(std::integral_constant<int, 16>{});
        }
        void (*kern)(const T *, const T *, T *, long long, int) = beta_exponential_kernel;
        hipLaunchKernelGGL(kern, dim3((unsigned)(want < 65536 ? want : 65536)), dim3(256), 0, stream, k, b, o, rows, dk);
    };
    if (is_bf16) launch((uint16_t)0);
    else launch(0.f);
    return hipGetLastError();
}

}  // namespace pf
