// Per-expert token counts n_e (the n_i of Eq. (1), p_hat_i = n_i / N): the
// "distribution" that Distribution-Only Prediction forecasts.  Counts are
// privatised in LDS per workgroup and merged with integer atomics, so the
// result does not depend on the launch shape.
#include "common.h"

namespace moegps {

constexpr int kHistThreads = 1024;
constexpr int kHistItemsPerBlock = 16384;  // elements one workgroup of the wide kernel covers

// Counts n indices into bins[0 .. E * copies) in LDS: bin e is kept `copies` times side by side and a
// lane takes the copy of its number, so that few experts do not mean that the lanes of a wavefront
// queue up at the same address (copies: a power of two with at most kHistBins bins in all).  The
// indices are read 16 bytes at a time, four reads under way (VEC: idx is 16-byte aligned).
// One workgroup, 16384 indices to 8 experts 8.2 -> 3.2 us, 32764 to 16 10.4 -> 4.0, 65536 to 128 11.2 ->
// 6.4; up to 2048 indices one copy is enough and adding up 32 costs more (2.2 against 2.8 us).
constexpr int kHistBins = 1024;
static_assert(kHistBins >= MOE_MAX_EXPERTS, "one copy of every bin fits");
__host__ __device__ inline int hist_copies(int E, int64_t n) {
    int c = n <= 2048 ? 1 : 32;
    while (c > 1 && c * E > kHistBins) c >>= 1;
    return c;
}
template <bool VEC>
__device__ __forceinline__ void count_into(const int32_t* __restrict__ idx, int64_t n, int E, int copies, int* bins) {
    for (int i = threadIdx.x; i < E * copies; i += blockDim.x) bins[i] = 0;
    __syncthreads();
    int* mine = bins + (threadIdx.x & (copies - 1));
    auto count = [&](int e) {
        if (e >= 0 && e < E) atomicAdd(&mine[e * copies], 1);
    };
    int64_t done = 0;
    if (VEC) {
        constexpr int U = 4;
        const int64_t n4 = n / 4;
        for (int64_t i0 = threadIdx.x; i0 < n4; i0 += (int64_t)blockDim.x * U) {
            int4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = i0 + (int64_t)u * blockDim.x;
                v[u] = i < n4 ? ((const int4*)idx)[i] : make_int4(-1, -1, -1, -1);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                count(v[u].x);
                count(v[u].y);
                count(v[u].z);
                count(v[u].w);
            }
        }
        done = n4 * 4;
    }
    for (int64_t i = done + threadIdx.x; i < n; i += blockDim.x) count(idx[i]);
    __syncthreads();
}
// count of expert e over its copies (neighbouring threads start at different ones)
__device__ __forceinline__ int sum_copies(const int* bins, int e, int copies) {
    int c = 0;
    for (int r = 0; r < copies; ++r) c += bins[e * copies + ((r + e) & (copies - 1))];
    return c;
}

// One workgroup counts everything and writes the result directly.
template <bool VEC>
__global__ __launch_bounds__(kHistThreads) void hist_single_kernel(const int32_t* __restrict__ idx, int64_t n,
                                                                    int E, int32_t* __restrict__ hist) {
    __shared__ int bins[kHistBins];
    const int copies = hist_copies(E, n);
    count_into<VEC>(idx, n, E, copies, bins);
    for (int e = threadIdx.x; e < E; e += blockDim.x) hist[e] = sum_copies(bins, e, copies);
}

__global__ void hist_zero_kernel(int32_t* __restrict__ hist, int E) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < E) hist[e] = 0;
}

template <bool VEC>
__global__ __launch_bounds__(kHistThreads) void hist_wide_kernel(const int32_t* __restrict__ idx, int64_t n,
                                                                  int E, int32_t* __restrict__ hist) {
    __shared__ int bins[kHistBins];
    const int copies = hist_copies(E, kHistItemsPerBlock);
    const int64_t lo = (int64_t)blockIdx.x * kHistItemsPerBlock;
    count_into<VEC>(idx + lo, lo + kHistItemsPerBlock < n ? kHistItemsPerBlock : n - lo, E, copies, bins);
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const int c = sum_copies(bins, e, copies);
        if (c) atomicAdd(&hist[e], c);
    }
}

}  // namespace moegps

extern "C" int moe_histogram(const int32_t* idx, int64_t n, int E, int32_t* hist, void* stream) {
    using namespace moegps;
    if (n < 0 || E < 1) return MOE_ERR_INVALID_ARG;
    if (E > MOE_MAX_EXPERTS) return MOE_ERR_UNSUPPORTED;
    if (!hist || (n > 0 && !idx)) return MOE_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    const bool vec = (uintptr_t)idx % 16 == 0;
    if (n <= 4 * kHistItemsPerBlock) {
        hipLaunchKernelGGL(vec ? hist_single_kernel<true> : hist_single_kernel<false>, dim3(1), dim3(kHistThreads), 0,
                           st, idx, n, E, hist);
        return check_launch();
    }
    hipLaunchKernelGGL(hist_zero_kernel, dim3(ceil_div(E, 256)), dim3(256), 0, st, hist, E);
    int rc = check_launch();
    if (rc != MOE_OK) return rc;
    const int64_t grid = ceil_div64(n, kHistItemsPerBlock);
    hipLaunchKernelGGL(vec ? hist_wide_kernel<true> : hist_wide_kernel<false>, dim3((unsigned)grid), dim3(kHistThreads), 0, st, idx, n, E, hist);
    return check_launch();
}
