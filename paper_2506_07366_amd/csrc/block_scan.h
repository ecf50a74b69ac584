// Prefix sums: of up to 2048 ints held in LDS, by a 1024-thread workgroup; over a wavefront.
#pragma once
#include "common.h"

namespace moegps {

// data[0..n) -> exclusive prefix sums in place, data[n] = total.  n <= 2048,
// blockDim.x == 1024, data has room for n+1 ints, wave_sum for 16 ints.
// Every thread of the workgroup must call it.
__device__ inline void block_exclusive_scan_2048(int* data, int n, int* wave_sum) {
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int i0 = 2 * tid, i1 = 2 * tid + 1;
    const int a0 = i0 < n ? data[i0] : 0;
    const int a1 = i1 < n ? data[i1] : 0;
    int incl = a0 + a1;
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        const int o = __shfl_up(incl, m, kWave);
        if (lane >= m) incl += o;
    }
    if (lane == kWave - 1) wave_sum[tid / kWave] = incl;
    __syncthreads();
    int ws[16];  // all reads first: they overlap
#pragma unroll
    for (int ww = 0; ww < 16; ++ww) ws[ww] = wave_sum[ww];
    int wbase = 0, total = 0;
#pragma unroll
    for (int ww = 0; ww < 16; ++ww) {
        wbase += ww < tid / kWave ? ws[ww] : 0;
        total += ws[ww];
    }
    const int excl = wbase + incl - (a0 + a1);
    if (i0 < n) data[i0] = excl;
    if (i1 < n) data[i1] = excl + a0;
    if (tid == 0) data[n] = total;
    __syncthreads();
}

// sum of v over the 64 lanes of a wavefront (every lane active), in every lane
__device__ __forceinline__ int wave_sum_i32(int v) {
#pragma unroll
    for (int m = kWave / 2; m > 0; m >>= 1) v += __shfl_xor(v, m, kWave);
    return v;
}

// inclusive prefix sums over the 64 lanes of a wavefront (every lane active), by DPP: inside rows of 16
// lanes by shifts, then the last lane of a row added to the rows above
__device__ __forceinline__ int wave_prefix_i32(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Between LDS writes and reads of one wavefront's lanes of each other's words: a wavefront's LDS
// accesses are served in order, so this only keeps the compiler from moving them.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace moegps
