// The row copy of the permutation, x_perm[row_of_assign[t*k + j], :] = x[t, :]: as a launch of its own
// (permute.hip), or as further workgroups of the launch of the first product (grouped_ffn.hip), which
// then reads its rows from x.
#pragma once
#include "common.h"

namespace moegps {

struct RowCopy {
    const uint4* x;
    uint4* x_perm;                 // null: nothing to copy
    const int32_t* row_of_assign;
    int T, k;
    int chunks;                    // 16-byte pieces of a row
    int slices;                    // wavefronts that share a token's row
    int per_wave;                  // (token, slice) pairs of a wavefront
};

// 16-byte pieces under way per lane: four where a row has that many for every lane, else one
inline int row_copy_unroll(int chunks) { return chunks >= 4 * kWave ? 4 : 1; }

inline RowCopy row_copy(const void* x, int dtype, int T, int d, int k, const int32_t* row_of_assign, void* x_perm) {
    RowCopy c{(const uint4*)x, (uint4*)x_perm, row_of_assign, T, k, (int)((size_t)d * dtype_size(dtype) / 16), 1, 1};
    // a small batch: split every row over several wavefronts until there are a few thousand
    const int unroll = row_copy_unroll(c.chunks);
    while (c.slices < 16 && (int64_t)T * c.slices < 4096 && c.chunks >= 2 * c.slices * kWave * unroll) c.slices *= 2;
    return c;
}

// Wavefront wv's share: slice s % slices of token s / slices for per_wave consecutive s.  The slice of the row is read once
// (16 bytes per lane per piece, UNROLL pieces in flight) and stored to its k destinations.
template <int UNROLL>
__device__ __forceinline__ void copy_rows(const RowCopy& c, int wv) {
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
    const int lane = threadIdx.x & (kWave - 1);
    for (int i = 0; i < c.per_wave; ++i) {
        const int s = wv * c.per_wave + i;
        const int t = s / c.slices, slice = s % c.slices;
        if (t >= c.T) return;
        int rows[MOE_MAX_TOPK];
#pragma unroll
        for (int j = 0; j < MOE_MAX_TOPK; ++j) rows[j] = j < c.k ? c.row_of_assign[(size_t)t * c.k + j] : 0;
        const u32x4* src = (const u32x4*)c.x + (size_t)t * c.chunks;
        u32x4* dst = (u32x4*)c.x_perm;
        for (int c0 = lane + slice * kWave * UNROLL; c0 < c.chunks; c0 += kWave * UNROLL * c.slices) {
            u32x4 v[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                if (c0 + u * kWave < c.chunks) v[u] = src[c0 + u * kWave];
#pragma unroll
            for (int j = 0; j < MOE_MAX_TOPK; ++j)
                if (j < c.k) {
#pragma unroll
                    for (int u = 0; u < UNROLL; ++u)
                        if (c0 + u * kWave < c.chunks) dst[(size_t)rows[j] * c.chunks + c0 + u * kWave] = v[u];
                }
        }
    }
}

// The same in pieces of up to a kilobyte of a row, numbered token by token: pieces [first, end), dealt to the NW wavefronts of the
// workgroup; four reads under way per wavefront.
constexpr int kCopyPieceBytes = kWave * 16;
template <int NW>
__device__ __forceinline__ void copy_pieces(const RowCopy& c, int first, int end, int wave) {
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
    constexpr int U = 4;
    const int lane = threadIdx.x & (kWave - 1);
    const int per_row = ceil_div(c.chunks, kWave);
    for (int p0 = first + wave; p0 < end; p0 += NW * U) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u * NW, t = p / per_row, at = (p - t * per_row) * kWave + lane;
            if (p < end && at < c.chunks) v[u] = ((const u32x4*)c.x)[(size_t)t * c.chunks + at];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u * NW, t = p / per_row, at = (p - t * per_row) * kWave + lane;
            if (p >= end) break;
            for (int j = 0; j < c.k; ++j) {
                const int row = c.row_of_assign[(size_t)t * c.k + j];
                if (at < c.chunks) __builtin_nontemporal_store(v[u], (u32x4*)c.x_perm + (size_t)row * c.chunks + at);
            }
        }
    }
}

}  // namespace moegps
