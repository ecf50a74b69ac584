// Grouped SwiGLU expert FFN (Section 3.4: Mixtral-style FFN with SwiGLU; the
// dominant cost of the layer per the Background's performance discussion):
//     y = ( silu(x W1_e) * (x W3_e) ) W2_e      for every row of a segment whose
//                                               slot hosts expert e.
//
// bf16 path: two persistent grouped GEMMs on the MFMA units.
//   GEMM-1: H[A, ffn]  = swiglu( X[A, d] * [W1|W3]_e )    (gate/up columns interleaved
//           by 32 in the packed weights, so the SwiGLU happens on the accumulators)
//   GEMM-2: Y[A, d]    = H[A, ffn] * W2_e
// Packed weights are stored transposed and by MFMA fragment (see packed_index), activations by row.
// Weights go from memory into registers fragment by fragment, activations through LDS, both to
// v_mfma_f32_16x16x32_bf16 (ffn_tiles.h; with a few rows per expert ffn_stream.h).
//
// Rows are tiled by EXPERT, not by segment: replicas of an expert hold the same
// weights, so the rows of all its segments in the launched slot range are listed
// one after the other (a device-built row list) and cut into M-tiles together;
// an expert then has one ragged tile however many replicas the plan gave it, and
// its weight panels stream once.  The hidden activations are stored in list
// order; the second product writes each result to its own row of y_perm.
// Workgroups claim (M-tile, N-tile) pairs from per-XCD counters in an order that
// keeps the tiles running at the same time on a shared set of weight and
// activation panels.  When the second product has only a few tiles per
// workgroup, its closing tiles are computed as several parts of K (fp32 partial
// sums, added up by a small kernel in a fixed order), so that the last items a
// workgroup claims are short.  The hidden width is padded to a multiple of 64
// inside the packed weights.
//
// The ReLU form (Discussion: Switch Transformer's FFN), y = max(x W1_e, 0) W2_e, runs
// the same two products with another epilogue on the first.
//
// fp32 path (small reference-precision configs): the fp32 matrix instruction, operands from memory.
#include "ffn_tables.h"
#include <atomic>
#include <type_traits>
#include <utility>

namespace moegps {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef f32x4 __attribute__((aligned(4))) f32x4_any;  // four floats at any float's address, still one access
typedef unsigned short bf16_t;  // storage

// ---------------------------------------------------------------------------
// weight packing (one-off, weights are static across inputs)
// ---------------------------------------------------------------------------
// The packed form of a weight matrix is what the GEMM's loads want to find: the transposed
// matrix W^T [N_out][K_out] cut into tiles of kPackN rows by kPackK columns, tiles of one
// row block side by side along K, every tile 32 KiB in one piece.  Inside a tile the matrix is
// stored by MFMA fragment: the 16 rows x 32 columns one v_mfma_f32_16x16x32_bf16 takes are
// 1 KiB in one piece, in lane order (lane 16*q + r holds row r, columns 8q .. 8q+7), the two
// fragments of a 16-row group along K side by side.  So
//   - a k-tile of a weight panel is one contiguous read instead of 256 pieces of 128 bytes a row
//     apart, which the memory system serves a quarter slower at some row lengths (8 KiB among
//     them);
//   - a fragment is loaded into registers as one contiguous kilobyte, without a detour through LDS.
constexpr int kPackN = 256, kPackK = 64;
constexpr int kFragElems = 16 * 32;  // one MFMA operand fragment
__host__ __device__ inline size_t packed_index(int n, int k, int K_out) {
    const int row = n % kPackN, kk = k % kPackK;
    const size_t tile = (size_t)(n / kPackN) * (K_out / kPackK) + k / kPackK;
    const int frag = (row >> 4) * (kPackK / 32) + (kk >> 5);
    return tile * (kPackN * kPackK) + frag * kFragElems + (((kk >> 3) & 3) * 16 + (row & 15)) * 8 + (kk & 7);
}
// Activation tiles keep rows of 128 bytes in LDS: 16-byte piece `slot` of LDS row `row` holds
// piece slot ^ swz(row) of the row.  The LDS
// has 64 four-byte banks and serves a ds_read_b128 sixteen lanes at a time, so the
// 16 consecutive rows one such group touches must land on 16 distinct 16-byte bank
// groups of a 256-byte span: with 128-byte rows that is (row&1, slot) -> xor with
// (row>>1)&7.
__host__ __device__ inline int swz(int row) { return (row >> 1) & 7; }

// out[packed_index(n, k)] = in[k][n] for one expert per blockIdx.z, zero where k >= K or
// n >= N (the output is K_out x N_out, padded); optional interleave of the output row
// index: rows of W1 go to (n/32)*64 + n%32, rows of W3 32 further.  A workgroup turns 32 k x
// 64 n through LDS: 16-byte reads along n (VEC: row length N a multiple of 8, matrix 16-byte aligned), whole
// fragments of 1 KiB written by a wavefront each.
template <bool VEC>
__global__ __launch_bounds__(256) void pack_transpose_kernel(const bf16_t* __restrict__ in, bf16_t* __restrict__ out,
                                                              int K, int N, int K_out, int N_out,
                                                              size_t in_expert_stride, size_t out_expert_stride,
                                                              int interleave, int sel) {
    constexpr int TK = 32, TN = 64, PITCH = TK + 8;
    __shared__ __align__(16) bf16_t tile[TN * PITCH];
    const bf16_t* src = in + (size_t)blockIdx.z * in_expert_stride;
    bf16_t* dst = out + (size_t)blockIdx.z * out_expert_stride;
    const int n0 = blockIdx.x * TN, k0 = blockIdx.y * TK;
    const int tid = threadIdx.x;
    {
        const int kr = tid >> 3, nc = (tid & 7) * 8;
        const int kk = k0 + kr, nn = n0 + nc;
        alignas(16) bf16_t v[8];
        if (VEC && kk < K && nn < N) {
            *(uint4*)v = *(const uint4*)(src + (size_t)kk * N + nn);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = (kk < K && nn + i < N) ? src[(size_t)kk * N + nn + i] : (bf16_t)0;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) tile[(nc + i) * PITCH + kr] = v[i];
    }
    __syncthreads();
    const int row = (tid >> 6) * 16 + (tid & 15), q = (tid >> 4) & 3;
    const int nn = n0 + row;
    if (nn < N_out) {
        const int orow = interleave ? ((nn / 32) * 64 + sel * 32 + (nn % 32)) : nn;
        *(uint4*)(dst + packed_index(orow, k0 + 8 * q, K_out)) = *(const uint4*)&tile[row * PITCH + 8 * q];
    }
}

__global__ void copy_u4_kernel(const uint4* __restrict__ in, uint4* __restrict__ out, size_t n) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) out[i] = in[i];
}

// Workgroup 0 makes the first table, workgroup 1 the second (ffn_tables.h).
__global__ __launch_bounds__(1024) void build_tables_kernel(const int32_t* __restrict__ seg_offsets,
                                                             const int32_t* __restrict__ slot_expert, TableJob job) {
    __shared__ TableScratch<MOE_MAX_SEGMENTS, MOE_MAX_EXPERTS, 1> sh;
    build_tables(sh, blockIdx.x, gridDim.x, blockIdx.x, seg_offsets, slot_expert, job);
}

// ---------------------------------------------------------------------------
// bf16 grouped GEMM on MFMA
// ---------------------------------------------------------------------------
// s_waitcnt with only vmcnt set (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[15:14])
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xf) | (0x7 << 4) | (0xf << 8) | ((N >> 4) << 14));
}

// compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// LDS fragment read issued as an instruction of its own: the compiler does not track
// when the data lands, the kernel waits with lds_wait<N>() ("at most N LDS reads of
// this wavefront still in flight"; LDS reads complete in issue order) and then ties
// the destination registers with lds_landed() before they are used.
template <int OFF>
__device__ __forceinline__ void lds_read_b128(bf16x8& dst, unsigned addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}
template <int N>
__device__ __forceinline__ void lds_wait() {
    static_assert(N >= 0 && N < 16, "lgkmcnt range");
    __builtin_amdgcn_s_waitcnt(0xc07f | (N << 8));  // vmcnt and expcnt untouched
}
__device__ __forceinline__ void lds_landed(bf16x8& v) { asm volatile("" : "+v"(v)); }

// A copy of a lane-dependent value that the compiler cannot trace back: what is computed
// from it is computed where it is used (per tile) instead of once per kernel and then kept
// in a register, or in scratch memory, across the K loop.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
// the same for a value that is uniform over the wavefront (scalar register)
__device__ __forceinline__ int opaque_uniform(int v) {
    asm volatile("" : "+s"(v));
    return v;
}

// With the wavefront seen as four quarters of 16 lanes, p = [p0 p1 p2 p3] and q = [q0 q1 q2 q3]
// become p = [p0 p2 q0 q2] and q = [p1 p3 q1 q3] (two register-to-register swap instructions).
__device__ __forceinline__ void lane_swap_pairs(unsigned& p, unsigned& q) {
    auto r = __builtin_amdgcn_permlane32_swap(p, q, false, false);  // p: [p0 p1 q0 q1], q: [p2 p3 q2 q3]
    auto t = __builtin_amdgcn_permlane16_swap(r[0], r[1], false, false);
    p = t[0];
    q = t[1];
}

// two floats rounded to bf16 (nearest even) and packed, low half first: one conversion instruction
__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// silu(g) = g / (1 + exp(-g)) with the hardware reciprocal (1 ulp) and the hardware
// exponential in place of an IEEE division and expf; the result is rounded to bf16 right after.
__device__ __forceinline__ float silu_f(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// EPI selects what happens to the accumulators before they are stored: kEpiNone (plain
// product, optionally scaled per row), kEpiSwiglu (silu(gate) * up on interleaved column
// pairs, half as many output columns), kEpiRelu (max(., 0)).
constexpr int kEpiNone = 0, kEpiSwiglu = 1, kEpiRelu = 2;

// Where the rows of a product live.  List position p of an M-tile is
//   operand row  a_rows ? a_rows[p] : p, and then, with a_rows2, a_rows2[that] / a_div
//                (the first product reads x_perm through the row list, or rows of x through the list
//                of their tokens, or through the row list and assign_of_row);
//   output row   c_rows ? c_rows[p] : p  (the second product writes y_perm through the row list);
//   output scale scale ? scale[scale_idx[output row]] : 1  (gate weight of the row's assignment).
struct RowMap {
    const int32_t* a_rows;
    const int32_t* a_rows2;
    int a_div;
    const int32_t* c_rows;
    const int32_t* scale_idx;
    const float* scale;
};

// A wavefront's share of the row copy that goes with the first product.
__device__ __forceinline__ void copy_part(const RowCopy& copy, int wv) {
    if (copy.chunks >= 4 * kWave) copy_rows<4>(copy, wv);
    else copy_rows<1>(copy, wv);
}

// n pieces of the row copy (row_copy.h) from number `first` on, and the rows they go to, asked for by a wavefront into
// its LDS at `lds`, kCopyPieceLds bytes each (a piece's bytes past the end of its row and destinations past the k-th come as
// zeros, out of the buffers' ranges) ...
constexpr int kCopyPieceLds = kCopyPieceBytes + kWave * 4;
__device__ __forceinline__ void request_pieces(const RowCopy& c, int first, int n, unsigned char* lds) {
    const unsigned lane = threadIdx.x & (kWave - 1);
    const int per_row = ceil_div(c.chunks, kWave);
    int t = first / per_row, q = first - t * per_row;
    for (int i = 0; i < n; ++i) {
        const auto row = __builtin_amdgcn_make_buffer_rsrc((void*)(c.x + (size_t)t * c.chunks + q * kWave), 0,
                                                           (c.chunks - q * kWave) * 16, 0x00027000);
        const auto ids = __builtin_amdgcn_make_buffer_rsrc((void*)(c.row_of_assign + (size_t)t * c.k), 0, c.k * 4, 0x00027000);
        unsigned char* at = lds + i * kCopyPieceLds;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(row, (__attribute__((address_space(3))) void*)at, 16, lane * 16, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ids, (__attribute__((address_space(3))) void*)(at + kCopyPieceBytes), 4,
                                                 lane * 4, 0, 0, 0);
        if (++q == per_row) {
            q = 0;
            ++t;
        }
    }
}

// ... and, once they have landed (LDS address `at`), stored to these rows, which nothing in the call reads: past the caches.
__device__ __forceinline__ void store_pieces(const RowCopy& c, int first, int n, unsigned at) {
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
    const int lane = opaque((int)threadIdx.x) & (kWave - 1);
    const int per_row = ceil_div(c.chunks, kWave);
    int q = first % per_row;
    for (int i = 0; i < n; ++i, at += kCopyPieceLds) {
        bf16x8 v;
        int row;
        lds_read_b128<0>(v, at + lane * 16);
        asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(row) : "v"(at + lane * 4), "n"(kCopyPieceBytes) : "memory");
        lds_wait<0>();
        lds_landed(v);
        asm volatile("" : "+v"(row));
        u32x4* dst = (u32x4*)c.x_perm + q * kWave + lane;
        if (q * kWave + lane < c.chunks)
            for (int j = 0; j < c.k; ++j)
                __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v),
                                            dst + (size_t)__builtin_amdgcn_readlane(row, j) * c.chunks);
        if (++q == per_row) q = 0;
    }
}

#include "ffn_tiles.h"
#include "ffn_stream.h"

// Adds up the fp32 slabs of every split M-tile in the order of the parts and writes the rows
// as bf16: y[c_rows[list0 + r]] = scale * (((P_0[r] + P_1[r]) + P_2[r]) + ...).  blockIdx.x =
// split tile, blockIdx.y strides over its rows; counts[kCntSplit] = number of such tiles.
__global__ __launch_bounds__(256) void add_partials_kernel(const float* __restrict__ partials,
                                                            const SplitInfo* __restrict__ splits,
                                                            const int32_t* __restrict__ counts, int parts,
                                                            bf16_t* __restrict__ C, int ldc, int N, RowMap rm) {
    const int n_split = counts[kCntSplit];
    const int n4 = N / 4;
    for (int t = blockIdx.x; t < n_split; t += gridDim.x) {
        const SplitInfo si = splits[t];
        const float* p0 = partials + (size_t)t * parts * kPartRows * N;
        for (int r = blockIdx.y; r < si.rows; r += gridDim.y) {
            int crow = si.list0 + r;
            float sc = 1.0f;
            if (rm.c_rows) crow = rm.c_rows[crow];
            if (rm.scale) sc = rm.scale[rm.scale_idx[crow]];
            uint2* out = (uint2*)(C + (size_t)crow * ldc);
            for (int c = threadIdx.x; c < n4; c += blockDim.x) {
                float4 s = ((const float4*)(p0 + (size_t)r * N))[c];
                for (int q = 1; q < parts; ++q) {
                    const float4 v = ((const float4*)(p0 + ((size_t)q * kPartRows + r) * N))[c];
                    s.x += v.x;
                    s.y += v.y;
                    s.z += v.z;
                    s.w += v.w;
                }
                uint2 o;
                o.x = pack_bf16x2(s.x * sc, s.y * sc);
                o.y = pack_bf16x2(s.z * sc, s.w * sc);
                out[c] = o;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// fp32 grouped GEMM on the fp32 matrix instruction
// ---------------------------------------------------------------------------
// The fp32 layers are small (8 experts of 128 x 256 and a few hundred rows), so a product is bound
// by how often it waits for memory one request after the other, not by arithmetic or bytes.  A
// workgroup is four wavefronts side by side, 16 columns each, over 16 * MT rows; every wavefront
// takes its operands from memory straight into registers (the rows are shared between the four
// through the L1), two chunks of CH 16-deep steps in flight, and nothing synchronises.  A
// v_mfma_f32_16x16x4_f32 takes four k at a time: lane (l16, g16) holds k = 16 s + 4 g16 + j for
// instruction j of step s, so that a lane's four activation values are one 16-byte load.
// Against a 64 x 64 LDS tile with vector FMAs (two barriers and an exposed memory round trip per
// 16 k), the whole FFN: 8 experts of 128 x 256, 512 rows 78 -> 32 us (down product alone before: 37),
// 4096 rows 80 -> 46; 8 experts of 1024 x 2048, 512 rows 616 -> 254 us, 8192 rows 2464 -> 1658.
// Relative error against 64 bits, old and new: 4.1e-7 and 4.1e-7 (128 x 256), 1.2e-6 and 1.2e-6 (1024 x 2048).
// MT = 2 where 64-row tiles would leave most of the 256 CUs without one, else MT = 4, which reads
// the weights half as often.
template <int MT, bool SWIGLU>
__global__ __launch_bounds__(256) void grouped_gemm_f32_kernel(const float* __restrict__ A, int lda,
                                                                const float* __restrict__ B1,
                                                                const float* __restrict__ B3, size_t b_stride,
                                                                float* __restrict__ C, int ldc,
                                                                const MTile* __restrict__ mtiles,
                                                                const int32_t* __restrict__ counts, int N,
                                                                int K, RowMap rm, int relu, int grid, RowCopy copy) {
    constexpr int BN = 64;
    constexpr int CH = MT == 2 ? 4 : 2;  // 16-deep steps per chunk
    constexpr int NB = SWIGLU ? 2 : 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int l16 = lane & 15, g16 = lane >> 4;
    const int n_ntiles = (N + BN - 1) / BN;
    const int total = counts[kCntEntries] * n_ntiles;
    const int n_chunks = (K + 16 * CH - 1) / (16 * CH);
    if (blockIdx.x < gridDim.x - grid) {
        copy_part(copy, (int)blockIdx.x * (int)(blockDim.x / kWave) + wave);
        return;
    }
    for (int tile = (int)blockIdx.x - (int)(gridDim.x - grid); tile < total; tile += grid) {
        const MTile mt = mtiles[tile / n_ntiles];
        const int n0 = (tile % n_ntiles) * BN + wave * 16;
        if (n0 >= N) continue;
        const int col = n0 + l16 < N ? n0 + l16 : N - 1;  // columns past the edge repeat the last one and are dropped
        const float* b[NB];
        b[0] = B1 + (size_t)mt.expert * b_stride + col;
        if constexpr (SWIGLU) b[1] = B3 + (size_t)mt.expert * b_stride + col;
        const float* arow[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            int r = i * 16 + l16;
            r = mt.list0 + (r < mt.rows ? r : mt.rows - 1);
            if (rm.a_rows) {
                r = rm.a_rows[r];
                if (rm.a_rows2) r = rm.a_rows2[r] / rm.a_div;
            }
            arow[i] = A + (size_t)r * lda;
        }
        f32x4 acc[NB][MT];
#pragma unroll
        for (int m = 0; m < NB; ++m)
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[m][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        struct Chunk {
            f32x4 a[CH][MT];
            float w[CH][NB][4];
        };
        // K is a multiple of 4, so a lane's four k are all inside or all outside; outside both
        // operands are zero (a zero against whatever the weights hold would not do: inf * 0)
        auto load = [&](int c, Chunk& o) {
#pragma unroll
            for (int s = 0; s < CH; ++s) {
                const int k = (c * CH + s) * 16 + 4 * g16;
                const bool in = k < K;
                const int kc = in ? k : 0;
#pragma unroll
                for (int i = 0; i < MT; ++i) {
                    const f32x4 v = *(const f32x4_any*)(arow[i] + kc);
                    o.a[s][i] = in ? v : f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int m = 0; m < NB; ++m)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float v = b[m][(size_t)(kc + j) * N];
                        o.w[s][m][j] = in ? v : 0.f;
                    }
            }
        };
        auto multiply = [&](const Chunk& o) {
#pragma unroll
            for (int s = 0; s < CH; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int m = 0; m < NB; ++m)
                            acc[m][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.w[s][m][j], o.a[s][i][j], acc[m][i], 0, 0, 0);
        };
        Chunk even, odd;
        load(0, even);
        for (int c = 0; c < n_chunks; c += 2) {  // (chunks past the end are all zeros)
            load(c + 1, odd);
            multiply(even);
            if (c + 1 >= n_chunks) break;
            load(c + 2, even);
            multiply(odd);
        }
        // lane (l16, g16) holds columns n0 + 4 g16 .. + 3 of row i * 16 + l16
        const int c0 = n0 + 4 * g16;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int row = i * 16 + l16;
            if (row >= mt.rows || c0 >= N) continue;
            int crow = mt.list0 + row;
            float sc = 1.0f;
            if (rm.c_rows) crow = rm.c_rows[crow];
            if (rm.scale) sc = rm.scale[rm.scale_idx[crow]];
            f32x4 v = acc[0][i];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (SWIGLU) v[j] = v[j] / (1.0f + expf(-v[j])) * acc[NB - 1][i][j];
                else if (relu) v[j] = fmaxf(v[j], 0.f);
                v[j] *= sc;
            }
            *(f32x4_any*)(C + (size_t)crow * ldc + c0) = v;
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct FfnWs {
    void* h;            // [A, ffn] hidden activations, in row-list order
    int32_t* rowlist;   // [A] row of x_perm / y_perm at each list position
    MTile* tiles1;      // M-tile table of the first product
    MTile* tiles2;      // and of the second
    int32_t* counts;    // kCntStride ints per table
    int32_t* queues;    // [0..7], [8..15]: per-XCD claim counters of the two products
    SplitInfo* splits;  // split M-tiles of the second product, else null
    float* partials;    // their fp32 slabs: [split tile][part][kPartRows][d]
    int capacity;       // entries per table
    int split_capacity; // split M-tiles (0: the second product is never split)
    int parts;          // parts of K of a split tile
    int split_all;      // every tile is split (tests)
};

constexpr int kMinBM = 32;  // the lowest tile shape

// Process-wide overrides of the automatic choices (moe_grouped_ffn_set_option); -1 / 0 = automatic.
static std::atomic<int> g_opt_tile1{-1}, g_opt_tile2{-1}, g_opt_split{-1}, g_opt_group_n{0}, g_opt_stream{-1};

FfnOptions ffn_options() {
    return {g_opt_tile1.load(), g_opt_tile2.load(), g_opt_split.load(), g_opt_group_n.load(), g_opt_stream.load()};
}

// The bf16 kernels work on a hidden width padded to a multiple of 64: the packed weights
// carry zero columns (W1, W3) and zero rows (W2) for the padding, so the padded hidden
// activations are exact zeros and add nothing to the second product.
// Widths above this are refused: it keeps every size computed on the host inside 64 bits and
// every tile offset computed on the device inside 32.
constexpr int kMaxWidth = 1 << 22;
static inline bool ffn_shape_in_range(int64_t A, int d, int ffn, int nseg, int dtype) {
    return (dtype == MOE_DTYPE_F32 || dtype == MOE_DTYPE_BF16) && A >= 0 && A < (1ll << 31) && d >= 1 &&
           d <= kMaxWidth && ffn >= 1 && ffn <= kMaxWidth && nseg >= 1 && nseg <= MOE_MAX_SEGMENTS;
}

static inline int padded_ffn(int ffn, int dtype) {
    return dtype == MOE_DTYPE_BF16 ? (int)align_up((size_t)ffn, 64) : ffn;
}
// rows of a packed bf16 weight matrix: whole tiles
static inline size_t packed_rows(size_t n) { return align_up(n, (size_t)kPackN); }
// elements of one expert's packed matrices: the first product's n1 matrices, the second product's
static inline size_t packed_elems1(int n1, int d, int fp) { return packed_rows((size_t)n1 * fp) * d; }
static inline size_t packed_elems2(int d, int fp) { return packed_rows((size_t)d) * fp; }

// Whether (and how) the closing tiles of the second product are computed as parts of K.  It
// pays when the product has only a few rounds of tiles per workgroup, so that the uneven end
// of the launch matters, and the segments are not slivers (splitting K would only add
// traffic).  Decided from the sizes the workspace is laid out for, so that the layout and the call
// agree; the number of experts is not among them, so a batch that streams its weights (stream_form) has
// room for slabs that it leaves unused.  split_capacity bounds the M-tiles the table builder may split: more than 5/8 of a
// round of tiles, and no more than there are of 128 rows.  Lower tiles can be more; where the builder's rule asks
// for more than there is room for, which takes narrow outputs and a batch that is less than a round in all, it splits
// none.  Room for all of them would be worse, both products, us, none split -> all: 8 experts of 512 x 1024, 1001 / 2048
// tokens 35 -> 44 / 41 -> 59; 8 of 1024 x 4096, 1001 tokens 83 -> 98; 8 of 768 x 3072, 3000 tokens 60 -> 73.
// mode: 0 never, 1 every tile whenever the kernels can (for tests), -1 the rule.
static void split_plan(int64_t A, int d, int ffn, int nseg, int dtype, int mode, int* split_capacity, int* parts,
                       int* split_all) {
    *split_capacity = *parts = *split_all = 0;
    if (dtype != MOE_DTYPE_BF16 || A < 1) return;
    if (mode == 0) return;
    const int kt = padded_ffn(ffn, dtype) / 64;
    const int n_ntiles = ceil_div(d, 256);
    const int64_t all_mtiles = ceil_div64(A, 128) + (A < nseg ? A : nseg);
    if (mode == 1) {
        if (kt < 2) return;
        *parts = kt >= kMaxParts ? kMaxParts : 2;
        *split_all = 1;
        *split_capacity = (int)(ceil_div64(A, kMinBM) + (A < nseg ? A : nseg));  // every M-tile of any shape
        return;
    }
    if (kt < 4 * kMaxParts) return;
    // fewer than 64 rows per slot: splitting a tile of a few k-tiles only adds traffic, but a
    // long one (64 k-tiles and more) is worth splitting where the tiles do not fill the chip (8 experts
    // of hidden width 14336, 128 to 512 tokens: 96 tiles of 224 k-tiles for 256 workgroups; eight parts
    // instead of four were 5-20 % slower there, adding up the slabs cost more than the extra round saved)
    if (A < (int64_t)64 * nseg && kt < 64) return;
    const int64_t est_tiles = (A / 256 + (nseg + 1) / 2) * n_ntiles;
    if (est_tiles > 8 * kGemmGrid) return;
    *parts = kMaxParts;
    const int64_t by_rule = (int64_t)2 * ceil_div(5 * kGemmGrid / 8, n_ntiles) + 2;
    *split_capacity = (int)(by_rule < all_mtiles ? by_rule : all_mtiles);
}

static size_t ffn_ws_layout(int64_t A, int d, int ffn, int nseg, int dtype, int split, char* base, FfnWs* ws) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void* p = base ? (void*)(base + off) : nullptr;
        off += align_up(bytes, 256);
        return p;
    };
    const int64_t A1 = A > 0 ? A : 1;
    FfnWs w;
    split_plan(A, d, ffn, nseg, dtype, split, &w.split_capacity, &w.parts, &w.split_all);
    w.capacity = (int)(ceil_div64(A1, kMinBM) + nseg + (int64_t)w.split_capacity * kMaxParts);
    w.h = take((size_t)A1 * padded_ffn(ffn, dtype) * dtype_size(dtype));
    w.rowlist = (int32_t*)take((size_t)A1 * sizeof(int32_t));
    w.tiles1 = (MTile*)take((size_t)w.capacity * sizeof(MTile));
    w.tiles2 = (MTile*)take((size_t)w.capacity * sizeof(MTile));
    w.counts = (int32_t*)take(256);
    w.queues = w.counts ? w.counts + 2 * kCntStride : nullptr;
    w.splits = nullptr;
    w.partials = nullptr;
    if (w.split_capacity > 0) {
        w.splits = (SplitInfo*)take((size_t)w.split_capacity * sizeof(SplitInfo));
        w.partials = (float*)take((size_t)w.split_capacity * w.parts * kPartRows * d * sizeof(float));
    }
    if (ws) *ws = w;
    return off;
}

// Tile heights of the options: tables of up to 256, 128 or 32 rows per tile.
constexpr int kNumShapes = 3;
constexpr int kShapeRows[kNumShapes] = {256, 128, 32};

// timing hook: events recorded around the two products of the next call on this thread
static thread_local hipEvent_t g_time_events[4];
static thread_local bool g_time_armed = false;

static int num_cus() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            cus = prop.multiProcessorCount;
        if (cus <= 0) cus = 256;
    }
    return cus;
}

// Weights of a product above this are read past the caches by tiles that share them with no other tile: the
// next product or call would not find them there anyway.  128 MiB is half the memory-side cache, which the weights
// of both products pass through.  Below it the caches are worth more: 16 experts of 1024 x 512 (16 + 8 MiB), 1500 tokens,
// both products 33 us through the caches, 35 past them.  Above it: see the K loop of the tile kernel.
constexpr size_t kCachedWeights = (size_t)128 << 20;

// Workgroups that a row copy adds to a launch of workgroups of `threads` threads: none without one.  A wavefront moves
// 32 KiB at least, once there are a few thousand of them.  They come first in the grid where a workgroup of the
// product goes on to another as soon as it has run out of units: last, they are what the launch waits for (16 tokens on 8 experts of
// 4096 x 14336, whole step 333 -> 326 us).  In the second streaming form, whose workgroups all fit on the chip at once, they come last: first,
// they keep some of these waiting (128 tokens on 128 experts of 4096 x 1536 542 -> 533).
static int copy_blocks(RowCopy& copy, int threads) {
    if (!copy.x_perm || copy.T < 1) return 0;
    const int64_t bytes = (int64_t)(copy.k + 1) * copy.chunks * 16 / copy.slices;
    const int64_t spare = (int64_t)copy.T * copy.slices / 4096, most = ceil_div64(32768, bytes);
    copy.per_wave = (int)(spare < 1 ? 1 : spare < most ? spare : most);
    return (int)ceil_div64((int64_t)copy.T * copy.slices, (int64_t)copy.per_wave * (threads / kWave));
}

static bool past_caches(int E, size_t b_stride) { return (size_t)E * b_stride * sizeof(bf16_t) > kCachedWeights; }

// A kernel that uses more LDS than the default limit: raised once per kernel (`raised`: bit per device).
static int raise_lds(const void* kern, size_t bytes, std::atomic<unsigned long long>& raised) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    const unsigned long long bit = 1ull << (dev & 63);
    if (raised.load() & bit) return MOE_OK;
    const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) {
        set_last_hip_error(e);
        return MOE_ERR_HIP;
    }
    raised.fetch_or(bit);
    return MOE_OK;
}

template <int EPI>
static int launch_tiles(const bf16_t* A, int lda, const bf16_t* Bp, size_t b_stride, int E, bf16_t* C, int ldc,
                        const MTile* tiles, const int32_t* counts, int32_t* queues, int N, int K, int group_n,
                        const RowMap& rm, float* partials, RowCopy copy, hipStream_t st) {
    // (the kernel multiplies by it: an option beyond the N-tiles there are means all of them)
    if (group_n > ceil_div(N, kPackN)) group_n = ceil_div(N, kPackN);
    const auto kern = grouped_gemm_tile_kernel<EPI>;
    static std::atomic<unsigned long long> raised{0};
    if (const int rc = raise_lds((const void*)kern, kTileLds<EPI>, raised); rc != MOE_OK) return rc;
    // 32 workgroups for each of the 8 XCDs; they claim tiles from `queues` (cleared by the table builder)
    hipLaunchKernelGGL(kern, dim3(kGemmGrid), dim3(512), kTileLds<EPI>, st, A, lda, Bp, b_stride, C, ldc, tiles, counts, queues, N, K,
                       group_n, past_caches(E, b_stride), rm, partials, copy);
    return check_launch();
}

// Whether both products share a launch (ffn_tiles.h).  It saves what the uneven end of the first product costs, half a tile
// per workgroup on average, and costs what writing the hidden rows through to memory does (2 % at 16 rounds of tiles).  Whole
// steps, us, a launch each -> one, by the rounds of 256 tiles that the first product has at 256 rows per tile: 1.8 (64 experts of
// 2048 x 1408, 400 tokens) 222 -> 206, 2.0 (16 of 4096 x 688, 5000) 420 -> 398, 5.5 (64 of 2048 x 1408, 4096) 555 -> 546, 5.9 (128
// of 4096 x 1536, 2000) 971 -> 954, 7.4 (64 of 2048 x 1408, 6000) 674 -> 670, 8.8 (8 of 4096 x 14336, 2000) 1270 -> 1277, 10.4 (64
// of 2048 x 1408, 9000) 918 -> 929.  Below a round there is little to fill (64 of 768 x 3072, 2000 tokens 142 -> 143).
// A first product of few k-tiles is done before the hand-over is.  d / 64 = 6 / 8 / 9 / 10 / 11 at hidden width 2048: 8 experts, 4096
// tokens 105 -> 111 / 105 -> 111 / 114 -> 122 / 119 -> 126 / 132 -> 139; 64 experts, 8192 tokens, popularity 10 186 -> 195 /
// 204 -> 205 / 234 -> 230 / 255 -> 252 / 266 -> 261.
// A long second product keeps its launch: a tile of all its k-tiles is what the shared launch ends with, where a launch of its own has
// closing tiles in parts of K.  8 experts of 4096 x 14336 (224 k-tiles), rows as a popularity of 0.1 / 1 / 10 has them, 384 tokens 373 ->
// 385 / 567 -> 560 / 566 -> 554, 640 500 -> 499 / 674 -> 672 / 646 -> 636, 1001 659 -> 673 / 814 -> 852 / 775 -> 790, 1024 674 -> 694 /
// 840 -> 821 / 789 -> 792, 1400 821 -> 848 / 984 -> 1005 / 946 -> 958; below 384 it is further behind (128 tokens 252 -> 332 at 0.1).
// 70 shapes drawn inside these lines (12 to 64 and 4 to 60 k-tiles, 8 to 128 experts): 3.2 % ahead on average, 0.91 to 1.30; behind
// is above all 8 experts with a first product of 12 to 16 k-tiles (0.91 to 1.02).
static bool one_launch(int64_t A, int E, int n_ntiles1, int k_tiles1, int k_tiles2) {
    const int64_t tiles = (ceil_div64(A, kTallest) + (A < E ? A : E) / 2) * n_ntiles1;
    return tiles >= kGemmGrid && tiles <= 7 * kGemmGrid && k_tiles1 >= 12 && k_tiles2 < 64;
}

template <int EPI>
static int launch_both(const bf16_t* X, int d, const bf16_t* P13, size_t stride1, const bf16_t* P2, size_t stride2, int E,
                       const FfnWs& ws, int fp, bf16_t* Y, const MTile* tiles2, const int32_t* counts2, const RowMap& rm1,
                       const RowMap& rm2, const RowCopy& copy, int32_t* left, hipStream_t st) {
    const auto kern = grouped_ffn_tiles_kernel<EPI>;
    static std::atomic<unsigned long long> raised{0};
    if (const int rc = raise_lds((const void*)kern, kTileLds<EPI>, raised); rc != MOE_OK) return rc;
    hipLaunchKernelGGL(kern, dim3(kGemmGrid), dim3(512), kTileLds<EPI>, st, X, d, P13, stride1, P2, stride2, (bf16_t*)ws.h, fp,
                       Y, ws.tiles1, tiles2, ws.counts, counts2, ws.queues, past_caches(E, stride1), past_caches(E, stride2),
                       rm1, rm2, copy, left);
    return check_launch();
}

// Whether a product streams its weights through registers (ffn_stream.h): 0 no, else the form.
// The rule goes by the whole batch (A rows, E experts), not by the launched slot range, so that
// a row gets the same bits from a launch over some slots as from one over all.  How the rows lie is
// only known on the device, so a line has to do for all rows on one expert as well as for an equal share
// on each.  The lines were drawn against tiles that took longer for few rows than the present ones: what they give up for
// batches on a few experts is now more than they gain on spread ones.  Both products, us, tiles -> streaming, rows on so
// many experts, with the present tiles:
//   up to 16 rows per expert on average: 128 experts of 4096 x 1536 on 128 / 16 / 1, 512 rows 721 -> 704 / 121 -> 107 /
//     58 -> 50, 1024 rows 721 -> 718 / 125 -> 118 / 62 -> 60, 1536 rows 734 -> 727 / 131 -> 155 / 76 -> 100, 2048 rows 743 -> 737 /
//     136 -> 165 / 91 -> 105; 64 of 2048 x 1408, 1024 rows on 64 / 16 / 1 187 -> 190 / 78 -> 67 / 43 -> 40; 8 of 4096 x 14336
//     on 8 / 2 / 1, 64 rows 472 -> 451 / 155 -> 136 / 135 -> 112, 128 rows 466 -> 422 / 161 -> 174 / 125 -> 134; but not with
//     so many experts that the tiles of A rows on one of them are more than 128 k-tiles per CU (512 experts of 4096 x 1536,
//     first product, 6144 rows on 512 / 64 / 8 1875 -> 1983 / 263 -> 372 / 132 -> 218);
//   up to 24 where those are no more than 18 per CU and K is not short (64 experts of 2048 x 1408, 132 tiles of 32 and 96 of
//     22, 1536 rows on 64 / 16 / 1 191 -> 190 / 83 -> 80 / 47 -> 59); with more than that too much is lost (128 experts of
//     4096 x 1536, 240 tiles of 64 and 320 of 24, 2560 rows on 128 / 32 / 16 745 -> 763 / 237 -> 282 / 144 -> 211; 64 of
//     4096 x 4096, second product, 160 tiles of 64, 1280 rows on 16 / 8 / 4 97 -> 125 / 64 -> 90 / 64 -> 85; 1024 of
//     1024 x 512, second product, 8 k-tiles, 18432 rows on 16 / 1 36 -> 46 / 31 -> 45);
//   up to 64 where even every expert's own ragged 128 x 256 tiles would not go once round the chip (16 experts of 4096 x
//     688, 1024 rows on 16 / 4 / 1 88 -> 67 / 54 -> 49 / 53 -> 49).
// Above 16 rows per expert a long K is left to the tiles in any case, their closing ones are computed as parts of K (8
// experts, K = 14336, second product, 192 rows on 8 / 2 / 1 189 -> 145 / 90 -> 113 / 63 -> 110).
// Of the two, form 1 (finer units) takes what the 128-column units of form 2 would not bring round the 512
// workgroups the chip holds, up to 16 rows per expert (8 experts, K = 14336, second product, 32 rows on 8 / 4
// 139 against 148 / 74 against 94), and small batches of up to 4 (64 experts of 2048 x 1408, first
// product, 256 rows on 64 118 against 128).  The rest is form 2's, which reads the activations half as
// often: 128 experts of 4096 x 1536, first product, 512 rows on 128 / 1 580 against 486 / 57 against 33; 512
// experts, 2048 rows on 512 / 8 2235 against 1893 / 176 against 88.
static int stream_form(int opt, int forced_tile, int64_t A, int E, int n_cols, int k_tiles) {
    if (forced_tile >= 0 || opt == 0 || A > 65536) return 0;
    if (opt > 0) return opt;
    const int64_t m_tiles = ceil_div64(A, 128), n_tiles = ceil_div(n_cols, 256);
    const int64_t work = m_tiles * n_tiles * k_tiles;  // k-tiles of A rows on one expert
    if (work > 128 * kGemmGrid) return 0;
    if (A > (int64_t)16 * E) {
        const bool idle = work <= 18 * kGemmGrid && k_tiles > 16;
        const bool once = (m_tiles + E) * n_tiles <= kGemmGrid;
        return k_tiles <= 64 && ((A <= (int64_t)24 * E && idle) || (A <= (int64_t)64 * E && once)) ? 2 : 0;
    }
    if (A <= (int64_t)4 * E && A <= 256) return 1;
    return (A < E ? A : E) * (n_cols / 128) >= 2 * kGemmGrid ? 2 : 1;
}

template <int EPI>
static int launch_stream(int form, int64_t A, int E, const bf16_t* X, int lda, const bf16_t* Bp, size_t b_stride,
                         bf16_t* C, int ldc, const MTile* tiles, const int32_t* counts, int N, int K, const RowMap& rm,
                         RowCopy copy, hipStream_t st) {
    auto go = [&](auto kern, int grid, int threads) {
        const int all = grid + copy_blocks(copy, threads);
        hipLaunchKernelGGL(kern, dim3(all), dim3(threads), 0, st, X, lda, Bp, b_stride, C, ldc, tiles, counts, N, K, rm, grid,
                           copy);
        return check_launch();
    };
    // The registers let a CU hold two workgroups of form 2; of form 1 one (<4, 8>) or two, its kernels
    // having been compiled for M-tiles of up to 64 rows.  Form 1 is launched with more than that, so
    // that a CU goes on to the next one as soon as one has run out of units.
    if (form == 2) return go(grouped_gemm_stream_shared_kernel<EPI>, 2 * kGemmGrid, 512);
    // Units of 32 columns where those of 64 would make fewer than three per CU (one token, 8 experts
    // of 3072 columns: 37 -> 35 us; 16 tokens, 4096 columns over K = 14336: 107 -> 98 us) and the
    // activation fragments, read for every unit, are few.  A short K is split four ways instead of
    // eight: three k-tiles per wavefront and less would be mostly prologue (24 k-tiles, 128 experts:
    // 170 -> 166 us; 64 k-tiles: 307 against 315 us the other way).
    const int64_t experts = A < E ? A : E;
    if (A <= (int64_t)8 * E && experts * (N / 64) < 3 * kGemmGrid)
        return go(grouped_gemm_stream_ksplit_kernel<2, 8, EPI>, 3 * kGemmGrid, 512);
    if (K / kPackK <= 32) return go(grouped_gemm_stream_ksplit_kernel<4, 4, EPI>, 4 * kGemmGrid, 256);
    return go(grouped_gemm_stream_ksplit_kernel<4, 8, EPI>, 3 * kGemmGrid, 512);
}

}  // namespace moegps

extern "C" int moe_grouped_ffn_set_option(int option, int value) {
    using namespace moegps;
    switch (option) {
        case MOE_FFN_OPT_TILE1:
        case MOE_FFN_OPT_TILE2:
            if (value < -1 || value >= kNumShapes) return MOE_ERR_INVALID_ARG;
            (option == MOE_FFN_OPT_TILE1 ? g_opt_tile1 : g_opt_tile2).store(value);
            return MOE_OK;
        case MOE_FFN_OPT_SPLIT_K:
            if (value < -1 || value > 1) return MOE_ERR_INVALID_ARG;
            g_opt_split.store(value);
            return MOE_OK;
        case MOE_FFN_OPT_GROUP_N:
            if (value < 0) return MOE_ERR_INVALID_ARG;
            g_opt_group_n.store(value);
            return MOE_OK;
        case MOE_FFN_OPT_STREAM:
            if (value < -1 || value > 2) return MOE_ERR_INVALID_ARG;
            g_opt_stream.store(value);
            return MOE_OK;
        default:
            return MOE_ERR_INVALID_ARG;
    }
}

extern "C" size_t moe_packed_weights_bytes(int E, int d, int ffn, int dtype) {
    using namespace moegps;
    if (E < 1 || E > MOE_MAX_EXPERTS || !ffn_shape_in_range(0, d, ffn, 1, dtype)) return 0;
    if (dtype != MOE_DTYPE_BF16) return (size_t)3 * E * d * ffn * dtype_size(dtype);
    const int fp = padded_ffn(ffn, dtype);
    return (size_t)E * (packed_elems1(2, d, fp) + packed_elems2(d, fp)) * sizeof(bf16_t);
}

namespace moegps {
// W3 == nullptr packs the ReLU form (no gate matrix): [W1 | W2] instead of [W1 W3 | W2]
static int pack_weights_impl(const void* W1, const void* W3, const void* W2, int dtype, int E, int d, int ffn,
                             void* packed, void* stream) {
    if (dtype != MOE_DTYPE_F32 && dtype != MOE_DTYPE_BF16) return MOE_ERR_INVALID_ARG;
    if (E < 1 || d < 1 || ffn < 1 || !W1 || !W2 || !packed) return MOE_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    const size_t per = (size_t)E * d * ffn;
    if (dtype == MOE_DTYPE_F32) {
        if ((per * 4) % 16 != 0) return MOE_ERR_UNSUPPORTED;
        const void* src[3] = {W1, W3 ? W3 : W2, W2};
        const int n = W3 ? 3 : 2;
        for (int i = 0; i < n; ++i) {
            hipLaunchKernelGGL(copy_u4_kernel, dim3(1024), dim3(256), 0, st, (const uint4*)src[i],
                               (uint4*)((float*)packed + i * per), per * 4 / 16);
            int rc = check_launch();
            if (rc != MOE_OK) return rc;
        }
        return MOE_OK;
    }
    if (d % 64 != 0) return MOE_ERR_UNSUPPORTED;
    if (E > 65535) return MOE_ERR_UNSUPPORTED;
    const int fp = padded_ffn(ffn, dtype);
    const int n1 = W3 ? 2 : 1;              // matrices in the first product
    const size_t es = (size_t)d * ffn;      // one expert's matrix as given
    const size_t e1 = packed_elems1(n1, d, fp), e2 = packed_elems2(d, fp);  // and packed
    bf16_t* p1 = (bf16_t*)packed;           // [E] packed [n1*fp][d]; gate/up interleaved by 32 columns when n1 = 2
    bf16_t* p2 = p1 + (size_t)E * e1;       // [E] packed [d][fp]
    // W1 (, W3): in[k = d][n = ffn] -> rows n' of the packed matrix, zero rows for n >= ffn and up
    // to whole tiles of rows
    const int rows1 = (int)(packed_rows((size_t)n1 * fp) / n1);  // rows per matrix, padding included
    auto pack = [&](const void* W, bf16_t* out, int K, int N, int K_out, int N_out, size_t out_stride, int interleave,
                    int sel) {
        const dim3 grid(ceil_div(N_out, 64), K_out / 32, E);
        if (N % 8 == 0 && (uintptr_t)W % 16 == 0)
            hipLaunchKernelGGL(pack_transpose_kernel<true>, grid, dim3(256), 0, st, (const bf16_t*)W, out, K, N, K_out,
                               N_out, es, out_stride, interleave, sel);
        else
            hipLaunchKernelGGL(pack_transpose_kernel<false>, grid, dim3(256), 0, st, (const bf16_t*)W, out, K, N, K_out,
                               N_out, es, out_stride, interleave, sel);
        return check_launch();
    };
    int rc = pack(W1, p1, d, ffn, d, rows1, e1, W3 ? 1 : 0, 0);
    if (rc == MOE_OK && W3) rc = pack(W3, p1, d, ffn, d, rows1, e1, 1, 1);
    // W2: in[k = ffn][n = d] -> packed [n = d][k = fp], zero for k >= ffn and rows n >= d
    if (rc == MOE_OK) rc = pack(W2, p2, ffn, d, fp, (int)packed_rows((size_t)d), e2, 0, 0);
    return rc;
}
}  // namespace moegps

extern "C" int moe_pack_weights(const void* W1, const void* W3, const void* W2, int dtype, int E, int d, int ffn,
                                void* packed, void* stream) {
    if (!W3) return MOE_ERR_INVALID_ARG;
    return moegps::pack_weights_impl(W1, W3, W2, dtype, E, d, ffn, packed, stream);
}

extern "C" size_t moe_packed_weights_relu_bytes(int E, int d, int ffn, int dtype) {
    using namespace moegps;
    if (E < 1 || E > MOE_MAX_EXPERTS || !ffn_shape_in_range(0, d, ffn, 1, dtype)) return 0;
    if (dtype != MOE_DTYPE_BF16) return (size_t)2 * E * d * ffn * dtype_size(dtype);
    const int fp = padded_ffn(ffn, dtype);
    return (size_t)E * (packed_elems1(1, d, fp) + packed_elems2(d, fp)) * sizeof(bf16_t);
}

extern "C" int moe_pack_weights_relu(const void* W1, const void* W2, int dtype, int E, int d, int ffn, void* packed,
                                     void* stream) {
    return moegps::pack_weights_impl(W1, nullptr, W2, dtype, E, d, ffn, packed, stream);
}

extern "C" size_t moe_grouped_ffn_workspace_bytes(int64_t A, int d, int ffn, int nseg, int dtype) {
    using namespace moegps;
    if (!ffn_shape_in_range(A, d, ffn, nseg, dtype)) return 0;
    return ffn_ws_layout(A, d, ffn, nseg, dtype, ffn_options().split, nullptr, nullptr);
}

namespace moegps {
// Rows of the first product: x_perm rows in place (gather_rows == nullptr; `rows_in` = A), or
// row r is x[gather_rows[r] / gather_div] (`rows_in` = rows of x).  With `scale`, row r of
// the output is multiplied by scale[scale_idx[r]] before it is rounded.
int grouped_ffn_call(int relu, const void* x_in, int64_t rows_in, const int32_t* gather_rows, int gather_div,
                     const int32_t* scale_idx, const float* scale, int dtype, int64_t A, int d, int ffn, int E,
                     const int32_t* seg_offsets, const int32_t* slot_expert, int nseg, int seg_begin, int seg_end,
                     const void* packed, void* y_perm, void* workspace, size_t workspace_bytes, void* stream,
                     const FfnOptions& opt, FfnStage stage, TableJob* job_out, const RowCopy& copy, int32_t* tokens) {
    const bool armed = g_time_armed, timed = armed && stage != kFfnJobOnly;
    if (stage != kFfnJobOnly) g_time_armed = false;  // the hook belongs to this call, whatever becomes of it
    if (dtype != MOE_DTYPE_F32 && dtype != MOE_DTYPE_BF16) return MOE_ERR_INVALID_ARG;
    if (A < 0 || d < 1 || ffn < 1 || E < 1 || nseg < 1) return MOE_ERR_INVALID_ARG;
    if (seg_begin < 0 || seg_end > nseg || seg_begin > seg_end) return MOE_ERR_INVALID_ARG;
    if (nseg > MOE_MAX_SEGMENTS || E > MOE_MAX_EXPERTS || A >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;
    if (d > kMaxWidth || ffn > kMaxWidth) return MOE_ERR_UNSUPPORTED;
    if (dtype == MOE_DTYPE_BF16 && d % 64 != 0) return MOE_ERR_UNSUPPORTED;
    if (dtype == MOE_DTYPE_F32 && (d % 4 != 0 || ffn % 4 != 0)) return MOE_ERR_UNSUPPORTED;
    if ((int64_t)256 * (d > ffn + 63 ? d : ffn + 63) >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;  // 32-bit tile offsets
    if (dtype == MOE_DTYPE_BF16 && rows_in * (int64_t)d >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;  // 32-bit row offsets
    if (!seg_offsets || !slot_expert || !packed || !workspace) return MOE_ERR_INVALID_ARG;
    if (A > 0 && (!x_in || !y_perm)) return MOE_ERR_INVALID_ARG;
    if ((scale != nullptr) != (scale_idx != nullptr)) return MOE_ERR_INVALID_ARG;
    FfnWs ws;
    const size_t need = ffn_ws_layout(A, d, ffn, nseg, dtype, opt.split, (char*)workspace, &ws);
    if (workspace_bytes < need) return MOE_ERR_WORKSPACE_TOO_SMALL;
    if (A == 0 || seg_begin == seg_end) {
        if (job_out) *job_out = TableJob{};
        return MOE_OK;
    }
    hipStream_t st = (hipStream_t)stream;
    const size_t per = (size_t)E * d * ffn;
    const int nrange = seg_end - seg_begin;
    // one position of the row list per thread up to 256 workgroups
    const int build_grid = (int)(A <= 1024 ? 2 : (A > 255 * 1024 ? 256 : ceil_div64(A, 1024) + 1));
    int rc;
    // the table builder's turn; false: the call ends here
    auto tables = [&](const TableJob& job, int* rc_out) {
        *rc_out = MOE_OK;
        if (stage == kFfnJobOnly) {
            *job_out = job;
            return false;
        }
        if (stage == kFfnTablesBuilt) return true;
        hipLaunchKernelGGL(build_tables_kernel, dim3(build_grid), dim3(1024), 0, st, seg_offsets, slot_expert, job);
        *rc_out = check_launch();
        return *rc_out == MOE_OK;
    };
    // Forms of the first product's kernels, and how they find their rows: the streaming ones, with a handful of rows to an
    // M-tile, look a gathered row up twice (a list of tokens costs the workgroup that builds the tables a memory round trip, one token
    // on 128 experts 75.9 -> 76.7 us), the others once (16384 tokens on 64 experts of 768 x 3072 119 -> 113, the product alone).
    const int fp = padded_ffn(ffn, dtype);  // hidden width the kernels see
    const int n1 = relu ? 1 : 2;            // matrices in the first product
    const int s1 = dtype == MOE_DTYPE_F32 ? 0 : stream_form(opt.stream, opt.tile1, A, E, n1 * fp, d / kPackK);
    const int s2 = dtype == MOE_DTYPE_F32 || opt.split == 1 ? 0 : stream_form(opt.stream, opt.tile2, A, E, d, fp / kPackK);
    if (s1) tokens = nullptr;
    const RowMap rm1 = tokens ? RowMap{tokens, nullptr, 1, nullptr, nullptr, nullptr}
                              : RowMap{ws.rowlist, gather_rows, gather_div, nullptr, nullptr, nullptr};
    const RowMap rm2{nullptr, nullptr, 1, ws.rowlist, scale_idx, scale};
    const RowLists lists{ws.rowlist, tokens, gather_rows, gather_div};

    if (dtype == MOE_DTYPE_F32) {
        // 32-row tiles until 64-row ones would go twice round the CUs for the wider product
        const int64_t tiles64 = (ceil_div64(A, 64) + E) * ceil_div(ffn > d ? ffn : d, 64);
        const int bm = tiles64 < 2 * kGemmGrid ? 32 : 64;
        TableSpec t1{ws.tiles1, ws.counts, nullptr, bm, ws.capacity, 0, 0, 1, 0, 0};
        TableSpec none{};
        if (!tables(TableJob{E, seg_begin, seg_end, t1, none, lists, nullptr, 0, nullptr}, &rc)) return rc;
        const float* w1 = (const float*)packed;
        const float* w3 = w1 + per;
        const float* w2 = relu ? w3 : w3 + per;
        const int grid = 4 * num_cus();
        auto go = [&](auto kern, const float* X, int lda, const float* b1, const float* b3, float* Cp, int ldc, int N,
                      int K, const RowMap& rm, int is_relu, RowCopy cp) {
            const int all = grid + copy_blocks(cp, 256);
            hipLaunchKernelGGL(kern, dim3(all), dim3(256), 0, st, X, lda, b1, b3, (size_t)d * ffn, Cp, ldc, ws.tiles1,
                               ws.counts, N, K, rm, is_relu, grid, cp);
            return check_launch();
        };
        const bool low = bm == 32;
        if (relu)
            rc = go(low ? grouped_gemm_f32_kernel<2, false> : grouped_gemm_f32_kernel<4, false>, (const float*)x_in, d,
                    w1, nullptr, (float*)ws.h, ffn, ffn, d, rm1, 1, copy);
        else
            rc = go(low ? grouped_gemm_f32_kernel<2, true> : grouped_gemm_f32_kernel<4, true>, (const float*)x_in, d,
                    w1, w3, (float*)ws.h, ffn, ffn, d, rm1, 0, copy);
        if (rc != MOE_OK) return rc;
        return go(low ? grouped_gemm_f32_kernel<2, false> : grouped_gemm_f32_kernel<4, false>, (const float*)ws.h, ffn,
                  w2, nullptr, (float*)y_perm, d, d, ffn, rm2, 0, RowCopy{});
    }

    // Batches of a few rows per expert stream their weights; for the rest the table builder chooses the height of
    // the tiles.
    const int v1 = opt.tile1, v2 = opt.tile2;
    // N-tiles walked side by side over the M-tiles of an expert: see the tile order in ffn_tiles.h
    const int group_n = opt.group_n > 0 ? opt.group_n : kTileGroup;
    // one launch builds the row list and both tables; the second product shares the first one's
    // table when it has the same tile height and splits nothing
    const int bm1 = s1 ? kStreamBM : v1 >= 0 ? kShapeRows[v1] : 0;  // 0: the table builder chooses
    const int bm2 = s2 ? kStreamBM : v2 >= 0 ? kShapeRows[v2] : 0;
    // Both products in one launch: of the whole slot range, with nothing forced.  Where a product is to be timed, or walks its
    // tiles as an option says, they are a launch each all the same, with the same bits: no tile of a batch of such a size is split,
    // the second product's end is the launch's only one (split by the rule, whole steps: 64 experts of 2048 x 1408, 1000 / 4096
    // tokens 264 -> 268 / 532 -> 546 us).  What the second product waits for lies behind the first table's tiles, of which there
    // are less than there is room for.
    const int64_t spare = ws.capacity - (ceil_div64(A, kMinAutoHeight) + (A < nseg ? A : nseg));
    const int left_room = ceil_div(E * (int)sizeof(int32_t), (int)sizeof(MTile));
    const bool linked = !s1 && !s2 && v1 < 0 && v2 < 0 && opt.split <= 0 && nrange == nseg && spare >= left_room &&
                        one_launch(A, E, ceil_div(n1 * fp, kPackN), d / kPackK, fp / kPackK);
    // The same where the result lies on what the first product reads or copies (in place, for one): it is written while that goes on.
    const size_t row_bytes = (size_t)d * sizeof(bf16_t), result = (size_t)A * row_bytes;
    const bool in_place = share_bytes(y_perm, result, x_in, (size_t)rows_in * row_bytes) ||
                          (copy.x_perm && share_bytes(y_perm, result, copy.x_perm, result)) ||
                          (gather_rows && share_bytes(y_perm, result, gather_rows, (size_t)A * sizeof(int32_t)));
    // And where hidden rows share cache lines (they are multiples of 128 bytes, from the scratch's own address on, of which the ABI
    // asks 16 bytes of alignment): a line read for a complete row would be kept with what its neighbour held before.
    const bool own_lines = (uintptr_t)ws.h % kCacheLine == 0;
    static_assert(kPackK * sizeof(bf16_t) % kCacheLine == 0, "a hidden row is whole lines");
    const bool both = linked && !armed && opt.group_n == 0 && !in_place && own_lines;
    // (the first table ends where the counts begin, whatever the offsets say: one that does not fit is none, and nobody waits for it)
    const int room1 = both ? ws.capacity - left_room : ws.capacity;
    int32_t* const left = both ? (int32_t*)(ws.tiles1 + room1) : nullptr;
    const bool split = ws.split_capacity > 0 && !s2 && !linked;
    const bool own2 = bm2 != bm1 || bm2 == 0 || split;
    TableSpec t1{ws.tiles1, ws.counts, nullptr, bm1, room1, d / kPackK, 0,
                 ceil_div(n1 * fp, kPackN), 0, 0};
    TableSpec t2{own2 ? ws.tiles2 : nullptr, ws.counts + kCntStride, ws.splits, bm2, ws.capacity, fp / kPackK,
                 split ? ws.parts : 0, ceil_div(d, kPackN), ws.split_all, ws.split_capacity};
    if (!tables(TableJob{E, seg_begin, seg_end, t1, t2, lists, ws.queues, 16, left}, &rc)) return rc;
    const MTile* tiles2 = own2 ? ws.tiles2 : ws.tiles1;
    const int32_t* count2 = own2 ? ws.counts + kCntStride : ws.counts;
    const bf16_t* p13 = (const bf16_t*)packed;
    const bf16_t* p2 = p13 + (size_t)E * packed_elems1(n1, d, fp);
    if (timed) (void)hipEventRecord(g_time_events[0], st);
    if (left) {
        const auto go = relu ? launch_both<kEpiRelu> : launch_both<kEpiSwiglu>;
        rc = go((const bf16_t*)x_in, d, p13, packed_elems1(n1, d, fp), p2, packed_elems2(d, fp), E, ws, fp, (bf16_t*)y_perm,
                tiles2, count2, rm1, rm2, copy, left, st);
    } else if (s1) {
        rc = relu ? launch_stream<kEpiRelu>(s1, A, E, (const bf16_t*)x_in, d, p13, packed_elems1(n1, d, fp), (bf16_t*)ws.h,
                                            fp, ws.tiles1, ws.counts, n1 * fp, d, rm1, copy, st)
                  : launch_stream<kEpiSwiglu>(s1, A, E, (const bf16_t*)x_in, d, p13, packed_elems1(n1, d, fp),
                                              (bf16_t*)ws.h, fp, ws.tiles1, ws.counts, n1 * fp, d, rm1, copy, st);
    } else {
        const auto go = relu ? launch_tiles<kEpiRelu> : launch_tiles<kEpiSwiglu>;
        rc = go((const bf16_t*)x_in, d, p13, packed_elems1(n1, d, fp), E, (bf16_t*)ws.h, fp, ws.tiles1, ws.counts, ws.queues,
                n1 * fp, d, group_n, rm1, nullptr, copy, st);
    }
    if (timed) (void)hipEventRecord(g_time_events[1], st);
    if (rc != MOE_OK) return rc;
    if (timed) (void)hipEventRecord(g_time_events[2], st);
    if (s2)
        rc = launch_stream<kEpiNone>(s2, A, E, (const bf16_t*)ws.h, fp, p2, packed_elems2(d, fp), (bf16_t*)y_perm, d,
                                     tiles2, count2, d, fp, rm2, RowCopy{}, st);
    else if (!left)
        rc = launch_tiles<kEpiNone>((const bf16_t*)ws.h, fp, p2, packed_elems2(d, fp), E, (bf16_t*)y_perm, d, tiles2, count2,
                                    ws.queues + 8, d, fp, group_n, rm2, ws.partials, RowCopy{}, st);
    if (rc == MOE_OK && split) {
        hipLaunchKernelGGL(add_partials_kernel, dim3(ws.split_capacity < 64 ? ws.split_capacity : 64, 32), dim3(256),
                           0, st, ws.partials, ws.splits, count2, ws.parts, (bf16_t*)y_perm, d, d, rm2);
        rc = check_launch();
    }
    if (timed) (void)hipEventRecord(g_time_events[3], st);
    return rc;
}
}  // namespace moegps

extern "C" int moe_grouped_ffn(const void* x_perm, int dtype, int64_t A, int d, int ffn, int E,
                               const int32_t* seg_offsets, const int32_t* slot_expert, int nseg, int seg_begin,
                               int seg_end, const void* packed, void* y_perm, void* workspace,
                               size_t workspace_bytes, void* stream) {
    return moegps::grouped_ffn_call(0, x_perm, A, nullptr, 1, nullptr, nullptr, dtype, A, d, ffn, E, seg_offsets,
                                    slot_expert, nseg, seg_begin, seg_end, packed, y_perm, workspace, workspace_bytes,
                                    stream, moegps::ffn_options());
}

extern "C" int moe_grouped_ffn_relu(const void* x_perm, int dtype, int64_t A, int d, int ffn, int E,
                                    const int32_t* seg_offsets, const int32_t* slot_expert, int nseg, int seg_begin,
                                    int seg_end, const void* packed, void* y_perm, void* workspace,
                                    size_t workspace_bytes, void* stream) {
    return moegps::grouped_ffn_call(1, x_perm, A, nullptr, 1, nullptr, nullptr, dtype, A, d, ffn, E, seg_offsets,
                                    slot_expert, nseg, seg_begin, seg_end, packed, y_perm, workspace, workspace_bytes,
                                    stream, moegps::ffn_options());
}

extern "C" int moe_grouped_ffn_fused(const void* x, int dtype, int T, int k, const int32_t* assign_of_row,
                                     const float* topk_w, int d, int ffn, int E, const int32_t* seg_offsets,
                                     const int32_t* slot_expert, int nseg, int seg_begin, int seg_end,
                                     const void* packed, void* y_perm, void* workspace, size_t workspace_bytes,
                                     void* stream) {
    if (T < 0 || k < 1 || d < 1) return MOE_ERR_INVALID_ARG;
    if ((int64_t)T * d >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;  // 32-bit element offsets into x
    if (T > 0 && !assign_of_row) return MOE_ERR_INVALID_ARG;
    return moegps::grouped_ffn_call(0, x, T, assign_of_row, k, topk_w ? assign_of_row : nullptr, topk_w, dtype,
                                    (int64_t)T * k, d, ffn, E, seg_offsets, slot_expert, nseg, seg_begin, seg_end,
                                    packed, y_perm, workspace, workspace_bytes, stream, moegps::ffn_options());
}

extern "C" int moe_grouped_ffn_gather(const void* x, int dtype, int T, int k, const int32_t* assign_of_row, int d,
                                      int ffn, int E, const int32_t* seg_offsets, const int32_t* slot_expert,
                                      int nseg, int seg_begin, int seg_end, const void* packed, void* y_perm,
                                      void* workspace, size_t workspace_bytes, void* stream) {
    return moe_grouped_ffn_fused(x, dtype, T, k, assign_of_row, nullptr, d, ffn, E, seg_offsets, slot_expert, nseg,
                                 seg_begin, seg_end, packed, y_perm, workspace, workspace_bytes, stream);
}

extern "C" int moe_grouped_ffn_time_next_call(void* const* events) {
    using namespace moegps;
    if (!events) {
        g_time_armed = false;
        return MOE_OK;
    }
    for (int i = 0; i < 4; ++i) {
        if (!events[i]) return MOE_ERR_INVALID_ARG;
        g_time_events[i] = (hipEvent_t)events[i];
    }
    g_time_armed = true;
    return MOE_OK;
}
