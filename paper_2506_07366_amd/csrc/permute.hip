// Dispatch of assignments to replica segments and the token permutation: the
// dispatch d of Algorithm 1 for a given plan, standing where the all-to-all
// before the expert FFN is (Background, paragraph on the communication cost of
// routing).
//
// Everything is a deterministic stable counting sort, built from one primitive:
// the stable rank of an element among equal keys.  A workgroup owns a contiguous
// chunk of tokens; inside the chunk ranks come from wavefront ballots, across
// chunks from an exclusive scan of per-chunk key counts.  No atomics decide any
// position, so the permutation is identical for every launch.
//
//   count    : per-chunk histogram of the dispatch keys (expert ids); further workgroups of the
//              same launch turn the plan into per-expert replica tables
//   segment  : stable rank -> replica -> segment id; per-chunk segment histogram
//   place    : seg_offsets, rank_load, row_of_assign / assign_of_row
//   scatter  : each token row is read once and written to its k rows of x_perm (a whole step leaves that to
//              the launch of the first FFN product, row_copy.h)
//
// These kernels are bound by latency, each costs 4-5 us whatever it does, so a workgroup of
// "segment" and "place" adds up the counts of the chunks before its own by itself (a few hundred
// coalesced loads, served by the L2) and the scans are no launches of their own; and the chunks
// are cut small enough that a workgroup ranks 256 elements at a time in one or two rounds.  Only above
// kSelfScanChunks chunks, where every workgroup would read megabytes, two scan kernels turn the
// counts into bases first.  Index kernels against chunks of 2048 and always the scans (whole
// moe_permute without the row copy, modes 1 / 2):
//   12288 assignments,  64 experts, 80 slots    32.8 / 38.6 -> 14.5 / 14.9 us
//   98304               64          80          34.9 / 40.6 -> 22.4 / 24.5
//   262144              128         160         57.0 / 64.7 -> 40.0 / 47.4
//   65536               128         160         38.2 / 45.7 -> 27.1 / 28.6
//
// A batch of a few thousand assignments (decode, short prompts) takes the index steps in one
// workgroup and one launch: the same ranks and scans, the chunk being the whole batch (one_workgroup_limit).
#include "permute.h"
#include "block_scan.h"
#include "row_copy.h"
#include <initializer_list>
#include <mutex>

namespace moegps {

constexpr int kPermThreads = 256;
constexpr int kPermWaves = kPermThreads / kWave;
constexpr int kRounds = 8;                                  // max 64-element rounds per wavefront
constexpr int kChunk = kPermThreads * kRounds;              // max elements per workgroup (2048)
constexpr int kMaxKeys = MOE_MAX_SEGMENTS;                  // >= MOE_MAX_EXPERTS
constexpr int kChunksWanted = 128;                          // chunks a batch is cut into while rounds are left to give
constexpr int kSelfScanChunks = 256;

__host__ __device__ inline int tokens_per_chunk(int k, int rounds) {
    return kPermThreads * rounds / k > 0 ? kPermThreads * rounds / k : 1;
}

struct PermWs {
    int32_t* bh1;       // [nb, E]    per-chunk expert counts (-> chunk bases)
    int32_t* bh2;       // [nb, NSEG] per-chunk segment counts (-> chunk bases)
    uint16_t* seg;      // [A]        segment of each assignment
    int32_t* rep_cnt;   // [E]        replicas per expert (0 = everything to the home slot)
    int32_t* rep_slot;  // [E, G]     replica slots, ascending
    int32_t* rep_hi;    // [E, G]     exclusive upper bound of each replica's rank range
    int rounds;         // rounds per chunk
    int nb;             // chunks
};
static_assert(MOE_MAX_SEGMENTS <= (1 << 16), "segment ids are kept in 16 bits");

// Bytes of scratch of a batch.  (The figure is a fixed function of the sizes: chunks of 2048 with
// 4-byte segment ids.  The layout below keeps inside it, so callers that sized their scratch once,
// and the fixed array of moe_permute_static, serve the same batches at any chunk size.)
static size_t perm_ws_bytes(int T, int E, int k, int G, int S) {
    const int nb = ceil_div(T > 0 ? T : 1, tokens_per_chunk(k, kRounds));
    size_t off = 0;
    for (const size_t n : {(size_t)nb * E, (size_t)nb * G * S, (size_t)T * k, (size_t)E, (size_t)E * G, (size_t)E * G})
        off += align_up(n * sizeof(int32_t), 256);
    return off;
}

static PermWs perm_ws_layout(int T, int E, int k, int G, int S, char* base) {
    const size_t have = perm_ws_bytes(T, E, k, G, S);
    const int64_t A = (int64_t)T * k;
    PermWs w;
    int64_t want = ceil_div64(A, (int64_t)kPermThreads * kChunksWanted);
    for (w.rounds = (int)(want < 1 ? 1 : (want > kRounds ? kRounds : want));; ++w.rounds) {
        w.nb = T > 0 ? ceil_div(T, tokens_per_chunk(k, w.rounds)) : 0;
        size_t off = 0;
        auto take = [&](size_t bytes) {
            char* p = base ? base + off : nullptr;
            off += align_up(bytes, 256);
            return p;
        };
        w.bh1 = (int32_t*)take((size_t)w.nb * E * 4);
        w.bh2 = (int32_t*)take((size_t)w.nb * G * S * 4);
        w.seg = (uint16_t*)take((size_t)A * 2);
        w.rep_cnt = (int32_t*)take((size_t)E * 4);
        w.rep_slot = (int32_t*)take((size_t)E * G * 4);
        w.rep_hi = (int32_t*)take((size_t)E * G * 4);
        if (off <= have || w.rounds == kRounds) return w;
    }
}

// more chunks than the workgroups add up by themselves
static inline bool perm_scanned(const PermWs& ws) {
    return ws.nb == 0 || (ws.nb > kSelfScanChunks && ws.rounds == kRounds);
}

__device__ __forceinline__ int clamp_key(int v, int n) { return v < 0 ? 0 : (v >= n ? n - 1 : v); }

__device__ __forceinline__ int home_slot_of(int e, int H, int S) { return (e / H) * S + (e % H); }

// ---------------------------------------------------------------------------
// Stable rank of every element of a chunk among equal keys earlier in the chunk.
// Wavefront w owns `rounds` <= NR rounds of 64 elements; element p of the chunk is (w, r, lane)
// with p = (w * rounds + r) * 64 + lane.
// The workgroup has NWAVES wavefronts; wcnt is LDS scratch of NWAVES*nkeys ints.
// On return rank[r] holds the rank, and (if chunk_hist) chunk_hist[key] the chunk's
// count per key.  Only the first `rounds` rounds hold elements (uniform over the workgroup).
// ---------------------------------------------------------------------------
template <int NWAVES, int NR>
__device__ void chunk_stable_rank(const int (&key)[NR], const bool (&valid)[NR], int nkeys, int* wcnt, int (&rank)[NR],
                                  int32_t* chunk_hist, int rounds = NR) {
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = tid / kWave;
    for (int i = tid; i < NWAVES * nkeys; i += NWAVES * kWave) wcnt[i] = 0;
    __syncthreads();
    int nbits = 1;
    while ((1 << nbits) < nkeys) ++nbits;
    const unsigned long long lt = (1ull << lane) - 1ull;
    int* mine = wcnt + w * nkeys;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        rank[r] = 0;
        if (r >= rounds) continue;
        // lanes of this round holding the same key
        unsigned long long same = __ballot(valid[r]);
        for (int b = 0; b < nbits; ++b) {
            const bool bit = (key[r] >> b) & 1;
            const unsigned long long m = __ballot(valid[r] && bit);
            same &= bit ? m : ~m;
        }
        if (valid[r]) {
            const int prior = mine[key[r]];
            rank[r] = prior + __popcll(same & lt);
            if ((same & lt) == 0ull) mine[key[r]] = prior + __popcll(same);  // leader
        }
    }
    __syncthreads();
    // exclusive prefix over the wavefronts, per key
    for (int kk = tid; kk < nkeys; kk += NWAVES * kWave) {
        int c[NWAVES];  // all reads, then all writes: the reads overlap
#pragma unroll
        for (int ww = 0; ww < NWAVES; ++ww) c[ww] = wcnt[ww * nkeys + kk];
        int run = 0;
#pragma unroll
        for (int ww = 0; ww < NWAVES; ++ww) {
            wcnt[ww * nkeys + kk] = run;
            run += c[ww];
        }
        if (chunk_hist) chunk_hist[kk] = run;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (r < rounds && valid[r]) rank[r] += mine[key[r]];
}

// inclusive prefix sum over the 64 lanes of a wavefront (every lane active)
__device__ __forceinline__ long long wave_incl_scan(long long v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        const long long o = __shfl_up(v, m, kWave);
        if (lane >= m) v += o;
    }
    return v;
}

// inclusive prefix sum of 32-bit counts over the 64 lanes of a wavefront
__device__ __forceinline__ int wave_incl_scan_i32(int v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        const int o = __shfl_up(v, m, kWave);
        if (lane >= m) v += o;
    }
    return v;
}

// In-place exclusive scan down NC neighbouring columns (col0 .. col0 + NC - 1, those
// below ncols) of a [nb, ncols] table by one wavefront: lanes take consecutive rows, the
// NC loads of a step are independent and go out together.  total[i] = column sums.
template <int NC>
__device__ __forceinline__ void wave_columns_scan(int32_t* table, int nb, int ncols, int col0, int total[NC]) {
    const int lane = threadIdx.x & (kWave - 1);
    int carry[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) carry[i] = 0;
    for (int b0 = 0; b0 < nb; b0 += kWave) {
        const int b = b0 + lane;
        int c[NC], incl[NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) c[i] = (b < nb && col0 + i < ncols) ? table[(size_t)b * ncols + col0 + i] : 0;
#pragma unroll
        for (int i = 0; i < NC; ++i) incl[i] = wave_incl_scan_i32(c[i]);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            if (b < nb && col0 + i < ncols) table[(size_t)b * ncols + col0 + i] = carry[i] + incl[i] - c[i];
            carry[i] += __shfl(incl[i], kWave - 1, kWave);
        }
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) total[i] = carry[i];
}

// Replicas of expert e in ascending slot id with the exclusive upper bound of each
// replica's range of ranks, by one wavefront (every lane active).  In mode 1 without hist_true (a whole step, whose
// histogram is being counted by the same launch) the bound is the quota up to the replica, for segment_of to scale.
__device__ __forceinline__ void replica_table(int e, int mode, int G, int nseg, const int32_t* __restrict__ hist_true,
                                              const int32_t* __restrict__ hist_pred,
                                              const int32_t* __restrict__ slot_expert,
                                              const int32_t* __restrict__ slot_quota, const PermWs& ws) {
    const int lane = threadIdx.x & (kWave - 1);
    const unsigned long long lt = (1ull << lane) - 1ull;
    long long n_true = 0, n_hat = 0;
    if (mode == MOE_MODE_DISTRIBUTION) {
        if (hist_true) n_true = hist_true[e];
        n_hat = hist_pred[e];
    }
    int cnt = 0;
    long long cum = 0;
    if (!(mode == MOE_MODE_DISTRIBUTION && n_hat <= 0)) {
        for (int s0 = 0; s0 < nseg; s0 += kWave) {
            const int sigma = s0 + lane;
            const bool match = sigma < nseg && slot_expert[sigma] == e;
            const long long qv = match ? (long long)slot_quota[sigma] : 0ll;
            const long long incl = wave_incl_scan(qv);
            const unsigned long long m = __ballot(match);
            const int pos = cnt + __popcll(m & lt);
            if (match && pos < G) {
                long long hi = cum + incl;                                       // Q_{r+1}
                if (mode == MOE_MODE_DISTRIBUTION && hist_true) hi = (n_true * hi) / n_hat;  // floor(n_e * Q / nhat_e)
                if (hi > 0x7fffffffLL) hi = 0x7fffffffLL;
                ws.rep_slot[(size_t)e * G + pos] = sigma;
                ws.rep_hi[(size_t)e * G + pos] = (int)hi;
            }
            cnt += __popcll(m);
            cum += __shfl(incl, kWave - 1, kWave);
        }
    }
    if (lane == 0) ws.rep_cnt[e] = cnt < G ? cnt : G;
}

// per-chunk histogram of the dispatch keys (workgroups below ws.nb) and the replica tables of the
// plan (the workgroups above, one wavefront per expert); the histogram of the keys is added to hist_out, if
// there is one (ids of no expert are ranked as the nearest one and counted for none)
__global__ __launch_bounds__(kPermThreads) void perm_count_kernel(const int32_t* __restrict__ keys, int mode, int T,
                                                                   int k, int E, int G, int S,
                                                                   const int32_t* __restrict__ hist_true,
                                                                   const int32_t* __restrict__ hist_pred,
                                                                   const int32_t* __restrict__ slot_expert,
                                                                   const int32_t* __restrict__ slot_quota, PermWs ws,
                                                                   int32_t* __restrict__ hist_out) {
    __shared__ int bins[MOE_MAX_EXPERTS];
    __shared__ int strays[2];  // ids below 0, from E on
    if ((int)blockIdx.x >= ws.nb) {
        const int e = ((int)blockIdx.x - ws.nb) * kPermWaves + (int)threadIdx.x / kWave;
        if (e < E) replica_table(e, mode, G, G * S, hist_true, hist_pred, slot_expert, slot_quota, ws);
        return;
    }
    const int tpc = tokens_per_chunk(k, ws.rounds);
    const int64_t lo = (int64_t)blockIdx.x * tpc * k;
    const int64_t A = (int64_t)T * k;
    const int64_t hi = lo + (int64_t)tpc * k < A ? lo + (int64_t)tpc * k : A;
    for (int e = threadIdx.x; e < E; e += blockDim.x) bins[e] = 0;
    if (threadIdx.x < 2) strays[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
        const int id = keys[i];
        atomicAdd(&bins[clamp_key(id, E)], 1);
        if ((unsigned)id >= (unsigned)E) atomicAdd(&strays[id < 0 ? 0 : 1], 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const int n = bins[e];
        ws.bh1[(size_t)blockIdx.x * E + e] = n;
        const int counted = n - (e == 0 ? strays[0] : 0) - (e == E - 1 ? strays[1] : 0);
        if (hist_out && counted != 0) atomicAdd(&hist_out[e], counted);
    }
}

// chunk bases per expert (in place), one wavefront per expert column, columns dealt over the whole grid
constexpr int kScan1Threads = 256;
__global__ __launch_bounds__(kScan1Threads) void perm_scan1_kernel(int E, PermWs ws) {
    const int wave = threadIdx.x / kWave, nwaves = blockDim.x / kWave;
    for (int e = blockIdx.x * nwaves + wave; e < E; e += gridDim.x * nwaves) {
        int unused[1];
        wave_columns_scan<1>(ws.bh1, ws.nb, E, e, unused);
    }
}

// Sums down the columns of a [nb, ncols] table of counts by the whole workgroup: base[c] over the
// rows below `upto`, and, where total is given, total[c] over all rows (both in LDS, ncols ints).
// Threads lie side by side along a row; several groups of them share the rows.
__device__ __forceinline__ void block_column_sums(const int32_t* __restrict__ table, int nb, int ncols, int upto,
                                                  int* base, int* total) {
    const int tid = threadIdx.x;
    for (int c = tid; c < ncols; c += kPermThreads) {
        base[c] = 0;
        if (total) total[c] = 0;
    }
    __syncthreads();
    int width = kWave;
    while (width < ncols && width < kPermThreads) width <<= 1;
    const int groups = kPermThreads / width, grp = tid / width;
    const int rows = total ? nb : upto;
    constexpr int U = 8;  // loads in flight per thread
    for (int c = tid % width; c < ncols; c += width) {
        int below = 0, all = 0;
        for (int b0 = grp; b0 < rows; b0 += groups * U) {
            int v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int b = b0 + u * groups;
                v[u] = b < rows ? table[(size_t)b * ncols + c] : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                all += v[u];
                below += b0 + u * groups < upto ? v[u] : 0;
            }
        }
        if (below) atomicAdd(&base[c], below);
        if (total && all) atomicAdd(&total[c], all);
    }
    __syncthreads();
}

// Segment of an assignment to expert e that stands at place i of the plan's order for e
// (i < 0: the assignment is outside the plan's order and goes to the home slot).
// With hist_true the replicas' bounds are quotas Q of the predicted n_hat, and i is past floor(n Q / n_hat) exactly
// if (i + 1) n_hat > n Q.
__device__ __forceinline__ int segment_of(int e, int i, int H, int S, int G, const PermWs& ws,
                                          const int32_t* __restrict__ hist_true, const int32_t* __restrict__ hist_pred) {
    int sg = home_slot_of(e, H, S);
    if (i < 0) return sg;
    const int cnt = ws.rep_cnt[e];
    if (cnt > 0) {
        int rr = 0;
        if (hist_true) {
            const long long n = hist_true[e], past = (i + 1ll) * hist_pred[e];
            while (rr < cnt - 1 && past > n * ws.rep_hi[(size_t)e * G + rr]) ++rr;
        } else {
            while (rr < cnt - 1 && i >= ws.rep_hi[(size_t)e * G + rr]) ++rr;
        }
        sg = ws.rep_slot[(size_t)e * G + rr];
    }
    return sg;
}

// segment id per assignment + per-chunk segment histogram.  SCANNED: ws.bh1 holds chunk bases, else counts.
// In a whole step hist_true and hist_pred scale the replicas' bounds (mode 1), and in the modes whose count launch does not
// see topk_idx its histogram is added to hist_out here.
template <bool SCANNED>
__global__ __launch_bounds__(kPermThreads) void perm_segment_kernel(int mode, int T, int k, int E, int G, int S,
                                                                     const int32_t* __restrict__ topk_idx,
                                                                     const int32_t* __restrict__ pred_idx,
                                                                     PermWs ws, const int32_t* __restrict__ hist_true,
                                                                     const int32_t* __restrict__ hist_pred,
                                                                     int32_t* __restrict__ hist_out) {
    __shared__ int wcnt[kPermWaves * MOE_MAX_EXPERTS];
    __shared__ int prank[kChunk];
    __shared__ int seg_bins[MOE_MAX_SEGMENTS];
    __shared__ int ebase[MOE_MAX_EXPERTS];  // (its second life: counts for hist_out)
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = tid / kWave;
    const int nseg = G * S;
    const int H = (E + G - 1) / G;
    // (more than kSelfScanChunks chunks are always chunks of kRounds: fixed loops, 5 % of the index steps
    // of 600000 assignments to 8 experts)
    const int rounds = SCANNED ? kRounds : ws.rounds;
    const int tpc = tokens_per_chunk(k, rounds);
    const int64_t A = (int64_t)T * k;
    const int64_t base = (int64_t)blockIdx.x * tpc * k;
    const int n_b = (int)((base + (int64_t)tpc * k < A ? base + (int64_t)tpc * k : A) - base);

    for (int s = tid; s < nseg; s += kPermThreads) seg_bins[s] = 0;

    int key[kRounds], rank[kRounds];
    bool valid[kRounds];
    const int32_t* rank_keys = (mode == MOE_MODE_TOKEN) ? pred_idx : topk_idx;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int p = (w * rounds + r) * kWave + lane;
        valid[r] = r < rounds && p < n_b;
        key[r] = valid[r] ? clamp_key(rank_keys[base + p], E) : 0;
        rank[r] = 0;
    }
    if (mode != MOE_MODE_NONE) {
        if (!SCANNED) block_column_sums(ws.bh1, ws.nb, E, blockIdx.x, ebase, nullptr);
        chunk_stable_rank<kPermWaves, kRounds>(key, valid, E, wcnt, rank, nullptr, rounds);
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int p = (w * rounds + r) * kWave + lane;
            if (valid[r]) prank[p] = (SCANNED ? ws.bh1[(size_t)blockIdx.x * E + key[r]] : ebase[key[r]]) + rank[r];
        }
    }
    __syncthreads();
    if (hist_out) {
        for (int e = tid; e < E; e += kPermThreads) ebase[e] = 0;
        __syncthreads();
    }

#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int p = (w * rounds + r) * kWave + lane;
        if (!valid[r]) continue;
        const int id = topk_idx[base + p], e = clamp_key(id, E);
        if (hist_out && id == e) atomicAdd(&ebase[e], 1);
        int i = -1;  // place of this assignment in the plan's order for expert e
        if (mode == MOE_MODE_DISTRIBUTION) {
            i = prank[p];
        } else if (mode == MOE_MODE_TOKEN) {
            const int row0 = (p / k) * k;  // the token's predicted ids
            for (int jp = 0; jp < k; ++jp) {
                if (clamp_key(pred_idx[base + row0 + jp], E) == e) {
                    i = prank[row0 + jp];
                    break;
                }
            }
        }
        const int sg = segment_of(e, i, H, S, G, ws, hist_true, hist_pred);
        ws.seg[base + p] = (uint16_t)sg;
        atomicAdd(&seg_bins[sg], 1);
    }
    __syncthreads();
    for (int s = tid; s < nseg; s += kPermThreads) ws.bh2[(size_t)blockIdx.x * nseg + s] = seg_bins[s];
    if (hist_out)
        for (int e = tid; e < E; e += kPermThreads)
            if (ebase[e] > 0) atomicAdd(&hist_out[e], ebase[e]);
}

// chunk bases per segment (in place), seg_offsets, rank_load
__global__ __launch_bounds__(1024) void perm_scan2_kernel(int G, int S, PermWs ws, int32_t* __restrict__ seg_offsets,
                                                           int32_t* __restrict__ rank_load) {
    __shared__ int tot[MOE_MAX_SEGMENTS + 1];
    __shared__ int wave_sum[16];
    const int nseg = G * S;
    const int tid = threadIdx.x;
    const int wave = tid / kWave, nwaves = blockDim.x / kWave;
    constexpr int NC = 4;  // neighbouring segment columns one wavefront scans together
    for (int s0 = wave * NC; s0 < nseg; s0 += nwaves * NC) {
        int total[NC];
        wave_columns_scan<NC>(ws.bh2, ws.nb, nseg, s0, total);
        if ((tid & (kWave - 1)) == 0) {
#pragma unroll
            for (int i = 0; i < NC; ++i)
                if (s0 + i < nseg) tot[s0 + i] = total[i];
        }
    }
    __syncthreads();
    block_exclusive_scan_2048(tot, nseg, wave_sum);
    for (int s = tid; s <= nseg; s += blockDim.x) seg_offsets[s] = tot[s];
    for (int g = tid; g < G; g += blockDim.x) rank_load[g] = tot[(g + 1) * S] - tot[g * S];
}

// The plan of mode 0, the home placement with the batch's own counts, by a workgroup.
__device__ __forceinline__ void home_plan(const HomePlan& home, const int32_t* hist, int E, int G, int S) {
    const int H = ceil_div(E, G), tid = threadIdx.x, n = blockDim.x;
    for (int s = tid; s < G * S; s += n) {
        const int j = s % S, e = s / S * H + j;
        const bool held = j < H && e < E;
        home.slot_expert[s] = held ? e : -1;
        home.slot_quota[s] = held ? hist[e] : 0;
    }
    for (int g = tid; g < G; g += n) {
        int load = 0;
        for (int e = g * H; e < (g + 1) * H && e < E; ++e) load += hist[e];
        home.rank_load_pred[g] = load;
    }
    if (tid == 0) home.n_iters[0] = 0;
}

// final position of every assignment.  SCANNED: ws.bh2 holds chunk bases and seg_offsets / rank_load
// are written; else ws.bh2 holds counts, every workgroup works the offsets out and the first writes them, and
// with `home` the plan of mode 0 from the histogram.
template <bool SCANNED>
__global__ __launch_bounds__(kPermThreads) void perm_place_kernel(int T, int k, int G, int S, PermWs ws,
                                                                   int32_t* __restrict__ seg_offsets,
                                                                   int32_t* __restrict__ rank_load,
                                                                   int32_t* __restrict__ row_of_assign,
                                                                   int32_t* __restrict__ assign_of_row, HomePlan home,
                                                                   const int32_t* __restrict__ hist, int E) {
    __shared__ int wcnt[kPermWaves * kMaxKeys];
    __shared__ int first[MOE_MAX_SEGMENTS];    // first row of this chunk in the segment
    __shared__ int tot[MOE_MAX_SEGMENTS + 1];  // rows per segment -> seg_offsets
    __shared__ int wave_sum[kPermWaves];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = tid / kWave;
    const int nseg = G * S;
    // (more than kSelfScanChunks chunks are always chunks of kRounds: fixed loops, 5 % of the index steps
    // of 600000 assignments to 8 experts)
    const int rounds = SCANNED ? kRounds : ws.rounds;
    const int tpc = tokens_per_chunk(k, rounds);
    const int64_t A = (int64_t)T * k;
    const int64_t base = (int64_t)blockIdx.x * tpc * k;
    const int n_b = (int)((base + (int64_t)tpc * k < A ? base + (int64_t)tpc * k : A) - base);
    int key[kRounds], rank[kRounds];
    bool valid[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int p = (w * rounds + r) * kWave + lane;
        valid[r] = r < rounds && p < n_b;
        key[r] = valid[r] ? ws.seg[base + p] : 0;
    }
    if (!SCANNED) {
        block_column_sums(ws.bh2, ws.nb, nseg, blockIdx.x, first, tot);
        // exclusive scan of tot: every thread takes `per` neighbouring segments
        const int per = ceil_div(nseg, kPermThreads);
        const int s0 = tid * per < nseg ? tid * per : nseg, s1 = s0 + per < nseg ? s0 + per : nseg;
        int mine = 0;
        for (int s = s0; s < s1; ++s) mine += tot[s];
        const int incl = wave_incl_scan_i32(mine);
        if (lane == kWave - 1) wave_sum[w] = incl;
        __syncthreads();
        int run = incl - mine;
        for (int ww = 0; ww < w; ++ww) run += wave_sum[ww];
        for (int s = s0; s < s1; ++s) {
            const int c = tot[s];
            tot[s] = run;
            first[s] += run;
            run += c;
        }
        if (s1 == nseg && s0 < s1) tot[nseg] = run;
        __syncthreads();
        if (blockIdx.x == 0) {
            for (int s = tid; s <= nseg; s += kPermThreads) seg_offsets[s] = tot[s];
            for (int g = tid; g < G; g += kPermThreads) rank_load[g] = tot[(g + 1) * S] - tot[g * S];
            if (home.slot_expert) home_plan(home, hist, E, G, S);
        }
    }
    chunk_stable_rank<kPermWaves, kRounds>(key, valid, nseg, wcnt, rank, nullptr, rounds);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int p = (w * rounds + r) * kWave + lane;
        if (!valid[r]) continue;
        const int row =
            (SCANNED ? seg_offsets[key[r]] + ws.bh2[(size_t)blockIdx.x * nseg + key[r]] : first[key[r]]) + rank[r];
        row_of_assign[base + p] = row;
        assign_of_row[row] = (int)(base + p);
    }
}

// All five index steps for a batch of at most SR * 1024 assignments, E and G*S at most
// kSmallKeys, in one workgroup of 1024 threads: the chunk is the whole batch, so the chunk
// bases are zero and both scans run in LDS.  A thread's time here goes by the number of
// instructions it runs one after the other, so the batch is dealt over all 16 wavefronts in
// as few rounds of 64 as hold it.  The replica tables live in LDS, one entry per slot: the
// upper bound of the slot's range of ranks and the next slot of the same expert (ascending
// slot id), plus every expert's first slot.  Same ranks, same results as the kernels above.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kSmallKeys = 512;
constexpr int kSmallMaxRounds = 6;

// Assignments up to which one workgroup is used (-1: never).  It pays a round for every 1024 of them,
// the three launches pay their starts and, with many experts or slots, the chunks' tables of counts:
// us for the index steps, one workgroup against three launches (two in mode 0), modes 0 / 1 / 2 (one
// workgroup past the limits: with up to eight rounds compiled in, some 0.7 us slower for that):
//   3000 assignments,   8 experts in  16 slots    6.0 / 11.2 / 13.4    7.1 / 11.7 / 11.8
//                     128             160         7.4 / 15.7 / 20.4    8.6 / 16.8 / 18.1
//                     512             512         8.2 / 19.3 / 21.4   11.9 / 23.2 / 25.6
//   3600                8              16         7.4 / 13.2 / 15.2    7.0 / 11.7 / 11.8
//   4096              512             512         9.6 / 21.7 / 24.7   12.1 / 23.4 / 25.4
//   5000              512             512        11.2 / 24.3 / 28.1   12.1 / 23.5 / 26.0
static int one_workgroup_limit(int mode, int E, int nseg) {
    if (E > kSmallKeys || nseg > kSmallKeys) return -1;
    if (E > 256 || nseg > 256) return mode == MOE_MODE_NONE ? 6 * kSmallThreads : 4 * kSmallThreads;
    return mode == MOE_MODE_TOKEN ? 2 * kSmallThreads : 3 * kSmallThreads;
}

// The per-slot tables, by one wavefront, 64 slots at a time in ascending order: the lanes
// holding one expert find each other by ballots; what earlier chunks hold for the expert
// (slots, quota, last slot) is carried in LDS.
struct SmallTables {
    int* s_e;         // [kSmallKeys] expert of the slot (-1 beyond the plan's slots)
    int* s_q;         // [kSmallKeys] its quota
    long long* s_cum; // [kSmallKeys] quota of the expert's slots up to and including this one
    int* s_next;      // [kSmallKeys] next slot of the same expert, -1: none
    int* e_first;     // [kSmallKeys] first slot of the expert, -1: home slot only
    int* e_cnt;       // [kSmallKeys] slots of the expert so far
    int* e_last;      // [kSmallKeys] the last of them
    long long* e_cum; // [kSmallKeys] their quota
};
__device__ __forceinline__ void small_slot_tables(int E, int nseg, const SmallTables& t) {
    const int lane = threadIdx.x & (kWave - 1);
    const unsigned long long bit = 1ull << lane;
    const unsigned long long lt = bit - 1ull;
    int nbits = 1;
    while ((1 << nbits) < E) ++nbits;
    for (int s0 = 0; s0 < nseg; s0 += kWave) {
        const int sigma = s0 + lane;
        const int e = sigma < nseg ? t.s_e[sigma] : -1;
        const bool ok = e >= 0 && e < E;
        const int q = ok ? t.s_q[sigma] : 0;
        unsigned long long same = __ballot(ok);
        for (int b = 0; b < nbits; ++b) {
            const bool one = (e >> b) & 1;
            const unsigned long long m = __ballot(ok && one);
            same &= one ? m : ~m;
        }
        if (!ok) same = 0ull;
        // quota of the expert's slots of this chunk up to this one: lanes take the set bits of
        // their mask one by one, as many steps as the largest group of the chunk has lanes
        long long cum = 0;
        unsigned long long todo = same & (lt | bit);
        while (__any(todo != 0ull)) {
            const int src = todo ? __ffsll((long long)todo) - 1 : lane;
            const int qs = __shfl(q, src, kWave);
            cum += todo ? (long long)qs : 0ll;
            todo &= todo - 1ull;
        }
        if (ok) {
            const int prior = t.e_cnt[e];
            const int last = t.e_last[e];
            cum += t.e_cum[e];
            const unsigned long long above = same & ~(lt | bit);
            t.s_cum[sigma] = cum;
            t.s_next[sigma] = above ? s0 + __ffsll((long long)above) - 1 : -1;
            if ((same & lt) == 0ull) {  // first lane of the expert in this chunk
                if (prior == 0) t.e_first[e] = sigma;
                else t.s_next[last] = sigma;
            }
            if (above == 0ull) {        // last lane: hand the totals on
                t.e_cnt[e] = prior + __popcll(same);
                t.e_cum[e] = cum;
                t.e_last[e] = sigma;
            }
        }
    }
}

// SR: rounds of 64 elements per wavefront, at most.  WHOLE_STEP: the histogram of topk_idx is an output (hist_out)
// and not an input, in mode 0 the home plan is too (`home`), and the workgroup goes on to build the
// tables of the grouped FFN (`job`, if it has a row list).  The counts cost next to nothing here, where the ids pass by
// anyway (as calls 4.7 us, 9.4 in mode 0), the tables their own work without another launch.
template <int SR, bool WHOLE_STEP>
__global__ __launch_bounds__(kSmallThreads) void perm_small_kernel(
    int mode, int T, int k, int E, int G, int S, const int32_t* __restrict__ topk_idx,
    const int32_t* __restrict__ pred_idx, const int32_t* __restrict__ hist_true, const int32_t* __restrict__ hist_pred,
    const int32_t* __restrict__ slot_expert, const int32_t* __restrict__ slot_quota,
    int32_t* __restrict__ seg_offsets, int32_t* __restrict__ row_of_assign, int32_t* assign_of_row,
    int32_t* __restrict__ rank_load, int32_t* __restrict__ hist_out, HomePlan home, TableJob job) {
    // one buffer, three lives: wavefront counters of the first rank; rank and key by position
    // (token-to-expert mode looks up those of the token's predicted ids); counters of the second
    __shared__ int buf[kSmallWaves * kSmallKeys];
    constexpr int kMaxA = kSmallThreads * SR;
    static_assert(SR <= kSmallMaxRounds && kSmallWaves * kSmallKeys >= kMaxA, "ranks by position share the counters' buffer");
    static_assert(kMaxA <= (1 << 16) && kSmallKeys <= (1 << 15), "rank and key share one int");
    __shared__ int s_e[kSmallKeys], s_q[kSmallKeys], s_hi[kSmallKeys], s_next[kSmallKeys];
    __shared__ int e_first[kSmallKeys], e_cnt[kSmallKeys], e_last[kSmallKeys], e_true[kSmallKeys], e_hat[kSmallKeys];
    __shared__ int e_home[kSmallKeys];  // home slot of the expert
    __shared__ long long e_cum[kSmallKeys], s_cum[kSmallKeys];
    __shared__ int tot[kSmallKeys + 1];
    __shared__ int wave_sum[16];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = tid / kWave;
    const int nseg = G * S;
    const int H = (E + G - 1) / G;
    const int n_b = T * k;
    // rounds of 64 per wavefront that hold the batch; element p is (w, r, lane) with
    // p = (w * rounds + r) * 64 + lane
    const int rounds = (n_b + kSmallThreads - 1) / kSmallThreads;

    int key[SR], rank[SR], expert[SR];
    bool valid[SR];
    unsigned no_expert = 0;  // bit r: the id of round r is outside [0, E) (NaN logits), which no histogram counts
    const int32_t* rank_keys = (mode == MOE_MODE_TOKEN) ? pred_idx : topk_idx;
#pragma unroll
    for (int r = 0; r < SR; ++r) {
        const int p = (w * rounds + r) * kWave + lane;
        valid[r] = r < rounds && p < n_b;
        const int id = valid[r] ? rank_keys[p] : 0;
        key[r] = clamp_key(id, E);
        expert[r] = key[r];
        if (WHOLE_STEP && key[r] != id) no_expert |= 1u << r;
        rank[r] = 0;
    }
    if (mode == MOE_MODE_TOKEN) {
        no_expert = 0;
#pragma unroll
        for (int r = 0; r < SR; ++r) {
            const int p = (w * rounds + r) * kWave + lane;
            const int id = valid[r] ? topk_idx[p] : 0;
            expert[r] = clamp_key(id, E);
            if (WHOLE_STEP && expert[r] != id) no_expert |= 1u << r;
        }
    }
    for (int e = tid; e < E; e += kSmallThreads) e_home[e] = home_slot_of(e, H, S);
    const bool count = WHOLE_STEP && mode != MOE_MODE_DISTRIBUTION;  // (there the ranks' counters are the histogram)
    if (count)
        for (int e = tid; e < E; e += kSmallThreads) e_true[e] = 0;
    if (mode != MOE_MODE_NONE) {
        for (int i = tid; i < kSmallKeys; i += kSmallThreads) {
            s_e[i] = i < nseg ? slot_expert[i] : -1;
            s_q[i] = i < nseg ? slot_quota[i] : 0;
            e_first[i] = e_last[i] = -1;
            e_cnt[i] = 0;
            e_cum[i] = 0ll;
            if (mode == MOE_MODE_DISTRIBUTION && i < E) {
                if (!WHOLE_STEP) e_true[i] = hist_true[i];
                e_hat[i] = hist_pred[i];
            }
        }
        __syncthreads();
        if (w == kSmallWaves - 1) {
            const SmallTables t{s_e, s_q, s_cum, s_next, e_first, e_cnt, e_last, e_cum};
            small_slot_tables(E, nseg, t);
        }
        chunk_stable_rank<kSmallWaves, SR>(key, valid, E, buf, rank,
                                           WHOLE_STEP && mode == MOE_MODE_DISTRIBUTION ? e_true : nullptr, rounds);
        if (WHOLE_STEP && mode == MOE_MODE_DISTRIBUTION && no_expert != 0)
#pragma unroll
            for (int r = 0; r < SR; ++r)
                if ((no_expert >> r) & 1) atomicAdd(&e_true[key[r]], -1);
        __syncthreads();  // the counters are dead, the buffer becomes rank and key by position
#pragma unroll
        for (int r = 0; r < SR; ++r) {
            const int p = (w * rounds + r) * kWave + lane;
            if (valid[r]) buf[p] = rank[r] | (key[r] << 16);
        }
        // upper bound of every slot's range of ranks from the quota up to it, all slots at once
        if (tid < nseg) {
            const int e = s_e[tid];
            long long hi = s_cum[tid];                                                  // Q_{r+1}
            if (mode == MOE_MODE_DISTRIBUTION && e >= 0 && e < E && e_hat[e] > 0)
                hi = ((long long)e_true[e] * hi) / e_hat[e];                            // floor(n_e * Q / nhat_e)
            if (hi > 0x7fffffffLL) hi = 0x7fffffffLL;
            s_hi[tid] = (int)hi;
        }
        // an expert nobody is predicted for keeps its home slot
        if (mode == MOE_MODE_DISTRIBUTION && tid < E && e_hat[tid] <= 0) e_first[tid] = -1;
    }
    __syncthreads();
    if (count)
#pragma unroll
        for (int r = 0; r < SR; ++r)
            if (valid[r] && !((no_expert >> r) & 1)) atomicAdd(&e_true[expert[r]], 1);

    // segment of every assignment: its place i in the plan's order for its expert (-1: none),
    // then a walk over the expert's slots, at most G of them, to the one whose range holds i;
    // the rounds walk in step so that their LDS reads overlap
    int sg[SR], place[SR];
    bool walking[SR];
#pragma unroll
    for (int r = 0; r < SR; ++r) {
        const int p = (w * rounds + r) * kWave + lane;
        sg[r] = 0;
        place[r] = -1;
        walking[r] = false;
        if (!valid[r]) continue;
        if (mode == MOE_MODE_DISTRIBUTION) {
            place[r] = rank[r];
        } else if (mode == MOE_MODE_TOKEN) {
            const int row0 = (p / k) * k;  // the token's predicted ids
            for (int jp = 0; jp < k; ++jp) {
                const int v = buf[row0 + jp];
                if ((v >> 16) == expert[r]) {
                    place[r] = v & 0xffff;
                    break;
                }
            }
        }
        sg[r] = e_home[expert[r]];
        if (place[r] >= 0) {
            const int first = e_first[expert[r]];
            if (first >= 0) {
                sg[r] = first;
                walking[r] = true;
            }
        }
    }
    for (int seen = 1; mode != MOE_MODE_NONE && seen < G; ++seen) {
        bool more = false;
#pragma unroll
        for (int r = 0; r < SR; ++r) {  // no branches: sg[r] is a slot in any case, the reads overlap
            if (r >= rounds) continue;       // (uniform)
            const int nx = s_next[sg[r]];
            const int hi = s_hi[sg[r]];
            walking[r] = walking[r] && nx >= 0 && place[r] >= hi;
            sg[r] = walking[r] ? nx : sg[r];
            more = more || walking[r];
        }
        if (!__any(more)) break;
    }
    __syncthreads();  // every look-up of a rank is done before the buffer holds counters again

    chunk_stable_rank<kSmallWaves, SR>(sg, valid, nseg, buf, rank, tot, rounds);
    block_exclusive_scan_2048(tot, nseg, wave_sum);
    for (int s = tid; s <= nseg; s += kSmallThreads) seg_offsets[s] = tot[s];
    for (int g = tid; g < G; g += kSmallThreads) rank_load[g] = tot[(g + 1) * S] - tot[g * S];
    if (WHOLE_STEP) {  // (barriers lie between the counting and here)
        for (int e = tid; e < E; e += kSmallThreads) hist_out[e] = e_true[e];
        if (mode == MOE_MODE_NONE) {
            for (int s = tid; s < nseg; s += kSmallThreads) {
                const int j = s % S, e = s / S * H + j;
                const bool held = j < H && e < E;
                s_e[s] = home.slot_expert[s] = held ? e : -1;
                home.slot_quota[s] = held ? e_true[e] : 0;
            }
            for (int g = tid; g < G; g += kSmallThreads) {
                int load = 0;
                for (int e = g * H; e < (g + 1) * H && e < E; ++e) load += e_true[e];
                home.rank_load_pred[g] = load;
            }
            if (tid == 0) home.n_iters[0] = 0;
        }
    }
#pragma unroll
    for (int r = 0; r < SR; ++r) {
        const int p = (w * rounds + r) * kWave + lane;
        if (!valid[r]) continue;
        const int row = tot[sg[r]] + rank[r];
        row_of_assign[p] = row;
        assign_of_row[row] = p;
    }
    if (WHOLE_STEP && job.lists.rows) {
        __syncthreads();  // the counters are dead for good
        using Scratch = TableScratch<kSmallKeys, kSmallKeys, 2>;
        static_assert(sizeof(Scratch) <= sizeof(buf), "the tables' scratch takes the counters' place");
        build_tables(*(Scratch*)buf, 0, 1, 0, tot, s_e, job);
    }
}

template <int UNROLL>
__global__ __launch_bounds__(256) void perm_scatter_rows_kernel(RowCopy copy) {
    copy_rows<UNROLL>(copy, __builtin_amdgcn_readfirstlane((int)((blockIdx.x * (unsigned)blockDim.x + threadIdx.x) / kWave)));
}

}  // namespace moegps

extern "C" size_t moe_permute_workspace_bytes(int T, int E, int k, int G, int S) {
    using namespace moegps;
    if (T < 0 || E < 1 || k < 1 || G < 1 || S < 1) return 0;
    if (E > MOE_MAX_EXPERTS || k > MOE_MAX_TOPK || G > MOE_MAX_RANKS || S > MOE_MAX_SLOTS || G * S > MOE_MAX_SEGMENTS ||
        (int64_t)T * k >= (1ll << 31))
        return 0;
    return perm_ws_bytes(T, E, k, G, S);
}

namespace moegps {
template <bool WHOLE_STEP>
static void launch_small(int mode, int T, int k, int E, int G, int S, const int32_t* topk_idx, const int32_t* pred_idx,
                         const int32_t* hist_true, const int32_t* hist_pred, const int32_t* slot_expert,
                         const int32_t* slot_quota, int32_t* seg_offsets, int32_t* row_of_assign,
                         int32_t* assign_of_row, int32_t* rank_load, int32_t* hist_out, const HomePlan& home,
                         const TableJob& job, hipStream_t st) {
    const int64_t A = (int64_t)T * k;
    hipLaunchKernelGGL((A <= 2 * kSmallThreads ? perm_small_kernel<2, WHOLE_STEP>
                        : A <= 3 * kSmallThreads ? perm_small_kernel<3, WHOLE_STEP>
                        : A <= 4 * kSmallThreads ? perm_small_kernel<4, WHOLE_STEP>
                                                 : perm_small_kernel<kSmallMaxRounds, WHOLE_STEP>),
                       dim3(1), dim3(kSmallThreads), 0, st, mode, T, k, E, G, S, topk_idx, pred_idx, hist_true, hist_pred,
                       slot_expert, slot_quota, seg_offsets, row_of_assign, assign_of_row, rank_load, hist_out, home, job);
}

bool permute_in_one_workgroup(int mode, int64_t A, int E, int nseg) { return A <= one_workgroup_limit(mode, E, nseg); }

int permute_and_count(int mode, int T, int k, int E, int G, int S, const int32_t* topk_idx, const int32_t* pred_idx,
                      const int32_t* hist_pred, const int32_t* slot_expert, const int32_t* slot_quota,
                      int32_t* seg_offsets, int32_t* row_of_assign, int32_t* assign_of_row, int32_t* rank_load,
                      int32_t* hist_out, const HomePlan& home, const TableJob& job, hipStream_t st) {
    launch_small<true>(mode, T, k, E, G, S, topk_idx, pred_idx, nullptr, hist_pred, slot_expert, slot_quota, seg_offsets,
                       row_of_assign, assign_of_row, rank_load, hist_out, home, job, st);
    return check_launch();
}

static int scatter_rows(const RowCopy& copy, hipStream_t st) {
    const dim3 grid((unsigned)ceil_div64((int64_t)copy.T * copy.slices, 4));
    if (row_copy_unroll(copy.chunks) == 4) hipLaunchKernelGGL(perm_scatter_rows_kernel<4>, grid, dim3(256), 0, st, copy);
    else hipLaunchKernelGGL(perm_scatter_rows_kernel<1>, grid, dim3(256), 0, st, copy);
    return check_launch();
}

// The index steps by many workgroups.  hist_out: the histogram, zero so far, is an output (not for batches that are scanned),
// and in mode 0 the plan, `home`.
static int permute_wide(int mode, int T, int k, int E, int G, int S, const int32_t* topk_idx, const int32_t* pred_idx,
                        const int32_t* hist_true, const int32_t* hist_pred, const int32_t* slot_expert,
                        const int32_t* slot_quota, const PermWs& ws, int32_t* seg_offsets, int32_t* row_of_assign,
                        int32_t* assign_of_row, int32_t* rank_load, int32_t* hist_out, const HomePlan& home,
                        hipStream_t st) {
    const int nb = ws.nb;
    const bool scanned = perm_scanned(ws);
    const bool dist = mode == MOE_MODE_DISTRIBUTION;
    const int32_t* scale = hist_out && dist ? hist_out : nullptr;
    int rc;
    if (mode != MOE_MODE_NONE) {
        const int32_t* keys = (mode == MOE_MODE_TOKEN) ? pred_idx : topk_idx;
        hipLaunchKernelGGL(perm_count_kernel, dim3(nb + ceil_div(E, kPermWaves)), dim3(kPermThreads), 0, st, keys, mode, T, k,
                           E, G, S, hist_out ? nullptr : hist_true, hist_pred, slot_expert, slot_quota, ws,
                           dist ? hist_out : nullptr);
        if ((rc = check_launch()) != MOE_OK) return rc;
        if (scanned && nb > 0) {
            hipLaunchKernelGGL(perm_scan1_kernel, dim3(ceil_div(E, kScan1Threads / kWave)), dim3(kScan1Threads), 0, st, E, ws);
            if ((rc = check_launch()) != MOE_OK) return rc;
        }
    }
    if (nb > 0) {
        hipLaunchKernelGGL(scanned ? perm_segment_kernel<true> : perm_segment_kernel<false>, dim3(nb), dim3(kPermThreads), 0,
                           st, mode, T, k, E, G, S, topk_idx, pred_idx, ws, scale, scale ? hist_pred : nullptr,
                           dist ? nullptr : hist_out);
        if ((rc = check_launch()) != MOE_OK) return rc;
    }
    if (scanned) {
        hipLaunchKernelGGL(perm_scan2_kernel, dim3(1), dim3(1024), 0, st, G, S, ws, seg_offsets, rank_load);
        if ((rc = check_launch()) != MOE_OK) return rc;
    }
    if (nb > 0) {
        hipLaunchKernelGGL(scanned ? perm_place_kernel<true> : perm_place_kernel<false>, dim3(nb), dim3(kPermThreads), 0, st, T,
                           k, G, S, ws, seg_offsets, rank_load, row_of_assign, assign_of_row, home, hist_out, E);
        if ((rc = check_launch()) != MOE_OK) return rc;
    }
    return MOE_OK;
}

bool permute_counts(int T, int E, int k, int G, int S) {
    const PermWs ws = perm_ws_layout(T, E, k, G, S, nullptr);
    return ws.nb > 0 && !perm_scanned(ws);
}

int permute_and_count_wide(int mode, int T, int k, int E, int G, int S, const int32_t* topk_idx, const int32_t* pred_idx,
                           const int32_t* hist_pred, const int32_t* slot_expert, const int32_t* slot_quota,
                           int32_t* seg_offsets, int32_t* row_of_assign, int32_t* assign_of_row, int32_t* rank_load,
                           int32_t* hist_out, const HomePlan& home, void* workspace, hipStream_t st) {
    return permute_wide(mode, T, k, E, G, S, topk_idx, pred_idx, nullptr, hist_pred, slot_expert, slot_quota,
                        perm_ws_layout(T, E, k, G, S, (char*)workspace), seg_offsets, row_of_assign, assign_of_row, rank_load,
                        hist_out, mode == MOE_MODE_NONE ? home : HomePlan{}, st);
}

static int permute_impl(int mode, const void* x, int dtype, int T, int d, int E, int k, int G, int S,
                        const int32_t* topk_idx, const int32_t* pred_idx, const int32_t* hist_true,
                        const int32_t* hist_pred, const int32_t* slot_expert, const int32_t* slot_quota,
                        int32_t* seg_offsets, int32_t* row_of_assign, int32_t* assign_of_row, void* x_perm,
                        int32_t* rank_load, void* workspace, size_t workspace_bytes, void* stream) {
    if (mode < MOE_MODE_NONE || mode > MOE_MODE_TOKEN) return MOE_ERR_INVALID_ARG;
    if (dtype != MOE_DTYPE_F32 && dtype != MOE_DTYPE_BF16) return MOE_ERR_INVALID_ARG;
    if (T < 0 || d < 1 || E < 1 || k < 1 || k > E || G < 1 || S < 1) return MOE_ERR_INVALID_ARG;
    if (E > MOE_MAX_EXPERTS || k > MOE_MAX_TOPK || G > MOE_MAX_RANKS || S > MOE_MAX_SLOTS ||
        G * S > MOE_MAX_SEGMENTS)
        return MOE_ERR_UNSUPPORTED;
    if (ceil_div(E, G) > S) return MOE_ERR_INVALID_ARG;
    if ((int64_t)T * k >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;
    if (((size_t)d * dtype_size(dtype)) % 16 != 0) return MOE_ERR_UNSUPPORTED;
    if (!seg_offsets || !rank_load || !slot_expert || !slot_quota || !workspace) return MOE_ERR_INVALID_ARG;
    if (T > 0 && (!topk_idx || !row_of_assign || !assign_of_row)) return MOE_ERR_INVALID_ARG;
    if (mode == MOE_MODE_TOKEN && T > 0 && !pred_idx) return MOE_ERR_INVALID_ARG;
    if (mode == MOE_MODE_DISTRIBUTION && (!hist_true || !hist_pred)) return MOE_ERR_INVALID_ARG;
    if (x_perm && T > 0 && !x) return MOE_ERR_INVALID_ARG;
    if (workspace_bytes < perm_ws_bytes(T, E, k, G, S)) return MOE_ERR_WORKSPACE_TOO_SMALL;
    const PermWs ws = perm_ws_layout(T, E, k, G, S, (char*)workspace);

    hipStream_t st = (hipStream_t)stream;
    const int nb = ws.nb;
    int rc;
    const int64_t A = (int64_t)T * k;
    if (A <= one_workgroup_limit(mode, E, G * S)) {
        launch_small<false>(mode, T, k, E, G, S, topk_idx, pred_idx, hist_true, hist_pred, slot_expert, slot_quota,
                            seg_offsets, row_of_assign, assign_of_row, rank_load, nullptr, HomePlan{},
                            TableJob{}, st);
        if ((rc = check_launch()) != MOE_OK) return rc;
    } else {
        if ((rc = permute_wide(mode, T, k, E, G, S, topk_idx, pred_idx, hist_true, hist_pred, slot_expert, slot_quota, ws,
                               seg_offsets, row_of_assign, assign_of_row, rank_load, nullptr, HomePlan{}, st)) != MOE_OK)
            return rc;
    }
    if (nb > 0) {
        if (x_perm && (rc = scatter_rows(row_copy(x, dtype, T, d, k, row_of_assign, x_perm), st)) != MOE_OK) return rc;
    }
    return MOE_OK;
}
}  // namespace moegps

extern "C" int moe_permute(int mode, const void* x, int dtype, int T, int d, int E, int k, int G, int S,
                           const int32_t* topk_idx, const int32_t* pred_idx, const int32_t* hist_true,
                           const int32_t* hist_pred, const int32_t* slot_expert, const int32_t* slot_quota,
                           int32_t* seg_offsets, int32_t* row_of_assign, int32_t* assign_of_row, void* x_perm,
                           int32_t* rank_load, void* workspace, size_t workspace_bytes, void* stream) {
    return moegps::permute_impl(mode, x, dtype, T, d, E, k, G, S, topk_idx, pred_idx, hist_true, hist_pred,
                                slot_expert, slot_quota, seg_offsets, row_of_assign, assign_of_row, x_perm, rank_load,
                                workspace, workspace_bytes, stream);
}

// ---------------------------------------------------------------------------
// The same permutation for callers that cannot allocate: the counters, chunk bases and
// segment ids live in a fixed array in device memory that belongs to the library.
// ---------------------------------------------------------------------------
namespace moegps {
static __device__ __align__(256) unsigned char scratch[MOE_PERMUTE_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each GPU, looked up once

// Address of this GPU's copy of the array (every GPU that loads the library holds its own,
// at its own address).  The array's name is only a host-side handle: kernels get this pointer.
static int static_scratch(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_last_hip_error(e);
        return MOE_ERR_HIP;
    }
    if (dev < 0 || dev >= kMaxDevices) return MOE_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_last_hip_error(e);
            return MOE_ERR_HIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MOE_OK;
}
}  // namespace moegps

extern "C" int moe_permute_static(int mode, const void* x, int dtype, int T, int d, int E, int k, int G, int S,
                                  const int32_t* topk_idx, const int32_t* pred_idx, const int32_t* hist_true,
                                  const int32_t* hist_pred, const int32_t* slot_expert, const int32_t* slot_quota,
                                  int32_t* seg_offsets, int32_t* row_of_assign, int32_t* assign_of_row, void* x_perm,
                                  int32_t* rank_load, void* stream) {
    using namespace moegps;
    if (T < 0 || E < 1 || k < 1 || G < 1 || S < 1) return MOE_ERR_INVALID_ARG;
    // sizes whose counters do not fit the fixed array are refused before anything is enqueued
    if (perm_ws_bytes(T, E, k, G, S) > (size_t)MOE_PERMUTE_STATIC_SCRATCH_BYTES)
        return MOE_ERR_WORKSPACE_TOO_SMALL;
    void* ptr = nullptr;
    const int rc = static_scratch(&ptr);
    if (rc != MOE_OK) return rc;
    return permute_impl(mode, x, dtype, T, d, E, k, G, S, topk_idx, pred_idx, hist_true, hist_pred, slot_expert,
                        slot_quota, seg_offsets, row_of_assign, assign_of_row, x_perm, rank_load, ptr,
                        (size_t)MOE_PERMUTE_STATIC_SCRATCH_BYTES, stream);
}
