// Row list and M-tile tables of the grouped FFN (grouped_ffn.hip), built on the device from the ragged
// segments: by a launch of their own, or by the workgroup that has just done the permutation (permute.hip).
#pragma once
#include "common.h"
#include "block_scan.h"
#include "row_copy.h"

namespace moegps {

// One entry of an M-tile table: consecutive positions of the row list, all of one
// expert, and the part of the K range this entry covers.
struct MTile {
    int list0;   // first position in the row list
    int rows;    // valid rows
    int expert;  // expert whose weights the rows take
    int kt0;     // k-tiles [kt0, kt1) of the product belong to this entry; kt1 == 0: all of them
    int kt1;
    int part;    // < 0: results go to the output (kPartAlone: from the expert's only tile of the table); else
                 //   fp32 partial sums go to slab `part`
    int first;   // whole tiles: the expert's whole tiles are the entries [first, first + n_same)
    int n_same;
};
// An M-tile whose K range is split, for the pass that adds up the partial sums
struct SplitInfo {
    int list0, rows;
};
constexpr int kPartWhole = -1, kPartAlone = -2;
constexpr int kGemmGrid = 256;  // persistent workgroups of a GEMM launch: 8 XCDs x 32
constexpr int kPartRows = 256;  // rows of one slab of partial sums (the tallest tile shape)
constexpr int kMaxParts = 4;    // parts of K of a split tile

// counts[] of a table: number of entries, how many of them are whole tiles (they come first; behind
// them the parts of split tiles), number of split M-tiles
constexpr int kCntEntries = 0, kCntWhole = 1, kCntSplit = 2, kCntStride = 4;

// What one product's table is built for.
struct TableSpec {
    MTile* tiles;       // out
    int32_t* counts;    // out, kCntStride ints
    SplitInfo* splits;  // out (split tiles only), may be null when parts <= 1
    int bm;             // most rows of a tile, 0: chosen from the batch
    int capacity;       // entries `tiles` has room for
    int kt;             // k-tiles of the product
    int parts;          // parts of K of a split tile (<= 1: no tile is split)
    int n_ntiles;       // N-tiles of the product (tile heights and split tiles go by the tiles
                        //   that the kGemmGrid workgroups of its launch get)
    int split_all;      // split every tile (tests)
    int split_capacity; // split M-tiles `splits` and the slabs have room for
};

// Row list: position p holds a row of x_perm; the rows of an expert's segments (ascending
// slot id, rows ascending) are consecutive, experts ascending.
// M-tile tables: an expert's rows are cut into as few tiles as the height allows, evenly (a tile costs by
// its rows, ffn_tiles.h, so two of 160 and 140 rows are done before one of 256 and one of 44), in steps of the
// 32 rows the kernels have loops for.  An expert's tiles stay together, in expert order (they share weight
// panels; the kernels walk them by MTile::first and n_same), experts with tiles of up to kShortTile rows
// behind the others: what is left for the end of the launch is then short, while tall tiles, bound by the matrix pipe,
// stay mixed with middling ones, bound by their weights (tallest first altogether: 64 experts of 2048 x 1408, 4096
// tokens, second product 189 us, as it is 184; short ones where they fall: 206).
// The height is worked out here, where the rows per expert are known, one lane per candidate: the
// launch's time is taken as the longest of (a) for every height in the table, the rounds that the
// tiles of that height and above make of the workgroups, and (b) the mean work of a workgroup and a quarter of a
// closing tile; where tiles may be split as the work, a third dearer, and the pass that adds them up.  A tile's cost is
// kCostFixed + its 16-row groups.  The constants are fitted to 78 products of 39 batches (five shapes, 8 to 224 k-tiles,
// 2 to 112 N-tiles, 150 to 16384 tokens), each timed with all seven heights: the height taken is 0.9 % above the best one
// on average, 7 % at most.  Both products, us, 256- or 128-row tiles by a rule on the mean rows per expert ->
// this: 777 tokens, top-8 of 128 experts of 4096 x 1536 389 -> 354; 1001 tokens, top-2 of 8 of 4096 x 14336 819 ->
// 730; 2048 tokens, top-6 of 64 of 2048 x 1408 345 -> 310; 3000 tokens, top-4 of 16 of 4096 x 688 261 -> 223; 4096
// tokens, top-2 of 8 of 512 x 1024 83 -> 48.
// With parts > 1 the closing M-tiles are listed once per part of K instead, behind the
// whole ones and part by part, each entry writing fp32 partial sums to a slab of its own (slab =
// split tile * parts + part).  What is split is what goes beyond whole rounds of one tile per workgroup,
// unless it is most of a round anyway (more than 5/8: splitting would add traffic and save little), the last tiles of the
// order.  The rule counts tiles and not their cost, and goes its own way where the height was taken for whole tiles.  Both
// products, us, whole tiles -> by the rule: 8 experts of 1024 x 4096, 300 tokens 81 -> 58, 8 of 4096 x 14336, 1001 tokens 839
// -> 790; but 64 of 2048 x 1408, 2048 tokens 305 -> 350, 8 of 512 x 1024, 600 tokens 31 -> 36.
//
// The work is small and what it costs is waiting: for barriers of 16 wavefronts and for chains of LDS
// round trips.  So one wavefront does the parts that need an order (64 segments or experts at a
// time, equal keys found by ballots, counts carried in LDS, prefix sums by DPP), without a
// barrier between its steps, and the workgroup meets three times: segments loaded, list order
// known, table prepared; the row list and the table entries are written by everybody.
// Every workgroup works out the list order and fills its stripe of the row list; workgroup 0
// writes the first table and sets the claim counters, workgroup 1 the second (the launch has two at least).
// Against pairs of segments and of experts dealt over the workgroup, some 30 barriers, and stripes of
// 4096 positions: 8 experts in 12 slots 10.3 -> 6.5 us (in 16 slots 9.4 -> 5.5); 128 experts in 160
// slots, one token 15.8 -> 8.5, 128 tokens 17.5 -> 9.4, 777 tokens and two tables 19.6 -> 10.5; 64 experts
// in 80 slots, 98304 rows 16.7 -> 11.  Pairs cost nothing for slots without rows; with hundreds of
// experts, groups of 64 slots or experts without rows are therefore skipped and the scans keep four reads
// under way (1024 experts in as many slots, 1024 rows on 16 of them, whole FFN of 64 x 64 weights: pairs 26.1,
// without the skip 38.7, now 25.2 us; on all 1024 216, 48.4, 48.2).

// exclusive prefix sums of data[0 .. n) in LDS, in place, by one wavefront; data[n] = total, returned
template <int UNROLL = 1>  // reads under way together: more than one pays with eight words per lane and up
__device__ __forceinline__ int wave_scan_lds(int* data, int n) {
    const int lane = threadIdx.x & (kWave - 1);
    const int per = ceil_div(n, kWave);
    const int i0 = lane * per < n ? lane * per : n, i1 = i0 + per < n ? i0 + per : n;
    int mine = 0;
#pragma unroll UNROLL
    for (int i = i0; i < i1; ++i) mine += data[i];
    const int incl = wave_prefix_i32(mine);
    int run = incl - mine;
#pragma unroll UNROLL
    for (int i = i0; i < i1; ++i) {
        const int c = data[i];
        data[i] = run;
        run += c;
    }
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    if (lane == 0) data[n] = total;
    wave_lds_order();
    return total;
}

// the same over the experts
__device__ __forceinline__ int wave_scan_experts(int* data, int E) {
    return E >= 8 * kWave ? wave_scan_lds<4>(data, E) : wave_scan_lds(data, E);
}

// lanes that hold the same key (below 1 << nbits) among the lanes with `live`
__device__ __forceinline__ unsigned long long same_key_lanes(int key, bool live, int nbits) {
    unsigned long long same = __ballot(live);
    for (int b = 0; b < nbits; ++b) {
        const bool one = (key >> b) & 1;
        const unsigned long long m = __ballot(live && one);
        same &= one ? m : ~m;
    }
    return live ? same : 0ull;
}

constexpr int kTallest = 256, kHeightStep = 32;      // rows of the tallest tile; heights are multiples of the step
constexpr int kHeights = kTallest / kHeightStep;
constexpr int kMinAutoHeight = 64;                   // lowest height that is chosen from the batch
constexpr int kCandidates = (kTallest - kMinAutoHeight) / kHeightStep + 1;
constexpr int kShortTile = 64;                       // tiles of up to so many rows come last
constexpr int kCostFixed = 8;                        // cost of a tile: this and its 16-row groups
static_assert(MOE_MAX_EXPERTS <= 1 << 12 && MOE_MAX_SEGMENTS <= 1 << 19, "expert and place share one int");

// Height of the tiles that `rows` rows of one expert are cut into, at most `most` each (a multiple of the step).
__device__ __forceinline__ int even_height(int rows, int most) {
    const int n = (rows + most - 1) / most;
    if (n > kHeights) return most;  // (n - 1) / n of the limit is less than a step below it
    return ((rows + n - 1) / n + kHeightStep - 1) / kHeightStep * kHeightStep;
}

// Row list, and the list of the rows' tokens, rows r being the assignments of[r], `per_token` to a token (null: not wanted).
struct RowLists {
    int32_t* rows;
    int32_t* tokens;
    const int32_t* of;
    int per_token;
};

// Everything a builder needs to know.
struct TableJob {
    int E, seg_begin, seg_end;
    TableSpec t1, t2;    // of the two products; tiles null: none wanted
    RowLists lists;
    int32_t* queues;     // claim counters to set
    int n_queues;
    int32_t* left;       // both products in one launch: what the second waits for (ffn_tiles.h); null: a launch each
};

// LDS of a builder for up to MAXSEG segments and MAXE experts that makes NT tables.
template <int MAXSEG, int MAXE, int NT>
struct TableScratch {
    int s_rows[MAXSEG];       // rows of the segment
    int s_ex[MAXSEG];         // its expert and, from bit 12, its place there; -1: not live
    int s_first[MAXSEG];      // first row of x_perm
    int srt_base[MAXSEG + 1]; // list position of the j-th segment in list order
    int srt_first[MAXSEG];    // its first row of x_perm
    int e_segs[MAXE + 1];     // live segments per expert -> base in list order
    struct {
        int o_base[MAXE + 1]; // tiles of the o-th expert in tile order -> those before it
        int o_expert[MAXE];   // that expert, and from bit 12 the height of its tiles
        int c_tiles[kCandidates][kHeights + 1];  // tiles of a height, per candidate
        int plan[4];          // ordered experts, tiles, split ones of them
    } t[NT];
};

// Workgroup `block` of `n_blocks`, 1024 threads: its stripe of the row list and tables first_table ..
// first_table + NT - 1 (table 2 and up: none).  seg_offsets may be in LDS.
template <int MAXSEG, int MAXE, int NT>
__device__ __forceinline__ void build_tables(TableScratch<MAXSEG, MAXE, NT>& sh, int block, int n_blocks, int first_table,
                                             const int32_t* seg_offsets, const int32_t* slot_expert,
                                             const TableJob& job) {
    const int E = job.E;
    int (&s_rows)[MAXSEG] = sh.s_rows, (&s_ex)[MAXSEG] = sh.s_ex, (&s_first)[MAXSEG] = sh.s_first;
    int (&srt_base)[MAXSEG + 1] = sh.srt_base, (&srt_first)[MAXSEG] = sh.srt_first, (&e_segs)[MAXE + 1] = sh.e_segs;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int ns = job.seg_end - job.seg_begin;
    const bool many = E > 4 * kWave;  // experts enough that looking for groups of 64 without rows pays
    if (block == 0)
        for (int i = tid; i < job.n_queues; i += blockDim.x)
            job.queues[i] = job.left ? 0 : kGemmGrid / 8;  // (a launch each: first tiles are claimed)
    for (int e = tid; e < E; e += blockDim.x) e_segs[e] = 0;
    for (int i = tid; i < ns; i += blockDim.x) {
        const int s = job.seg_begin + i;
        const int lo = seg_offsets[s];
        const int rows = seg_offsets[s + 1] - lo;
        const int e = slot_expert[s];
        s_rows[i] = rows;
        s_ex[i] = rows > 0 && e >= 0 && e < E ? e : -1;
        s_first[i] = lo;
    }
    __syncthreads();
    if (wave == 0) {
        const int nbits = E > 1 ? 32 - __builtin_clz(E - 1) : 0;
        for (int i0 = 0; i0 < ns; i0 += kWave) {
            const int i = i0 + lane;
            const int e = i < ns ? s_ex[i] : -1;
            if (many && __ballot(e >= 0) == 0ull) continue;
            const unsigned long long same = same_key_lanes(e, e >= 0, nbits);
            if (e >= 0) {
                const int before = e_segs[e];
                s_ex[i] = e | (before + __popcll(same & lt)) << 12;
                if ((same & ~lt) == (1ull << lane)) e_segs[e] = before + __popcll(same);  // the last of them
            }
            wave_lds_order();
        }
        wave_scan_experts(e_segs, E);
        for (int i = lane; i < ns; i += kWave) {
            const int v = s_ex[i];
            if (v < 0) continue;
            const int j = e_segs[v & 0xfff] + (v >> 12);
            srt_base[j] = s_rows[i];
            srt_first[j] = s_first[i];
        }
        wave_lds_order();
        wave_scan_lds(srt_base, e_segs[E]);
    }
    __syncthreads();
    const int n_live = e_segs[E], n_list = srt_base[n_live];
    // row list: binary search of the position among the segments in list order
    auto fill_rows = [&] {
        for (int p = block * blockDim.x + tid; p < n_list; p += n_blocks * blockDim.x) {
            int lo = 0, hi = n_live - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (srt_base[mid] <= p) lo = mid;
                else hi = mid - 1;
            }
            const int r = srt_first[lo] + (p - srt_base[lo]);
            job.lists.rows[p] = r;
            if (job.lists.tokens) job.lists.tokens[p] = job.lists.of[r] / job.lists.per_token;
        }
    };
    // tables
    auto list_base = [&](int e) { return srt_base[e_segs[e]]; };  // first list position of expert e
    if (block == 0 && job.left)
        for (int e = tid; e < E; e += blockDim.x) job.left[e] = -((list_base(e + 1) - list_base(e)) * job.t1.n_ntiles);
    // wavefront j < NT prepares table first_table + j while the others fill in the row list
    auto spec_of = [&](int j) -> const TableSpec& { return first_table + j == 0 ? job.t1 : job.t2; };
    auto wanted = [&](int j) { return first_table + j < 2 && spec_of(j).tiles != nullptr; };
    const bool busy = wave < NT && wanted(wave);
    if (!busy) fill_rows();
    bool any_table = false;  // (uniform)
    for (int j = 0; j < NT; ++j) any_table = any_table || wanted(j);
    if (any_table) {
        if (busy) {
            const TableSpec& ts = spec_of(wave);
            int (&o_base)[MAXE + 1] = sh.t[wave].o_base, (&o_expert)[MAXE] = sh.t[wave].o_expert;
            int (&c_tiles)[kCandidates][kHeights + 1] = sh.t[wave].c_tiles, (&s_plan)[4] = sh.t[wave].plan;
            const int P = ts.parts > kMaxParts ? kMaxParts : ts.parts;
            auto rows_of = [&](int e) { return e < E ? list_base(e + 1) - list_base(e) : 0; };
            auto none = [&](int e0) {  // no segment holds any of the 64 experts
                return many && e_segs[e0] == e_segs[e0 + kWave < E ? e0 + kWave : E];
            };
            int most = ts.bm;
            if (most == 0) {
                for (int i = lane; i < kCandidates * (kHeights + 1); i += kWave) (&c_tiles[0][0])[i] = 0;
                wave_lds_order();
                for (int e0 = 0; e0 < E; e0 += kWave) {
                    if (none(e0)) continue;
                    const int rows = rows_of(e0 + lane);
                    if (rows == 0) continue;
#pragma unroll
                    for (int c = 0; c < kCandidates; ++c) {
                        const int h = kTallest - c * kHeightStep;
                        atomicAdd(&c_tiles[c][even_height(rows, h) / kHeightStep], (rows + h - 1) / h);
                    }
                }
                wave_lds_order();
                const int c = lane < kCandidates ? lane : kCandidates - 1;
                float n = 0.f, work = 0.f, time = 0.f, first = 0.f, last = 0.f;
#pragma unroll
                for (int k = kHeights; k > 0; --k) {
                    const float m = (float)c_tiles[c][k] * (float)ts.n_ntiles;
                    if (m == 0.f) continue;
                    last = (float)(kCostFixed + 2 * k);
                    if (n == 0.f) first = last;
                    n += m;
                    work += m * last;
                    time = fmaxf(time, ceilf(n * (1.f / kGemmGrid)) * last);
                }
                time = fmaxf(time, work * (1.f / kGemmGrid) + 0.25f * last) + 0.1f * first;
                const float rem = n - floorf(n * (1.f / kGemmGrid)) * kGemmGrid;
                if (P > 1 && rem <= 0.625f * kGemmGrid)
                    time = fminf(time, work * (1.3f / kGemmGrid) + 0.4f * last + 400.f / ts.kt);
                // the taller of two that are as good
                int key = lane < kCandidates ? (int)(fminf(time, 1e7f) * 16.f) * 8 + lane : 0x7fffffff;
                for (int m = 1; m < 8; m <<= 1) {
                    const int o = __shfl_xor(key, m, kWave);
                    key = o < key ? o : key;
                }
                most = kTallest - (__builtin_amdgcn_readfirstlane(key) & 7) * kHeightStep;
            }
            // tile order: experts with tall tiles, then those with short ones, each group ascending
            int o = 0;
            for (int pass = 0; pass < 2; ++pass) {
                for (int e0 = 0; e0 < E; e0 += kWave) {
                    if (none(e0)) continue;
                    const int rows = rows_of(e0 + lane);
                    const int height = rows > 0 ? even_height(rows, most) : 0;
                    const bool mine = pass == 0 ? height > kShortTile : rows > 0 && height <= kShortTile;
                    const unsigned long long them = __ballot(mine);
                    if (mine) {
                        const int at = o + __popcll(them & lt);
                        o_expert[at] = (e0 + lane) | height << 12;
                        o_base[at] = (rows + height - 1) / height;
                    }
                    o += __popcll(them);
                }
            }
            if (lane == 0) s_plan[0] = o;
            wave_lds_order();
            const int n_tiles = wave_scan_experts(o_base, o);
            int n_split = 0;
            if (P > 1) {
                if (ts.split_all) n_split = n_tiles;
                else {
                    const int rem = (int)((long long)n_tiles * ts.n_ntiles % kGemmGrid);
                    if (rem * 8 <= kGemmGrid * 5) n_split = (rem + ts.n_ntiles - 1) / ts.n_ntiles;
                }
                if (n_split > ts.split_capacity) n_split = 0;  // no room (split_plan): whole ones then
            }
            if (lane == 0) {
                s_plan[1] = n_tiles;
                s_plan[2] = n_split;
            }
        }
        __syncthreads();
        for (int j = 0; j < NT; ++j) {
            if (!wanted(j)) continue;
            const TableSpec& ts = spec_of(j);
            const int (&o_base)[MAXE + 1] = sh.t[j].o_base, (&o_expert)[MAXE] = sh.t[j].o_expert;
            const int P = ts.parts > kMaxParts ? kMaxParts : ts.parts;
            const int n_order = sh.t[j].plan[0], n_tiles = sh.t[j].plan[1], n_split = sh.t[j].plan[2];
            const int n_whole = n_tiles - n_split;
            const int n_entries = n_whole + n_split * P;
            const bool fits = n_entries <= ts.capacity;
            auto part_range = [&](int part, int& k0, int& k1) {
                const unsigned a = (unsigned)(ts.kt * part), b = (unsigned)(ts.kt * (part + 1));  // (at most 2^16 k-tiles)
                k0 = (int)(P == kMaxParts ? a / kMaxParts : a / (unsigned)P);
                k1 = (int)(P == kMaxParts ? b / kMaxParts : b / (unsigned)P);
            };
            for (int t = tid; fits && t < n_tiles; t += blockDim.x) {
                int lo = 0, hi = n_order - 1;  // the expert whose range of tile numbers holds t
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (o_base[mid] <= t) lo = mid;
                    else hi = mid - 1;
                }
                const int expert = o_expert[lo] & 0xfff, height = o_expert[lo] >> 12;
                const int left = list_base(expert + 1) - list_base(expert) - (t - o_base[lo]) * height;
                MTile mt;
                mt.list0 = list_base(expert + 1) - left;
                mt.rows = left < height ? left : height;
                mt.expert = expert;
                mt.kt0 = mt.kt1 = 0;
                mt.part = o_base[lo + 1] - o_base[lo] == 1 ? kPartAlone : kPartWhole;
                mt.first = o_base[lo];
                mt.n_same = (o_base[lo + 1] < n_whole ? o_base[lo + 1] : n_whole) - mt.first;
                if (t < n_whole) {
                    ts.tiles[t] = mt;
                    continue;
                }
                const int split_index = t - n_whole;
                for (int part = 0; part < P; ++part) {
                    part_range(part, mt.kt0, mt.kt1);
                    mt.part = split_index * P + part;
                    ts.tiles[n_whole + part * n_split + split_index] = mt;
                }
                ts.splits[split_index].list0 = mt.list0;
                ts.splits[split_index].rows = mt.rows;
            }
            if (tid == 0) {
                ts.counts[kCntEntries] = fits ? n_entries : 0;
                ts.counts[kCntWhole] = fits ? n_whole : 0;
                ts.counts[kCntSplit] = fits ? n_split : 0;
            }
        }
    }
    if (busy) fill_rows();
}

// Overrides of the automatic choices (moe_grouped_ffn_set_option).  A call reads them once: another thread may
// set one at any time, and its kernels must be those that its tables were built for.
struct FfnOptions {
    int tile1, tile2, split, group_n, stream;
};
FfnOptions ffn_options();

// How much of a grouped FFN call is done: all of it; nothing but its checks and the job of its table
// builder; or everything behind the builder, which has run (with the options that the job was made with).
// `copy`: rows that the launch of the first product copies besides (to a place that the call does not read).
// `tokens`: A ints for the list of the rows' tokens, with gather_rows; without it the first product looks a row up twice.
enum FfnStage { kFfnAll, kFfnJobOnly, kFfnTablesBuilt };
int grouped_ffn_call(int relu, const void* x_in, int64_t rows_in, const int32_t* gather_rows, int gather_div,
                     const int32_t* scale_idx, const float* scale, int dtype, int64_t A, int d, int ffn, int E,
                     const int32_t* seg_offsets, const int32_t* slot_expert, int nseg, int seg_begin, int seg_end,
                     const void* packed, void* y_perm, void* workspace, size_t workspace_bytes, void* stream,
                     const FfnOptions& opt, FfnStage stage = kFfnAll, TableJob* job_out = nullptr,
                     const RowCopy& copy = RowCopy{}, int32_t* tokens = nullptr);

}  // namespace moegps
