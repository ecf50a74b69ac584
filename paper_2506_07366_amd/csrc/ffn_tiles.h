// Tiled form of the grouped bf16 GEMM, for batches with more than a few rows per expert.
// Included by grouped_ffn.hip inside namespace moegps (uses its types).
//
// A tile is up to 256 rows x 256 packed columns, worked on by eight wavefronts side by side along
// the columns, 32 each over all rows of the tile.  The two operands take different ways:
//   - weights go from memory straight into registers.  They are packed by MFMA fragment, so a
//     fragment is one contiguous kilobyte, and no two wavefronts of a workgroup want the same one;
//   - activation rows are wanted by all eight, so they are staged in LDS (buffer loads that write LDS
//     directly), three stages of 64 of K.
// What bounds a tile decides the split.  Above about 200 rows it is the matrix pipe under the chip's power
// limit; below, how fast a k-tile arrives: a request takes 1 to 2 us from memory under load, a k-tile
// of matrix work 0.1 to 1.1.  So three k-tiles are under way at a time, four where 128 rows and less leave
// the registers for it (four at 256 rows spill and are 1 % slower; three at 128 rows 1-2 % slower).  A tile of few rows
// then costs what its weights cost: us per k-tile in a launch with all kinds of tiles (4096 x 14336
// experts, 8192 rows on seven of eight), 16 / 80 / 144 / 256 rows: 0.60 / 0.83 / 1.12 / 1.45, against 1.26 / 1.26 / 1.36 /
// 1.40 with both operands through two LDS stages and the wavefronts in two rows of four.
// Both products, us, that form -> this: 4096 x 1536 experts, top-8 of 128, 777 tokens 398 -> 389, 4096 tokens
// 1527 -> 1362; 2048 x 1408, top-6 of 64, 2048 tokens 361 -> 343, 16384 tokens 1520 -> 1447; 4096 x 14336, top-2 of
// 8, 1001 tokens 850 -> 818, 4096 tokens 2347 -> 2264; 768 x 3072, top-1 of 64, 16384 tokens 239 -> 216; 4096 x 688,
// top-4 of 16, 8191 tokens 580 -> 548.
#pragma once

constexpr int kTileMaxRows = 256;  // rows of the tallest tile
constexpr int kTileGroup = 4;      // N-tiles walked side by side
constexpr int kNonTemporal = 2;    // cache policy of a buffer load: nt
constexpr int kThrough = 16;       // of a buffer store: sc1, written through to memory
constexpr int kCacheLine = 128;    // bytes, of the vector L1 and the L2
constexpr int kCopyPieces = 6;     // pieces of the row copy that a wavefront takes along with a tile
constexpr size_t kStageLds = (size_t)3 * kTileMaxRows * kPackK * 2;
// dynamic LDS of a workgroup: the stages, in the first product the copy's pieces, the number of the next tile
template <int EPI>
constexpr size_t kNextTileAt = kStageLds + (EPI != kEpiNone ? 8 * kCopyPieces * kCopyPieceLds : 0);
template <int EPI>
constexpr size_t kTileLds = kNextTileAt<EPI> + 16;

// Both products of an FFN in one launch (grouped_ffn_tiles_kernel): a workgroup that finds no tile of the first product
// left goes on to those of the second, and the uneven end of the first (a launch of few rounds of 256 tiles loses up to
// a fifth of one there) fills up with them.  A tile of the second needs the hidden rows of its expert: left[e] starts at
// -(rows of expert e) x (N-tiles of the first product), a finished tile of the first adds its rows, and at 0 all are there.
// A workgroup that waits for that waits for tiles that others are working on: it got to the second product because every
// tile of the first had been claimed, by a workgroup that was running, and a workgroup goes from a tile that it has claimed
// to telling so without waiting for anybody.  So a launch needs no number of its workgroups on the chip at a time.
// The XCDs' L2 caches are not coherent with each other inside a launch, so the hidden rows are written through to memory
// (kThrough) and the tile is told once every wavefront has seen its own stores acknowledged (at the start of the next
// tile, where the row list is waited for anyway); no cache can hold older hidden rows, nobody in the launch reads a
// row before it is complete, and a row is whole cache lines (the host sees to that: elsewhere a launch each).
//
// Whether a product shares its launch with the other one of the FFN.
constexpr int kAlone = 0, kMakesRows = 1, kWantsRows = 2;

typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;

// waits until *left is 0 (every wavefront by itself; uniform address)
__device__ __forceinline__ void wait_rows(int32_t* left) {
    while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0)
        __builtin_amdgcn_s_sleep(4);
    asm volatile("" ::: "memory");
}
// (behind a wait for this wavefront's stores and a barrier, neither of which the compiler takes for memory accesses: the
// stores must be ahead of them in the code, too, and the count behind)
__device__ __forceinline__ void rows_stored() {
    asm volatile("" ::: "memory");
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void tell_rows(int32_t* left, int& expert, int rows) {
    asm volatile("" ::: "memory");
    if ((threadIdx.x & 63) == 0)
        (void)__hip_atomic_fetch_add(&left[expert], rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    expert = -1;
}

template <int EPI, int LINK>
__device__ __forceinline__ void tile_product(
    const bf16_t* A, int lda,                        // activations [rows, K]
    const bf16_t* __restrict__ Bp, size_t b_stride,  // packed weights [E][N-tile][k-tile][kPackN x kPackK]
    bf16_t* C, int ldc,                              // output [rows, SWIGLU ? N/2 : N]
    const MTile* __restrict__ mtiles, const int32_t* __restrict__ counts, int32_t* __restrict__ queues,
    int N, int K, int group_n, bool past_caches, RowMap rm,
    float* __restrict__ partials,  // [slab][kPartRows][N] fp32 sums of entries that cover part of K (plain product, a launch of its own)
    RowCopy copy,                  // first product: rows to be copied besides, a share of them with every tile
    int32_t* left) {               // [E] what the second product waits for, see above (LINK)
    constexpr bool SWIGLU = EPI == kEpiSwiglu;
    constexpr int BN = kPackN, BK = kPackK, NW = 8;
    constexpr int ROW_BYTES = BK * 2;      // of an activation row in a stage
    constexpr int B_BYTES = BN * BK * 2;   // of a weight tile
    constexpr int TM_MAX = kTileMaxRows / 16;

    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int n_entries = counts[kCntEntries];
    const int n_whole = counts[kCntWhole];  // behind the whole tiles come the parts of split ones
    const int n_ntiles = (N + BN - 1) / BN;

    // Tile order.  The (entry, N-tile) space is walked in two passes: the whole M-tiles, then
    // the parts of split ones (part by part).  The tiles of an expert (in the second pass: all)
    // are numbered in groups of group_n neighbouring N-tiles; inside a group the N-tile index runs
    // fastest, then the M-tile, so a run of 32 consecutive tiles is a patch of M-tiles and N-tiles that
    // share their activation and weight panels, and an expert's weights are wanted while it is worked on and
    // not again.  Workgroups are dealt to the 8 XCDs
    // round-robin (workgroup b runs on XCD b % 8) and every XCD has its own L2, so run c of
    // the numbering belongs to XCD c % 8: its workgroups claim the tiles of its runs one by
    // one from a counter (tiles differ in cost, a fixed deal would leave workgroups idle at
    // the end) and so work side by side on one patch, sharing its panels through that L2; the
    // 8 XCDs are on 8 consecutive runs (shared through the memory-side cache).  A workgroup whose own
    // XCD has no tile left claims from the other XCDs' counters.
    // Four N-tiles by the expert's M-tiles are 1.7 % faster on average of fourteen batches (1001 to 32768 tokens) than
    // groups over all experts' M-tiles by size (all of up to 12 N-tiles, else 4 to 8); 3, 5 and 6, or
    // a square patch for few M-tiles, are 0.3 to 0.9 % slower.
    const int xcd = blockIdx.x & 7;
    constexpr int run = kGemmGrid / 8;  // the launch is always kGemmGrid workgroups
    const int total = n_entries * n_ntiles;
    const int total_whole = n_whole * n_ntiles;
    int copy_share = 0;  // pieces of the row copy that go with a tile
    if constexpr (EPI != kEpiNone)
        if (copy.x_perm) copy_share = ceil_div(copy.T * ceil_div(copy.chunks, kWave), total > 0 ? total : 1);
    volatile __attribute__((address_space(3))) int& next_tile =
        *(volatile __attribute__((address_space(3))) int*)(__attribute__((address_space(3))) unsigned char*)(smem + kNextTileAt<EPI>);
    // The claims are the business of wavefront 0, and every value involved is the same in
    // all its lanes, so the state lives in scalar registers (lane 0 performs the atomic, its
    // result is broadcast): nothing of it occupies a vector register across the K loop
    // except the pending result of the claim made ahead.
    int dry = 0;  // bit q set = counter q has run out
    // tile number for claim i of XCD q's counter, -1 if that counter has run out
    auto tile_of_claim = [&](int q, int i) {
        const int t = (q + 8 * (i / run)) * run + i % run;
        return t < total ? t : -1;  // claims only grow: past the end once, past the end for good
    };
    // number of claims counter q can serve: its runs are q, q + 8, ... of which the first
    // total / run are whole and run number total / run holds the remainder
    auto claims_of = [&](int q, int total) {  // (total handed in opaque: worked out only when needed)
        const int whole = total / run, part = total - whole * run;
        return (whole > q ? (whole - q + 7) / 8 * run : 0) + ((whole >= q && ((whole - q) & 7) == 0) ? part : 0);
    };
    // the counter to claim from next, own XCD first; -1 when all have run out
    auto next_counter = [&]() {
        for (int j = 0; j < 8; ++j) {
            const int q = (xcd + j) & 7;
            if (!((dry >> q) & 1)) return q;
        }
        return -1;
    };
    auto claim_from = [&](int q) {  // one claim, result not yet waited for (lane 0 holds it)
        int r = 0;
        if (lane == 0) r = atomicAdd(&queues[q], 1);
        return r;
    };
    // Turns a claim made ahead of time (or none: q < 0) into a tile, making further claims as
    // needed; -1 when every counter has run out.  Once a claim has come back empty all eight
    // counters are read in one go (one round trip, not one per counter), and those that stand
    // at their limit are struck off.
    auto settle_claim = [&](int q, int i) {
        for (;;) {
            if (q >= 0) {
                const int t = tile_of_claim(q, i);
                if (t >= 0) return t;
                dry |= 1 << q;
                const int seen = __hip_atomic_load(&queues[opaque(lane) & 7], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int total_now = opaque_uniform(total);
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    if (__builtin_amdgcn_readlane(seen, c) >= claims_of(c, total_now)) dry |= 1 << c;
            }
            q = next_counter();
            if (q < 0) return -1;
            i = __builtin_amdgcn_readfirstlane(claim_from(q));
        }
    };
    // The first tile of a workgroup is its own claim of its XCD's counter, made in advance (the counters
    // start at `run`): no round trip before it, and a workgroup that starts early cannot take it.  In a shared launch
    // workgroups wait for tiles, so only one that runs may own a tile: another launch that waits the same way, on another stream,
    // can keep the rest of this one from starting.  Its counters start at 0.
    if (wave == 0) next_tile = LINK == kAlone ? settle_claim(xcd, (int)(blockIdx.x >> 3)) : settle_claim(-1, 0);
    int told_expert = -1, told_rows = 0;  // the tile whose results are on their way to memory
    for (;;) {
        lds_wait<0>();                 // thread 0's store of next_tile
        __builtin_amdgcn_s_barrier();  // also: every wavefront is done reading the previous tile's stages
        const int t_all = __builtin_amdgcn_readfirstlane(next_tile);
        if (t_all < 0) break;
        // This tile's share of the row copy: its pieces, and where they go, are asked for ahead of the first k-tiles, in LDS with
        // the first of these (loads return in order), and stored behind the tile's own results, whose drain they lengthen.  What does
        // not fit into LDS (many tokens for few tiles) is copied here.  It saves the copy's launch and costs the tiles a part of that.  Whole
        // steps, us, a launch of the copy's own -> this: 16384 tokens, top-6 of 64 experts of 2048 x 1408 1659 -> 1624,
        // 32768, top-8 of 128 of 4096 x 1536 8791 -> 8488, 16384, top-1 of 64 of 768 x 3072 283 -> 276, 2048, top-6
        // of 64 of 2048 x 1408 392 -> 384; none on 8 of 4096 x 14336, 4096 tokens 2425 -> 2424, the first product 1502 -> 1525.  Loaded
        // and stored at the tile's start instead (one memory round trip more per tile) 1679, 8956,
        // 279; copied by workgroups behind those of the product, as these run out of tiles, 1665, 8707, 294.
        int copy_first = 0, copy_n = 0;  // this wavefront's pieces
        if constexpr (EPI != kEpiNone) {
            if (copy.x_perm) {
                const int all = copy.T * ceil_div(copy.chunks, kWave), first = t_all * copy_share;
                const int end = first + copy_share < all ? first + copy_share : all;
                const int most = copy_share < NW * kCopyPieces ? ceil_div(copy_share, NW) : kCopyPieces;
                copy_first = first + wave * most;
                copy_n = end - copy_first < most ? end - copy_first : most;
                if (copy_share > NW * kCopyPieces) copy_pieces<NW>(copy, first + NW * kCopyPieces, end, wave);
            }
        }
        // The claim for the tile after this one is made towards the end of the K loop and looked at behind
        // it: late, so that the workgroups that are ahead take what is left.
        int ahead_q = -1, ahead_pending = 0;
        const bool whole = t_all < total_whole;
        int m_base = n_whole, m_count = n_entries - n_whole;
        if (whole) {
            const MTile& any = mtiles[t_all / n_ntiles];
            m_base = any.first;
            m_count = any.n_same;
        }
        const int t = t_all - m_base * n_ntiles;
        const int per_group = m_count * group_n;
        const int grp = t / per_group;
        const int rem = t - grp * per_group;
        const int gw = (n_ntiles - grp * group_n) < group_n ? (n_ntiles - grp * group_n) : group_n;
        const int mt_i = m_base + rem / gw;
        const int nt_i = grp * group_n + rem % gw;
        const MTile mt = mtiles[mt_i];
        if constexpr (LINK == kWantsRows) wait_rows(&left[mt.expert]);
        const int n0 = nt_i * BN;
        // k-tiles of this entry: all of K, or the part of it a split tile covers
        const int KT = mt.kt1 > 0 ? mt.kt1 - mt.kt0 : K / BK;
        // rows that go through a list are addressed from the start of A (32-bit byte offsets:
        // the host checks that A fits), rows in place from the tile's first row
        const bf16_t* Ab = (rm.a_rows ? A : A + (size_t)mt.list0 * lda) + mt.kt0 * BK;
        // The wavefront's 32 packed columns are two 16-row groups of the weight tile: neighbours, or with
        // SwiGLU a gate group and its up group, two further.
        const int grp0 = SWIGLU ? (wave >> 1) * 4 + (wave & 1) : wave * 2;
        constexpr int JB = (SWIGLU ? 2 : 1) * 2 * kFragElems * 2;  // bytes between the two
        const unsigned char* Bw = (const unsigned char*)(Bp + (size_t)mt.expert * b_stride +
                                                         ((size_t)nt_i * (K / BK) + mt.kt0) * (BN * BK)) +
                                  grp0 * 2 * kFragElems * 2;
        // Both operands are addressed through buffer descriptors: a uniform base and a 32-bit offset per
        // lane, and a k-tile past the end is asked for out of the buffer's range, which keeps the number of
        // loads per k-tile fixed (the waits count them) and costs no memory access.  What such a load
        // returns is never multiplied.  (A weight panel is at most 2^31 bytes: 2^16 k-tiles of 32 KiB.
        // Activations reach up to 2^32 - 144 bytes: fewer than 2^31 elements, a row is a multiple of 64.)
        constexpr unsigned kARange = 0xffffff80u, kAPast = 0xfffffff0u, kWRange = 0x80000000u, kWPast = 0xfffff000u;
        const auto a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Ab, 0, (int)kARange, 0x00027000);
        const auto w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Bw, 0, (int)kWRange, 0x00027000);
        const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;

        // Accumulators hold the transposed product: the weight fragment is the MFMA's row operand and
        // the activation fragment its column operand, so element r of lane (l16, g16) in tile (i, j)
        // is output row i*16 + l16 and column 4*g16 + r of the wavefront's column group j.
        f32x4 acc[TM_MAX][2];
        const int lane_p = opaque(lane);

        // K loop over TM 16-row groups.  Fragment f of a k-tile is row group f % TM, step f / TM (32 of K);
        // R fragments are in registers or on their way, fragment f + R is read as soon as the
        // MFMAs of fragment f have been issued.  LDS reads complete in issue order, which fixes the wait
        // counts.  The hand-over to the next k-tile stands where half of the R last fragments are still to
        // be multiplied: all reads of this k-tile have landed by then at no cost, and the first reads of the next one land
        // under what is left.  It waits for this wavefront's own loads of the next k-tile; the barrier
        // extends that to every wavefront's, and says that the stage of this k-tile is free.  The loads of
        // k-tile kt + D - 1 go into the buffers that k-tile kt - 1 has left, dealt over the fragments before the hand-over.
        // (k-tile kt uses buffers kt % D; the loop is unrolled by D so that these are registers by name.)
        // once_tag: no other tile wants these weights (the expert's only M-tile, over all of K), they are read past
        // the caches, which are left to the rows.  Products 1 and 2, us, without -> with it: 128 experts of 4096 x
        // 1536, 400 tokens 170 + 103 -> 151 + 98, 1024 on all of them 568 + 316 -> 515 + 312; 64 of 2048 x 1408, 1024
        // tokens 168 + 92 -> 152 + 88; 8 of 4096 x 14336, 256 tokens 289 + 197 -> 270 + 206, 512 tokens, most
        // experts with two M-tiles, 330 + 211 -> 322 + 222.  26 batches: 2.1 % on average, 0.991 the worst.
        auto k_loop = [&](auto TM_tag, auto once_tag) {
            constexpr int TM = decltype(TM_tag)::value;
            constexpr int kAux = decltype(once_tag)::value ? kNonTemporal : 0;
            constexpr int D = TM <= 8 ? 4 : 3;                          // k-tiles under way
            constexpr int STAGE = (TM <= 8 ? 128 : 256) * ROW_BYTES;    // activation bytes of one of them
            static_assert((size_t)D * STAGE <= kStageLds, "LDS of the launch");
            constexpr int IA = (TM + 3) / 4;  // activation loads per wavefront and k-tile, 8 rows each
            constexpr int NB = 4 + IA;        // loads per wavefront and k-tile
            constexpr int NF = 2 * TM;
            constexpr int R = NF % 8 == 0 ? 8 : 4;
            constexpr int H = NF - R / 2;     // the hand-over opens fragment H
            static_assert(NF % R == 0 && H >= 1, "fragment f sits in register f % R in every k-tile");
            unsigned offA[IA];
#pragma unroll
            for (int i = 0; i < IA; ++i) {
                const int p = (wave + i * NW) * 64 + lane_p;
                const int row = p >> 3, slot = p & 7;
                int r = row < mt.rows ? row : mt.rows - 1;  // rows past the end repeat the last one
                if (rm.a_rows) {
                    r = rm.a_rows[mt.list0 + r];
                    if (rm.a_rows2) r = rm.a_rows2[r] / opaque_uniform(rm.a_div);
                }
                offA[i] = ((unsigned)r * (unsigned)lda + (unsigned)((slot ^ swz(row)) * 8)) * 2u;
            }
            if constexpr (LINK == kMakesRows) rows_stored();  // the previous tile's results have reached memory
            if constexpr (EPI != kEpiNone)  // (behind the row list, whose wait would be for the pieces too)
                if (copy_n > 0)
                    request_pieces(copy, copy_first, copy_n, smem + kStageLds + wave * (kCopyPieces * kCopyPieceLds));
            bf16x8 w[D][2][2], af[R];
            const unsigned lane_off = (unsigned)(lane_p * 16);
            // load l of this wavefront's NB loads of k-tile kt, into buffers b
            auto load_n = [&](auto L, int kt, auto Bt) {
                constexpr int l = decltype(L)::value, b = decltype(Bt)::value;
                const bool in = kt < KT;
                if constexpr (l < 4) {
                    constexpr int j = l >> 1, ks = l & 1;
                    const unsigned off = in ? lane_off + (unsigned)kt * B_BYTES : kWPast;
                    w[b][j][ks] = __builtin_bit_cast(
                        bf16x8, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, off + ks * kFragElems * 2, j * JB, kAux));
                } else {
                    constexpr int i = l - 4;
                    const unsigned off = in ? offA[i] + (unsigned)kt * ROW_BYTES : kAPast;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(
                        a_rsrc,
                        (__attribute__((address_space(3))) void*)(smem + b * STAGE + (wave + i * NW) * 1024), 16,
                        off, 0, 0, 0);
                }
            };
            // the first k-tiles are requested before the accumulators are cleared
            static_for<D - 1>([&](auto Bt) {
                static_for<NB>([&](auto L) { load_n(L, decltype(Bt)::value, Bt); });
            });
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM_MAX; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int l16 = lane_p & 15, g16 = lane_p >> 4;
            const int sw = swz(l16);  // rows differ by multiples of 16 -> same swizzle
            unsigned a_lane[2][2];    // [step][lower 64 KiB of the stages, upper]: the read's offset field holds 16 bits
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                a_lane[ks][0] = lds_base + (unsigned)(l16 * ROW_BYTES + (((ks * 4 + g16) ^ sw) * 16));
                a_lane[ks][1] = a_lane[ks][0] + 0x10000;
            }
            auto read_frag = [&](auto F, auto Bt) {
                constexpr int f = decltype(F)::value;
                constexpr int at = decltype(Bt)::value * STAGE + (f % TM) * 16 * ROW_BYTES;
                lds_read_b128<(at & 0xffff)>(af[f % R], a_lane[f / TM][at >> 16]);
            };
            wait_vmcnt<NB*(D - 2)>();  // k-tile 0 has landed
            __builtin_amdgcn_s_barrier();
            if constexpr (LINK == kMakesRows)  // every wavefront's results have
                if (wave == 0 && told_expert >= 0) tell_rows(left, told_expert, told_rows);
            static_for<R>([&](auto F) { read_frag(F, std::integral_constant<int, 0>{}); });
            // k-tile kt in buffers U; LOAD: k-tile kt + D - 1 is asked for meanwhile
            auto body = [&](int kt, auto U, auto load_tag) {
                constexpr bool LOAD = decltype(load_tag)::value;
                constexpr int u = decltype(U)::value;
                constexpr std::integral_constant<int, (u + 1) % D> next{};
                constexpr std::integral_constant<int, (u + D - 1) % D> far{};
                static_for<NF>([&](auto F) {
                    constexpr int f = decltype(F)::value;
                    constexpr int i = f % TM, ks = f / TM;
                    if constexpr (f == H) {
                        lds_wait<0>();
                        // k-tile kt + 1 has landed: newer are those up to kt + D - 1, or in the closing ones
                        // of the entry (k-tiles 0 .. D - 2 of the buffers) those up to the last that was asked for
                        if constexpr (LOAD) wait_vmcnt<NB*(D - 2)>();
                        else wait_vmcnt<NB*(u < D - 2 ? D - 3 - u : 0)>();
                        __builtin_amdgcn_s_barrier();
                        static_for<R / 2>([&](auto G) { read_frag(G, next); });
                    } else if constexpr (f < H) {
                        lds_wait<(f <= NF - R ? R - 1 : NF - 1 - f)>();  // fragment f has landed
                    }
                    lds_landed(af[f % R]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][j][ks], af[f % R], acc[i][j], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (f + R < NF) read_frag(std::integral_constant<int, f + R>{}, U);
                    else if constexpr (f >= H) read_frag(std::integral_constant<int, f - H + R / 2>{}, next);
                    constexpr int l0 = f < H ? f * NB / H : NB, l1 = f < H ? (f + 1) * NB / H : NB;
                    if constexpr (LOAD)
                        static_for<l1 - l0>([&](auto X) {
                            load_n(std::integral_constant<int, l0 + decltype(X)::value>{}, kt + D - 1, far);
                        });
                    __builtin_amdgcn_sched_barrier(0);
                });
            };
            int kt = 0;
            const int claim_kt = wave == 0 ? (KT >= 3 * D ? (KT / D - 3) * D : 0) : -1;
            for (; kt + D <= KT; kt += D) {
                if (kt == claim_kt) {
                    ahead_q = next_counter();
                    if (ahead_q >= 0) ahead_pending = claim_from(ahead_q);
                }
                static_for<D>([&](auto U) { body(kt + decltype(U)::value, U, std::true_type{}); });
            }
            static_for<D - 1>([&](auto U) {
                if (kt + decltype(U)::value < KT) body(kt, U, std::false_type{});
            });
            // (the last hand-over read fragments that nobody multiplies)
            lds_wait<0>();
#pragma unroll
            for (int r = 0; r < R; ++r) lds_landed(af[r]);
        };
        // one K loop per 32 rows of height; every one runs the same barriers
        const bool once = past_caches && mt.part == kPartAlone;
        static_for<TM_MAX / 2>([&](auto H2) {
            constexpr int tm = 2 * decltype(H2)::value + 2;
            const std::integral_constant<int, tm> TM{};
            if (mt.rows > 16 * (tm - 2) && mt.rows <= 16 * tm) {
                if (once) k_loop(TM, std::true_type{});
                else k_loop(TM, std::false_type{});
            }
        });
        // every wavefront has read next_tile (the K loop holds a barrier)
        if (wave == 0) next_tile = settle_claim(ahead_q, __builtin_amdgcn_readfirstlane(ahead_pending));

        // Epilogue.  Rounded to bf16 a lane holds 8 bytes of a row per 16 x 16 tile.  Two tiles are regrouped
        // with the two lane-swap instructions (quarter q of the wavefront = lanes 16q .. 16q+15):
        // swapping the upper half of the first tile's register with the lower half of the second's, then
        // the odd quarters of the first with the even quarters of the second, leaves a lane with 16 bytes of one row, half
        // as many store instructions.  The two tiles are the two column groups of a row group (64-byte
        // pieces: quarter q holds columns 8q .. 8q+7 of the 32), or with SwiGLU, which makes one tile of
        // the two, two row groups (32-byte pieces: quarters 0 and 1 the two halves of the first group's
        // rows, 2 and 3 of the second's).
        const int lane_e = opaque(lane);
        const int l16e = lane_e & 15, g16e = lane_e >> 4;
        auto store_pair = [&](const float (&v0)[4], const float (&v1)[4], bf16_t* at, bool on) {
            unsigned px = pack_bf16x2(v0[0], v0[1]), py = pack_bf16x2(v0[2], v0[3]);
            unsigned qx = pack_bf16x2(v1[0], v1[1]), qy = pack_bf16x2(v1[2], v1[3]);
            lane_swap_pairs(px, qx);
            lane_swap_pairs(py, qy);
            if constexpr (LINK == kMakesRows) {
                // to memory, not to this XCD's L2 alone
                const u32x4 v = {px, py, qx, qy};
                const bf16_t* base = C + (size_t)mt.list0 * ldc;
                const auto c_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00027000);
                if (on)
                    __builtin_amdgcn_raw_buffer_store_b128(v, c_rsrc, (unsigned)((const char*)at - (const char*)base), 0,
                                                           kThrough);
            } else if (on) {
                *(uint4*)at = make_uint4(px, py, qx, qy);
            }
        };
        if constexpr (SWIGLU) {
            const int col = n0 / 2 + (wave >> 1) * 32 + (wave & 1) * 16 + (g16e & 1) * 8;
#pragma unroll
            for (int i = 0; i < TM_MAX; i += 2) {
                if (i * 16 < mt.rows) {
                    float v[2][4];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[h][c] = silu_f(acc[i + h][0][c]) * acc[i + h][1][c];
                    const int row = (i + (g16e >> 1)) * 16 + l16e;
                    store_pair(v[0], v[1], C + (size_t)(mt.list0 + row) * ldc + col, row < mt.rows && col < N / 2);
                }
            }
        } else {
            const int col0 = n0 + wave * 32;  // (N is a multiple of 64: the wavefront's columns exist or not together)
            float* slab = nullptr;
            if constexpr (EPI == kEpiNone && LINK == kAlone)
                if (mt.part >= 0) slab = partials + (size_t)mt.part * kPartRows * N;
            if (slab) {
#pragma unroll
                for (int i = 0; i < TM_MAX; ++i) {
                    const int row = i * 16 + l16e;
                    if (i * 16 < mt.rows && row < mt.rows && col0 < N) {
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            *(f32x4*)(slab + (size_t)row * N + col0 + j * 16 + g16e * 4) = acc[i][j];
                    }
                }
            } else {
                // output row and scale of this lane's rows, fetched eight at a time (one by one each
                // would wait out a memory round trip, and with it the stores of the row before)
#pragma unroll
                for (int i0 = 0; i0 < TM_MAX; i0 += 8) {
                    if (i0 * 16 < mt.rows) {
                        int crow_of[8];
                        float sc_of[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int row = (i0 + i) * 16 + l16e;
                            crow_of[i] = mt.list0 + (row < mt.rows ? row : mt.rows - 1);
                            sc_of[i] = 1.0f;
                        }
                        if constexpr (EPI == kEpiNone) {
                            if (rm.c_rows) {
#pragma unroll
                                for (int i = 0; i < 8; ++i) crow_of[i] = rm.c_rows[crow_of[i]];
                            }
                            if (rm.scale) {
                                int si[8];
#pragma unroll
                                for (int i = 0; i < 8; ++i) si[i] = rm.scale_idx[crow_of[i]];
#pragma unroll
                                for (int i = 0; i < 8; ++i) sc_of[i] = rm.scale[si[i]];
                            }
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            if ((i0 + i) * 16 >= mt.rows) continue;
                            float v[2][4];
#pragma unroll
                            for (int j = 0; j < 2; ++j)
#pragma unroll
                                for (int c = 0; c < 4; ++c) {
                                    const float a = acc[i0 + i][j][c];
                                    v[j][c] = EPI == kEpiRelu ? fmaxf(a, 0.f) : a * sc_of[i];
                                }
                            store_pair(v[0], v[1], C + (size_t)crow_of[i] * ldc + col0 + g16e * 8,
                                       (i0 + i) * 16 + l16e < mt.rows && col0 < N);
                        }
                    }
                }
            }
        }
        if constexpr (EPI != kEpiNone)
            if (copy_n > 0) store_pieces(copy, copy_first, copy_n, (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem + kStageLds + wave * (kCopyPieces * kCopyPieceLds));
        if constexpr (LINK == kMakesRows) {
            told_expert = mt.expert;
            told_rows = mt.rows;
        }
    }
    if constexpr (LINK == kMakesRows) {
        rows_stored();
        __builtin_amdgcn_s_barrier();
        if (wave == 0 && told_expert >= 0) tell_rows(left, told_expert, told_rows);
    }
}

template <int EPI>
__global__ __launch_bounds__(512, 2) void grouped_gemm_tile_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ Bp, size_t b_stride, bf16_t* __restrict__ C, int ldc,
    const MTile* __restrict__ mtiles, const int32_t* __restrict__ counts, int32_t* __restrict__ queues, int N, int K,
    int group_n, bool past_caches, RowMap rm, float* __restrict__ partials, RowCopy copy) {
    tile_product<EPI, kAlone>(A, lda, Bp, b_stride, C, ldc, mtiles, counts, queues, N, K, group_n, past_caches, rm, partials,
                              copy, nullptr);
}

// Both products in one launch.
template <int EPI>
__global__ __launch_bounds__(512, 2) void grouped_ffn_tiles_kernel(
    const bf16_t* __restrict__ X, int d, const bf16_t* __restrict__ P13, size_t stride1, const bf16_t* __restrict__ P2,
    size_t stride2, bf16_t* h, int fp, bf16_t* __restrict__ Y, const MTile* __restrict__ tiles1,
    const MTile* __restrict__ tiles2, const int32_t* __restrict__ counts1, const int32_t* __restrict__ counts2,
    int32_t* __restrict__ queues, bool past_caches1, bool past_caches2, RowMap rm1, RowMap rm2, RowCopy copy,
    int32_t* left) {
    tile_product<EPI, kMakesRows>(X, d, P13, stride1, h, fp, tiles1, counts1, queues, EPI == kEpiSwiglu ? 2 * fp : fp, d,
                                  kTileGroup, past_caches1, rm1, nullptr, copy, left);
    if (counts1[kCntEntries] == 0) return;  // (the first table did not fit: its tiles are not made, waiting for them would not end)
    tile_product<kEpiNone, kWantsRows>(h, fp, P2, stride2, Y, d, tiles2, counts2, queues + 8, d, fp, kTileGroup, past_caches2,
                                       rm2, nullptr, RowCopy{}, left);
}
