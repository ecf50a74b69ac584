// Weight-streaming forms of the grouped bf16 GEMM, for batches of a few rows per expert, where
// a product is bound by how fast the weights of the experts with rows arrive from memory.
// Included by grouped_ffn.hip inside namespace moegps (uses its types).
//
// Both forms load weight fragments from memory straight into registers (a fragment of the packed
// form is one contiguous kilobyte, so nothing is gained by a detour through LDS).  A wavefront asks for
// one k-tile of its columns at a time and eight to sixteen of them share a CU: two workgroups of
// eight with form 2 and with form 1's units of 32 columns, two of four or one of eight with its
// units of 64 (the registers of the 64-row body decide), so that except for the last a unit's
// prologue, exchange and stores run under the loads of another workgroup.  Asking two or three k-tiles
// ahead per wavefront was no faster.  The grid walks
// units (M-tile of up to 64 rows) x (32 .. 128 columns) with a fixed stride: units are short
// (0.1 - 1 MB of weights) and a workgroup that is left alone at the end gets the bandwidth of
// the ones that have finished.
//
// Against the LDS-staged 128- and 32-row tiles (whose waves all wait at one barrier per k-tile
// and whose 2 MiB tiles leave most CUs idle in the last round), both products of bench.py's batches:
// 4096 x 1536 experts, top-8 of 128 (cfg5_decode_m1, --tokens): 1 token (8 experts) 99 -> 55 us (5.5 TB/s of
// weights), 16 tokens (54) 382 -> 325 us (6.3 TB/s), 128 tokens (85) 569 -> 503 us (6.4 TB/s), 256 tokens (91)
// 638 -> 587 us (5.9 TB/s); 4096 x 14336 experts, top-2 of 8 (cfg2_mixtral_dist): 16 tokens 369 -> 280 us, 64
// tokens 421 -> 340 us (6.3 TB/s both).
#pragma once

// Form 1: the wavefronts of a workgroup share the unit's columns and split K between them; each
// reads its own activation fragments (16 rows x 64 bytes per load, from the L2) and nothing
// synchronises until the fp32 sums are added up through LDS, wavefront 0 first, so the result does
// not depend on timing.  The finest units, so it is the form for few experts and small
// batches; in others its activation loads, repeated for every 64 columns, cost more than form 2's
// barrier (stream_form).
//   NT  16-column groups per unit: 4, or 2 where the product has too few units
//   NW  wavefronts per workgroup = parts of K: 8, or 4 for short K
template <int NT, int NW, int EPI>
__global__ __launch_bounds__(NW * 64) void grouped_gemm_stream_ksplit_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ Bp, size_t b_stride, bf16_t* __restrict__ C,
    int ldc, const MTile* __restrict__ mtiles, const int32_t* __restrict__ counts, int N, int K, RowMap rm,
    int grid, RowCopy copy) {  // workgroups of the product; ahead of them those of the copy
    constexpr bool SWIGLU = EPI == kEpiSwiglu;
    constexpr int UC = NT * 16;     // packed columns of a unit
    constexpr int PITCH = UC + 4;   // floats per row of the exchange
    // 16-row groups of the packed matrix a unit reads: NT neighbours; with SwiGLU and NT = 2 a gate
    // group and its up group, two further
    constexpr int JSTEP = (SWIGLU && NT == 2) ? 2 : 1;
    static_assert(NT == 2 || NT == 4, "a unit lies inside 64 packed columns");
    __shared__ __align__(16) float xch[NW * 16 * PITCH];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g16 = lane >> 4;
    const int n_units = N / UC;     // N is a multiple of 64
    const int total = counts[kCntEntries] * n_units;
    const int KT = K / kPackK;
    const int kt0 = KT * wave / NW, nk = KT * (wave + 1) / NW - kt0;

    if constexpr (EPI != kEpiNone)
        if (blockIdx.x < gridDim.x - grid) {
            copy_part(copy, (int)blockIdx.x * NW + wave);
            return;
        }
    for (int u = (int)blockIdx.x - (int)(gridDim.x - grid); u < total; u += grid) {
        const int entry = u / n_units, nu = u - entry * n_units;
        const MTile mt = mtiles[entry];
        const int col0 = JSTEP == 2 ? (nu >> 1) * 64 + (nu & 1) * 16 : nu * UC;
        const bf16_t* Bb = Bp + (size_t)mt.expert * b_stride +
                           ((size_t)(col0 / kPackN) * KT + kt0) * (kPackN * kPackK) + (col0 % kPackN) * kPackK +
                           lane * 8;
        auto unit = [&](auto MT_tag) {
            constexpr int MT = decltype(MT_tag)::value;  // 16-row groups of the M-tile that hold rows, rounded up
            const bf16_t* arow[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                int r = i * 16 + l16;
                r = mt.list0 + (r < mt.rows ? r : mt.rows - 1);
                if (rm.a_rows) {
                    r = rm.a_rows[r];
                    if (rm.a_rows2) r = rm.a_rows2[r] / rm.a_div;
                }
                arow[i] = A + (size_t)r * lda + kt0 * kPackK + g16 * 8;
            }
            f32x4 acc[MT][NT];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            bf16x8 a[MT][2], b[NT][2];
            auto load = [&](int kt) {
                const bf16_t* p = Bb + (size_t)kt * (kPackN * kPackK);
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)  // weights are read once: past the caches
                        b[j][ks] = __builtin_nontemporal_load((const bf16x8*)(p + (j * JSTEP * 2 + ks) * kFragElems));
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) a[i][ks] = *(const bf16x8*)(arow[i] + kt * kPackK + ks * 32);
            };
            if (nk > 0) load(0);
            for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < NT; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][ks], a[i][ks], acc[i][j], 0, 0, 0);
                load(kt + 1 < nk ? kt + 1 : kt);  // (unconditional, so that the compiler can send it ahead)
            }
            // the parts of K added up, 16 rows at a time
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                __syncthreads();
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    *(f32x4*)&xch[(wave * 16 + l16) * PITCH + j * 16 + g16 * 4] = acc[i][j];
                __syncthreads();
                constexpr int THREADS = NW * 64;
                constexpr int OC = SWIGLU ? UC / 2 : UC;  // output columns
                constexpr int PER = 16 * OC >= 2 * THREADS ? 16 * OC / THREADS : 2;
                constexpr int TPR = OC / PER;              // threads per row
                const int row = tid / TPR, c = (tid % TPR) * PER;
                const int mrow = i * 16 + row;
                if (row < 16 && mrow < mt.rows) {
                    float v[PER], g[PER];
#pragma unroll
                    for (int q = 0; q < PER; ++q) v[q] = g[q] = 0.f;
#pragma unroll
                    for (int w = 0; w < NW; ++w)
#pragma unroll
                        for (int q = 0; q < PER; ++q) {
                            v[q] += xch[(w * 16 + row) * PITCH + c + q];
                            if (SWIGLU) g[q] += xch[(w * 16 + row) * PITCH + c + q + OC];
                        }
                    int crow = mt.list0 + mrow;
                    float sc = 1.f;
                    if (EPI == kEpiNone) {
                        if (rm.c_rows) crow = rm.c_rows[crow];
                        if (rm.scale) sc = rm.scale[rm.scale_idx[crow]];
                    }
                    bf16_t* out = C + (size_t)crow * ldc + nu * OC + c;
#pragma unroll
                    for (int q = 0; q < PER; q += 2) {
#pragma unroll
                        for (int s = q; s < q + 2; ++s)
                            v[s] = SWIGLU ? silu_f(v[s]) * g[s] : EPI == kEpiRelu ? fmaxf(v[s], 0.f) : v[s] * sc;
                        *(unsigned*)(out + q) = pack_bf16x2(v[q], v[q + 1]);
                    }
                }
            }
        };
        if (mt.rows <= 16) unit(std::integral_constant<int, 1>{});
        else if (mt.rows <= 32) unit(std::integral_constant<int, 2>{});
        else unit(std::integral_constant<int, 4>{});
    }
}

// Form 2: a unit is 128 columns; four wavefronts side by side along N take 32 of them each, and two
// such rows of wavefronts take half of K each.  The activation rows of a k-tile are shared: the
// workgroup copies them into LDS (double buffered, one 16-byte piece or two per thread, 128 bytes
// of a row side by side), so the L2 serves them once per 128 columns and not once per 64 and
// wavefront.  One barrier per k-tile; the global loads stay in flight across it.
constexpr int kStreamBM = 64;  // rows of an M-tile of both forms
template <int EPI>
__global__ __launch_bounds__(512, 4) void grouped_gemm_stream_shared_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ Bp, size_t b_stride, bf16_t* __restrict__ C,
    int ldc, const MTile* __restrict__ mtiles, const int32_t* __restrict__ counts, int N, int K, RowMap rm,
    int grid, RowCopy copy) {  // workgroups of the product; behind them those of the copy
    constexpr bool SWIGLU = EPI == kEpiSwiglu;
    constexpr int BM = kStreamBM, NT = 2, KS = 2, NWN = 4;
    constexpr int UC = NT * 16 * NWN;        // packed columns of a unit
    constexpr int JSTEP = SWIGLU ? 2 : 1;    // gate group and up group of one wavefront are two groups apart
    constexpr int ROW = kPackK * 2;          // bytes of a row of a k-tile
    constexpr int PART = BM * ROW;    // one half's rows of a k-tile
    constexpr int PITCH = NT * 16 + 4;
    typedef __attribute__((__vector_size__(16))) unsigned u32x4;
    __shared__ __align__(16) unsigned char abuf[2][KS * PART];
    static_assert(sizeof(abuf) >= NWN * 16 * PITCH * sizeof(float), "the exchange reuses the activation buffers");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % NWN, wk = wave / NWN;  // its columns, its half of K
    const int l16 = lane & 15, g16 = lane >> 4;
    const int n_units = (N + UC - 1) / UC;
    const int total = counts[kCntEntries] * n_units;
    const int KT = K / kPackK, kh = (KT + 1) / 2;  // k-tiles; of the first half
    const int my_kt = wk == 0 ? kh : KT - kh;

    // An expert's M-tiles follow each other under the same columns, and unit numbers are dealt in
    // chunks of 16 to the 8 XCDs (workgroup b runs on XCD b % 8; the launch is a multiple of 128
    // workgroups), so that the M-tiles of an expert run side by side behind one L2 and share its
    // weights there (popularity 0.1, 128 experts, 256 tokens, 35 of them with 58 rows on average:
    // 345 -> 284 us).
    if constexpr (EPI != kEpiNone)
        if ((int)blockIdx.x >= grid) {
            copy_part(copy, ((int)blockIdx.x - grid) * (NWN * KS) + wave);
            return;
        }
    const int slot = blockIdx.x >> 3;
    for (int u = ((slot >> 4) * 8 + (blockIdx.x & 7)) * 16 + (slot & 15); u < total; u += grid) {
        int entry = u / n_units, nu = u - entry * n_units;
        MTile mt = mtiles[entry];
        if (mt.n_same > 1) {
            const int v = u - mt.first * n_units;
            nu = v / mt.n_same;
            mt = mtiles[mt.first + v % mt.n_same];
        }
        // first packed column of this wavefront (N is a multiple of 64: the last unit may be half empty)
        const int col0 = nu * UC + (SWIGLU ? (wn >> 1) * 64 + (wn & 1) * 16 : wn * NT * 16);
        const bool live = col0 < N;
        const int colr = live ? col0 : 0;
        const bf16_t* Bb = Bp + (size_t)mt.expert * b_stride +
                           ((size_t)(colr / kPackN) * KT + wk * kh) * (kPackN * kPackK) + (colr % kPackN) * kPackK +
                           lane * 8;
        // SHARED: other M-tiles of the expert want the same weights; else they are read once, past
        // the caches (8 % faster)
        auto unit = [&](auto MT_tag, auto shared_tag) {
            constexpr int MT = decltype(MT_tag)::value;
            constexpr bool SHARED = decltype(shared_tag)::value;
            constexpr int PIECES = KS * MT * 16 * (ROW / 16);
            constexpr int PA = (PIECES + 511) / 512;  // 16-byte pieces of activations per thread and k-tile
            const bf16_t* src[PA];
            unsigned dst[PA];
            int last[PA];                             // last k-tile of the piece's half
            bool on[PA];
            static_for<PA>([&](auto I) {
                constexpr int i = decltype(I)::value;
                const int p = tid + i * 512;
                on[i] = p < PIECES;
                const int half = on[i] ? p / (PIECES / KS) : 0, row = (p >> 3) % (MT * 16), slot = p & 7;
                int r = mt.list0 + (row < mt.rows ? row : mt.rows - 1);
                if (rm.a_rows) {
                    r = rm.a_rows[r];
                    if (rm.a_rows2) r = rm.a_rows2[r] / rm.a_div;
                }
                src[i] = A + (size_t)r * lda + (half == 1 && KT > kh ? kh * kPackK : 0) + slot * 8;
                dst[i] = half * PART + row * ROW + ((slot ^ swz(row)) * 16);
                last[i] = (half == 0 ? kh : KT - kh) - 1;
            });
            f32x4 acc[MT][NT];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            bf16x8 b[NT][2];
            u32x4 areg[PA];
            auto load_b = [&](int kt) {
                if (kt >= my_kt) return;
                const bf16_t* p = Bb + (size_t)kt * (kPackN * kPackK);
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
                        if (SHARED) b[j][ks] = *(const bf16x8*)(p + (j * JSTEP * 2 + ks) * kFragElems);
                        else b[j][ks] = __builtin_nontemporal_load((const bf16x8*)(p + (j * JSTEP * 2 + ks) * kFragElems));
            };
            auto load_a = [&](int kt) {  // (the shorter half repeats its last k-tile, which nobody multiplies then)
                static_for<PA>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    const int k = kt < last[i] ? kt : (last[i] > 0 ? last[i] : 0);
                    if (on[i]) areg[i] = *(const u32x4*)(src[i] + k * kPackK);
                });
            };
            auto put_a = [&](int buf) {
                static_for<PA>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    if (PIECES % 512 == 0 || on[i]) *(u32x4*)&abuf[buf][dst[i]] = areg[i];
                });
            };
            load_a(0);
            load_b(0);
            put_a(0);
            if (kh > 1) load_a(1);
            __syncthreads();
            for (int kt = 0; kt < kh; ++kt) {
                const unsigned char* ab = abuf[kt & 1] + wk * PART;
                bf16x8 af[MT][2];
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
                        af[i][ks] = *(const bf16x8*)(ab + (i * 16 + l16) * ROW + (((ks * 4 + g16) ^ swz(l16)) * 16));
                if (kt < my_kt)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int i = 0; i < MT; ++i)
#pragma unroll
                            for (int j = 0; j < NT; ++j)
                                acc[i][j] =
                                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][ks], af[i][ks], acc[i][j], 0, 0, 0);
                if (kt + 1 < kh) {
                    put_a((kt + 1) & 1);
                    if (kt + 2 < kh) load_a(kt + 2);
                    load_b(kt + 1);
                }
                // own LDS traffic done, then everybody's: k-tile kt + 1 is in its buffer, and the buffer
                // of k-tile kt may be written (by the put after next barrier's reads)
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
            // the second half's sums added to the first's, 16 rows at a time
            float* xch = (float*)&abuf[0][0];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (wk == 1)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        *(f32x4*)&xch[(wn * 16 + l16) * PITCH + j * 16 + g16 * 4] = acc[i][j];
                __syncthreads();
                if (wk == 0)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[i][j] += *(const f32x4*)&xch[(wn * 16 + l16) * PITCH + j * 16 + g16 * 4];
                __syncthreads();
            }
            if (wk == 0 && live) {
                const int oc0 = SWIGLU ? nu * (UC / 2) + (wn >> 1) * 32 + (wn & 1) * 16 : col0;
#pragma unroll
                for (int i = 0; i < MT; ++i) {
                    const int row = i * 16 + l16;
                    if (row >= mt.rows) continue;
                    int crow = mt.list0 + row;
                    float sc = 1.f;
                    if (EPI == kEpiNone) {
                        if (rm.c_rows) crow = rm.c_rows[crow];
                        if (rm.scale) sc = rm.scale[rm.scale_idx[crow]];
                    }
                    bf16_t* out = C + (size_t)crow * ldc + oc0 + g16 * 4;
#pragma unroll
                    for (int j = 0; j < (SWIGLU ? 1 : NT); ++j) {
                        float v[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            v[q] = SWIGLU ? silu_f(acc[i][0][q]) * acc[i][1][q]
                                          : EPI == kEpiRelu ? fmaxf(acc[i][j][q], 0.f) : acc[i][j][q] * sc;
                        uint2 w;
                        w.x = pack_bf16x2(v[0], v[1]);
                        w.y = pack_bf16x2(v[2], v[3]);
                        *(uint2*)(out + j * 16) = w;
                    }
                }
            }
        };
        if (mt.n_same > 1) unit(std::integral_constant<int, 4>{}, std::true_type{});
        else if (mt.rows <= 16) unit(std::integral_constant<int, 1>{}, std::false_type{});
        else if (mt.rows <= 32) unit(std::integral_constant<int, 2>{}, std::false_type{});
        else unit(std::integral_constant<int, 4>{}, std::false_type{});
    }
}
