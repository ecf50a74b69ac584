// Expert duplication planner: Algorithm 1 (Section 3.1) in count-based form, run
// by one 64-wide wavefront.  Two versions: state in registers, one lane per rank
// (G <= 64, further down), and state in LDS for any G (first).  The loop is inherently serial
// (each move changes the loads the next one looks at); inside one iteration the
// wavefront evaluates every candidate cold rank in parallel and a cross-lane
// arg-min picks the coldest feasible one, which is exactly the candidate the
// serial scan "coldest rank first, hottest expert first" would reach first.
//
// State per slot sigma = g*S + s: hosted expert (-1 = empty) and planned rows.
// Ties (hottest rank, coldest rank, hottest expert) go to the lowest index.
#include "common.h"

namespace moegps {

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        unsigned long long o = __shfl_xor(v, m, kWave);
        v = o > v ? o : v;
    }
    return v;
}
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        unsigned long long o = __shfl_xor(v, m, kWave);
        v = o < v ? o : v;
    }
    return v;
}

__global__ __launch_bounds__(kWave) void plan_kernel(int mode, const int32_t* __restrict__ hist_pred, int E, int G,
                                                     int S, int c_max, int32_t* __restrict__ slot_expert,
                                                     int32_t* __restrict__ slot_quota,
                                                     int32_t* __restrict__ rank_load_pred,
                                                     int32_t* __restrict__ n_iters_out) {
    __shared__ int se[MOE_MAX_SEGMENTS];   // expert per slot
    __shared__ int q[MOE_MAX_SEGMENTS];    // planned rows per slot
    __shared__ int L[MOE_MAX_RANKS];       // planned rows per rank
    __shared__ int copies[MOE_MAX_EXPERTS];
    __shared__ int hot_ord[MOE_MAX_SLOTS];  // slots of the hot rank, hottest expert first
    __shared__ int n_hot_s;

    const int lane = threadIdx.x;
    const int nseg = G * S;
    const int H = (E + G - 1) / G;

    for (int s = lane; s < nseg; s += kWave) {
        se[s] = -1;
        q[s] = 0;
    }
    __syncthreads();
    // home placement; every predicted token starts on the only host of its expert
    for (int e = lane; e < E; e += kWave) {
        const int sigma = (e / H) * S + (e % H);
        se[sigma] = e;
        int n = hist_pred[e];
        q[sigma] = n > 0 ? n : 0;
        copies[e] = 1;
    }
    __syncthreads();
    for (int g = lane; g < G; g += kWave) {
        int sum = 0;
        for (int s = 0; s < S; ++s) sum += q[g * S + s];
        L[g] = sum;
    }
    __syncthreads();

    int n_iters = 0;
    if (mode != MOE_MODE_NONE) {
        const int i_max = 16 * nseg;
        while (n_iters < i_max) {
            // hottest rank (ties -> lowest g) and the smallest load
            unsigned long long kmax = 0ull, kmin = ~0ull;
            for (int g = lane; g < G; g += kWave) {
                const unsigned long long l = (unsigned long long)(unsigned)L[g];
                const unsigned long long hi = (l << 32) | (unsigned)(0xffffffffu - (unsigned)g);
                const unsigned long long lo = (l << 32) | (unsigned)g;
                kmax = hi > kmax ? hi : kmax;
                kmin = lo < kmin ? lo : kmin;
            }
            kmax = wave_max_u64(kmax);
            kmin = wave_min_u64(kmin);
            const int g_h = (int)(0xffffffffu - (unsigned)(kmax & 0xffffffffull));
            const int L_h = (int)(kmax >> 32);
            const int L_min = (int)(kmin >> 32);
            if (L_h - L_min <= 1) break;  // loop guard of Algorithm 1

            // slots of g_h with tokens, ordered by (rows descending, slot ascending)
            if (lane == 0) n_hot_s = 0;
            __syncthreads();
            if (lane < S) {
                const int mine = q[g_h * S + lane];
                if (mine > 0) {
                    int r = 0;
                    for (int s = 0; s < S; ++s) {
                        const int o = q[g_h * S + s];
                        if (o > mine || (o == mine && s < lane)) ++r;
                    }
                    hot_ord[r] = lane;
                    atomicAdd(&n_hot_s, 1);
                }
            }
            __syncthreads();
            const int n_hot = n_hot_s;

            // every lane tries cold ranks g_c = lane, lane+64, ...; for each it takes
            // the first feasible slot of g_h in hot order
            unsigned long long best = ~0ull;  // (L_c, g_c) packed, smaller is colder
            int best_s = -1, best_sp = -1, best_new = 0;
            for (int g_c = lane; g_c < G; g_c += kWave) {
                if (g_c == g_h) continue;
                const int L_c = L[g_c];
                if (L_h - L_c <= 1) continue;
                int f_s = -1, f_sp = -1, f_new = 0;
                for (int r = 0; r < n_hot && f_s < 0; ++r) {
                    const int s = hot_ord[r];
                    const int e = se[g_h * S + s];
                    int host = -1, empty = -1;
                    for (int sp = S - 1; sp >= 0; --sp) {
                        const int o = se[g_c * S + sp];
                        if (o == e) host = sp;
                        if (o < 0) empty = sp;
                    }
                    if (host >= 0) {
                        f_s = s;
                        f_sp = host;
                        f_new = 0;
                    } else if (copies[e] < c_max && empty >= 0) {
                        f_s = s;
                        f_sp = empty;
                        f_new = 1;
                    }
                }
                if (f_s >= 0) {
                    const unsigned long long key = ((unsigned long long)(unsigned)L_c << 32) | (unsigned)g_c;
                    if (key < best) {
                        best = key;
                        best_s = f_s;
                        best_sp = f_sp;
                        best_new = f_new;
                    }
                }
            }
            const unsigned long long win = wave_min_u64(best);
            if (win == ~0ull) break;  // nothing feasible
            // the lane that holds the winner applies the move
            if (best == win) {
                const int g_c = (int)(win & 0xffffffffull);
                const int L_c = (int)(win >> 32);
                const int from = g_h * S + best_s;
                const int to = g_c * S + best_sp;
                const int e = se[from];
                if (best_new) {  // copy weights of e* on g_c
                    se[to] = e;
                    copies[e] += 1;
                }
                const int delta = (L_h - L_c + 1) / 2;  // ceil((L_h - L_c) / 2)
                const int m = delta < q[from] ? delta : q[from];
                q[from] -= m;
                q[to] += m;
                L[g_h] = L_h - m;
                L[g_c] = L_c + m;
            }
            __syncthreads();
            ++n_iters;
        }
    }
    __syncthreads();
    for (int s = lane; s < nseg; s += kWave) {
        slot_expert[s] = se[s];
        slot_quota[s] = q[s];
    }
    for (int g = lane; g < G; g += kWave) rank_load_pred[g] = L[g];
    if (lane == 0) n_iters_out[0] = n_iters;
}

// ---------------------------------------------------------------------------
// Register-resident version for G <= 64: lane g owns rank g (its load and its S
// slots live in registers; the copy count of an expert is a ballot over the lanes).  One iteration
// is a few DPP reductions, ballots and lane reads; there is no barrier.  The loop is one wavefront
// running instructions one after the other (5-8 cycles each), so what counts is how many there
// are.  An iteration first looks at the pair the serial scan of Algorithm 1 starts with, the
// hottest expert of the hottest rank and the coldest rank: O(S) instructions.  Only if that
// move is infeasible every rank looks at every slot of the hot rank, O(S^2): the
// candidate a lane proposes is its first feasible slot of the hot rank in (rows
// descending, slot ascending) order; the coldest proposing lane wins, which is the
// candidate the serial scan (with the fall-through order of the header) reaches first.
// A copy goes into the lowest empty slot and home slots are the lowest, so the occupied slots of
// a rank are always a prefix and one counter stands for them.
// Per call against looking at every slot for every rank each time (and reductions whose lane
// permutes did not fold into the max): 8 ranks of 2 slots, 15 moves 10.5 -> 8.4 us; 32 of 5, 40 moves
// 38.3 -> 31.0, 70 moves 69 -> 58; 16 of 5, 33 moves 34.4 -> 27.7; 8 of 10, 28 moves 47.4 -> 33.2.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int dpp_max_step(int v, int o) { return o > v ? o : v; }
__device__ __forceinline__ int dpp_min_step(int v, int o) { return o < v ? o : v; }

// Reductions over the first ROWS rows of 16 lanes (the lanes that hold ranks; those without one hold
// neutral values): inside a row by DPP lane permutes, which fold into the max or min that takes
// them, the rows by lane reads.  Every lane must be active.
template <bool IS_MAX>
__device__ __forceinline__ int row_reduce_step(int v, int level) {
    const int o = level == 0   ? __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true)    // quad_perm [1,0,3,2]
                  : level == 1 ? __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true)    // quad_perm [2,3,0,1]
                  : level == 2 ? __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true)   // row_half_mirror
                               : __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true);  // row_mirror
    return IS_MAX ? dpp_max_step(v, o) : dpp_min_step(v, o);
}
template <bool IS_MAX, int ROWS>
__device__ __forceinline__ int rows_reduce(int v) {
    int r = __builtin_amdgcn_readlane(v, 0);
#pragma unroll
    for (int i = 1; i < ROWS; ++i) {
        const int o = __builtin_amdgcn_readlane(v, 16 * i);
        r = IS_MAX ? dpp_max_step(r, o) : dpp_min_step(r, o);
    }
    return __builtin_amdgcn_readfirstlane(r);
}
template <int ROWS>
__device__ __forceinline__ int wave_min_i32(int v) {
#pragma unroll
    for (int l = 0; l < 4; ++l) v = row_reduce_step<false>(v, l);
    return rows_reduce<false, ROWS>(v);
}
// maximum of a and minimum of b, step by step side by side
template <int ROWS>
__device__ __forceinline__ void wave_max_min_i32(int a, int b, int& mx, int& mn) {
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        a = row_reduce_step<true>(a, l);
        b = row_reduce_step<false>(b, l);
    }
    mx = rows_reduce<true, ROWS>(a);
    mn = rows_reduce<false, ROWS>(b);
}

template <int SMAX, int ROWS>
__global__ __launch_bounds__(kWave) void plan_kernel_regs(int mode, const int32_t* __restrict__ hist_pred, int E,
                                                          int G, int S, int c_max,
                                                          int32_t* __restrict__ slot_expert,
                                                          int32_t* __restrict__ slot_quota,
                                                          int32_t* __restrict__ rank_load_pred,
                                                          int32_t* __restrict__ n_iters_out) {
    const int lane = threadIdx.x;
    const bool valid = lane < G;
    const int H = (E + G - 1) / G;
    constexpr int NONE = -2;  // slot index >= S: neither empty nor an expert
    const int IMAX = 0x7fffffff;

    // slot of rank g that hosts expert e (one byte each), kNoHost: none
    constexpr int kNoHost = 255;
    __shared__ __align__(16) unsigned char host_of[MOE_MAX_EXPERTS * kWave];
    if (mode != MOE_MODE_NONE) {
        for (int i = lane * 16; i < E * kWave; i += kWave * 16)
            *(uint4*)&host_of[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
        __syncthreads();
    }
    int se[SMAX], q[SMAX];
    int L = 0, occupied = 0;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
        const int e = lane * H + s;
        const bool home = valid && s < H && e < E;
        se[s] = home ? e : (s < S ? -1 : NONE);
        occupied += home ? 1 : 0;
        if (home && mode != MOE_MODE_NONE) host_of[e * kWave + lane] = (unsigned char)s;
        int n = home ? hist_pred[e] : 0;
        q[s] = n > 0 ? n : 0;
        L += q[s];
    }

    int n_iters = 0;
    if (mode != MOE_MODE_NONE) {
        const int i_max = 16 * G * S;
        const unsigned long long ranks = G < kWave ? (1ull << G) - 1ull : ~0ull;  // lanes that hold a rank
        while (n_iters < i_max) {
            int L_h, L_min;
            wave_max_min_i32<ROWS>(valid ? L : -1, valid ? L : IMAX, L_h, L_min);
            if (L_h - L_min <= 1) break;  // loop guard of Algorithm 1
            // hottest and coldest rank, ties -> lowest g
            const int g_h = __builtin_ctzll(__ballot(L == L_h) & ranks);
            int g_c = __builtin_ctzll(__ballot(L == L_min) & ranks);
            int L_c = L_min;

            // hottest expert of every rank (equal rows keep the lower slot); the hot rank's is wanted
            int top_q = q[0];
#pragma unroll
            for (int t = 1; t < SMAX; ++t) top_q = q[t] > top_q ? q[t] : top_q;
            int top_s = 0, top_e = se[0];
#pragma unroll
            for (int t = SMAX - 1; t >= 0; --t) {
                top_s = q[t] == top_q ? t : top_s;
                top_e = q[t] == top_q ? se[t] : top_e;
            }
            int q_sel = __builtin_amdgcn_readlane(top_q, g_h);
            int s_sel = __builtin_amdgcn_readlane(top_s, g_h);
            int e_sel = __builtin_amdgcn_readlane(top_e, g_h);
            int host = -1;
#pragma unroll
            for (int t = SMAX - 1; t >= 0; --t) host = se[t] == e_sel ? t : host;
            // every rank hosts an expert at most once: copies = number of hosting lanes
            const int copies = __popcll((unsigned long long)__ballot(host >= 0));
            int sp_sel = __builtin_amdgcn_readlane(host, g_c);
            bool feasible = sp_sel >= 0;
            if (!feasible) {
                sp_sel = __builtin_amdgcn_readlane(occupied, g_c);
                feasible = copies < c_max && sp_sel < S;
            }
            if (!feasible) {
                // per slot of the hot rank: which ranks host its expert (one byte per rank and expert in
                // LDS, all slots' reads under way together) or have room for a copy
                int hq[SMAX], he[SMAX], hv[SMAX];
#pragma unroll
                for (int s = 0; s < SMAX; ++s) {
                    hq[s] = __builtin_amdgcn_readlane(q[s], g_h);
                    he[s] = __builtin_amdgcn_readlane(se[s], g_h);
                    hv[s] = host_of[(he[s] > 0 ? he[s] : 0) * kWave + lane];
                }
                const unsigned long long room = __ballot(occupied < S);
                const unsigned long long colder = __ballot(L_h - L > 1) & ranks;
                unsigned long long any = 0ull;
                bool spare[SMAX];  // the expert may have another copy
#pragma unroll
                for (int s = 0; s < SMAX; ++s) {
                    const unsigned long long hosts = __ballot(hv[s] != kNoHost);
                    spare[s] = __popcll(hosts) < c_max;
                    any |= hq[s] > 0 ? hosts | (spare[s] ? room : 0ull) : 0ull;
                }
                any &= colder;
                if (any == 0ull) break;  // nothing feasible
                const bool has = __builtin_amdgcn_inverse_ballot_w64(any);
                L_c = wave_min_i32<ROWS>(has ? L : IMAX);
                g_c = __builtin_ctzll(__ballot(L == L_c) & any);  // ties -> lowest g
                // that rank's first feasible slot of the hot rank, equal rows keep the lower slot
                const int free_slot = __builtin_amdgcn_readlane(occupied, g_c);
                q_sel = 0;
#pragma unroll
                for (int s = 0; s < SMAX; ++s) {
                    const int at = __builtin_amdgcn_readlane(hv[s], g_c);
                    const bool ok = at != kNoHost || (spare[s] && free_slot < S);
                    if (ok && hq[s] > q_sel) {
                        q_sel = hq[s];
                        s_sel = s;
                        e_sel = he[s];
                        sp_sel = at != kNoHost ? at : free_slot;
                    }
                }
            }
            const int delta = (L_h - L_c + 1) / 2;  // ceil((L_h - L_c) / 2)
            const int m = delta < q_sel ? delta : q_sel;
            // both ranks at once: the slot that changes hosts (or, with a copy, now hosts) e_sel
            const bool cold = lane == g_c;
            const int change = lane == g_h ? -m : (cold ? m : 0);
            const int slot = lane == g_h ? s_sel : (cold ? sp_sel : -1);
#pragma unroll
            for (int t = 0; t < SMAX; ++t) {
                q[t] += t == slot ? change : 0;
                se[t] = t == slot ? e_sel : se[t];
            }
            L += change;
            if (cold) host_of[e_sel * kWave + lane] = (unsigned char)sp_sel;
            occupied += cold && sp_sel == occupied ? 1 : 0;
            ++n_iters;
        }
    }
    if (valid) {
#pragma unroll
        for (int s = 0; s < SMAX; ++s)
            if (s < S) {
                slot_expert[lane * S + s] = se[s];
                slot_quota[lane * S + s] = q[s];
            }
        rank_load_pred[lane] = L;
    }
    if (lane == 0) n_iters_out[0] = n_iters;
}

}  // namespace moegps

extern "C" int moe_plan_duplicates(int mode, const int32_t* hist_pred, int E, int G, int S, int c_max,
                                   int32_t* slot_expert, int32_t* slot_quota, int32_t* rank_load_pred,
                                   int32_t* n_iters, void* stream) {
    using namespace moegps;
    if (mode < MOE_MODE_NONE || mode > MOE_MODE_TOKEN) return MOE_ERR_INVALID_ARG;
    if (E < 1 || G < 1 || S < 1 || c_max < 1) return MOE_ERR_INVALID_ARG;
    if (ceil_div(E, G) > S) return MOE_ERR_INVALID_ARG;  // every expert needs a home slot
    if (E > MOE_MAX_EXPERTS || G > MOE_MAX_RANKS || S > MOE_MAX_SLOTS || G * S > MOE_MAX_SEGMENTS)
        return MOE_ERR_UNSUPPORTED;
    if (!hist_pred || !slot_expert || !slot_quota || !rank_load_pred || !n_iters) return MOE_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (G <= kWave) {
        // one lane per rank, state in registers
        auto launch = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(1), dim3(kWave), 0, st, mode, hist_pred, E, G, S, c_max, slot_expert,
                               slot_quota, rank_load_pred, n_iters);
        };
        // one instantiation per slot count: every loop over a rank's slots is unrolled to exactly S
        switch (S) {
            case 1: launch(G <= 32 ? plan_kernel_regs<1, 2> : plan_kernel_regs<1, 4>); break;
            case 2: launch(G <= 32 ? plan_kernel_regs<2, 2> : plan_kernel_regs<2, 4>); break;
            case 3: launch(G <= 32 ? plan_kernel_regs<3, 2> : plan_kernel_regs<3, 4>); break;
            case 4: launch(G <= 32 ? plan_kernel_regs<4, 2> : plan_kernel_regs<4, 4>); break;
            case 5: launch(G <= 32 ? plan_kernel_regs<5, 2> : plan_kernel_regs<5, 4>); break;
            case 6: launch(G <= 32 ? plan_kernel_regs<6, 2> : plan_kernel_regs<6, 4>); break;
            case 7: launch(G <= 32 ? plan_kernel_regs<7, 2> : plan_kernel_regs<7, 4>); break;
            case 8: launch(G <= 32 ? plan_kernel_regs<8, 2> : plan_kernel_regs<8, 4>); break;
            case 9: launch(G <= 32 ? plan_kernel_regs<9, 2> : plan_kernel_regs<9, 4>); break;
            case 10: launch(G <= 32 ? plan_kernel_regs<10, 2> : plan_kernel_regs<10, 4>); break;
            case 11: launch(G <= 32 ? plan_kernel_regs<11, 2> : plan_kernel_regs<11, 4>); break;
            case 12: launch(G <= 32 ? plan_kernel_regs<12, 2> : plan_kernel_regs<12, 4>); break;
            case 13: launch(G <= 32 ? plan_kernel_regs<13, 2> : plan_kernel_regs<13, 4>); break;
            case 14: launch(G <= 32 ? plan_kernel_regs<14, 2> : plan_kernel_regs<14, 4>); break;
            case 15: launch(G <= 32 ? plan_kernel_regs<15, 2> : plan_kernel_regs<15, 4>); break;
            default: launch(G <= 32 ? plan_kernel_regs<16, 2> : plan_kernel_regs<16, 4>); break;
        }
        return check_launch();
    }
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kWave), 0, st, mode, hist_pred, E, G, S, c_max, slot_expert,
                       slot_quota, rank_load_pred, n_iters);
    return check_launch();
}
