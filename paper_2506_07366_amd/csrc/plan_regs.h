// The duplication planner for up to 64 ranks, by one wavefront with its state in registers (plan.hip holds
// the version for any number of ranks, and what both compute).
#pragma once
#include "common.h"
#include "block_scan.h"

namespace moegps {

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

// host_of: E * kWave bytes of LDS, 16-byte aligned.  hist_pred may be in LDS.
template <int SMAX, int ROWS>
__device__ __forceinline__ void plan_regs(int mode, const int32_t* hist_pred, int E, int G, int S, int c_max,
                                          unsigned char* host_of, int32_t* __restrict__ slot_expert,
                                          int32_t* __restrict__ slot_quota, int32_t* __restrict__ rank_load_pred,
                                          int32_t* __restrict__ n_iters_out) {
    const int lane = threadIdx.x;  // one wavefront, the first of its workgroup
    const bool valid = lane < G;
    const int H = (E + G - 1) / G;
    constexpr int NONE = -2;  // slot index >= S: neither empty nor an expert
    const int IMAX = 0x7fffffff;

    // slot of rank g that hosts expert e (one byte each), kNoHost: none
    constexpr int kNoHost = 255;
    if (mode != MOE_MODE_NONE) {
        for (int i = lane * 16; i < E * kWave; i += kWave * 16)
            *(uint4*)&host_of[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
        wave_lds_order();
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
