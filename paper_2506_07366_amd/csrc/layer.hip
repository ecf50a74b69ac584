// A whole step of the layer in one call: route, histogram, duplication plan, permutation, grouped FFN and
// combine of one batch, with launches shared between the small ones.
//
// The index steps of a decode or prompt batch are a chain of launches of 2 to 20 us of work, 4.7 us apart at
// least, and each is a call from the host.  Three things shorten it where the shape allows:
//   - under a prediction the plan does not need the routing: one workgroup makes it (under Token-to-Expert
//     after counting the predicted ids) while the others of the same launch route the tokens;
//   - where the permutation is one workgroup's work it also writes the histogram, without a prediction
//     the plan, which then is the home placement, and goes on to the tables of the grouped FFN.
//   - the permuted rows are for the caller alone: the first product reads its rows from x, and the copy goes with its
//     launch (ffn_tiles.h, grouped_ffn.hip).
// Anything else goes through the calls of the single steps, in their order; the results are the same integers
// either way.
// Whole steps, us, six calls (seven with predicted ids) -> one: 256 tokens of the small fp32 layer 45.0 -> 39.9 (no
// longer bound by the host, which takes 22), one token on 128 experts 80.2 -> 74.9, 777 tokens with Token-to-Expert 438 ->
// 427; batches of some 300 us and more gain less than the runs differ.
#include "permute.h"
#include "plan_regs.h"
#include "route_tokens.h"

namespace moegps {

constexpr int kPlanMaxExperts = 256;   // the planner's table of hosts takes 64 bytes of LDS per expert, and
                                       // every workgroup of the launch has it
constexpr int kPlanMaxSlots = 10;      // slots per rank the launch is compiled for, up to 32 ranks
constexpr int kPlanCountMax = 16384;   // predicted ids one workgroup counts ahead of its plan

struct PlanJob {
    int mode, E, G, S, c_max;
    const int32_t* hist_pred;  // null: counted from pred_idx
    const int32_t* pred_idx;
    int n_pred;
    int32_t *hist_plan, *slot_expert, *slot_quota, *rank_load_pred, *n_iters;
    int32_t* hist;             // counts that a later launch adds to, cleared here; null: none
};

// Workgroup 0 plans, the others route.  The plan is the longer of the two up to some 30000 tokens: us of
// the launch against those of its parts, 128 experts, 128 tokens 17.1 (17.8 and 4.9), 777 tokens with
// Token-to-Expert 29.2 (26.6, 5.1 and 4.9 for the count); 64 experts, 2048 tokens 23.6 (22.7 and 5.2).
template <int S>
__global__ __launch_bounds__(kRouteThreads) void route_plan_kernel(PlanJob p, const float* __restrict__ logits, int T,
                                                                    int k, int32_t* __restrict__ topk_idx,
                                                                    float* __restrict__ topk_w) {
    extern __shared__ __align__(16) unsigned char host_of[];
    __shared__ int bins[kPlanMaxExperts];
    const int E = p.E;
    if (blockIdx.x > 0) {
        const int block = blockIdx.x - 1;
        if (E <= 2) route_tokens<2, 1>(block, logits, T, E, k, topk_idx, topk_w);
        else if (E <= 4) route_tokens<4, 1>(block, logits, T, E, k, topk_idx, topk_w);
        else if (E <= 8) route_tokens<8, 1>(block, logits, T, E, k, topk_idx, topk_w);
        else if (E <= 16) route_tokens<16, 1>(block, logits, T, E, k, topk_idx, topk_w);
        else if (E <= 32) route_tokens<16, 2>(block, logits, T, E, k, topk_idx, topk_w);
        else if (E <= 64) route_tokens<16, 4>(block, logits, T, E, k, topk_idx, topk_w);
        else if (E <= 128) route_tokens<16, 8>(block, logits, T, E, k, topk_idx, topk_w);
        else route_tokens<16, 16>(block, logits, T, E, k, topk_idx, topk_w);
        return;
    }
    if (p.hist)
        for (int e = threadIdx.x; e < E; e += kRouteThreads) p.hist[e] = 0;
    if (p.mode == MOE_MODE_NONE) return;  // (the plan is the home placement, made from the batch's counts)
    const int32_t* hist = p.hist_pred;
    if (!hist) {
        static_assert(kPlanMaxExperts <= kRouteThreads, "a thread per expert");
        const int tid = threadIdx.x;
        bins[tid] = 0;
        __syncthreads();
        constexpr int U = 8;  // ids under way per thread
        for (int i0 = tid; i0 < p.n_pred; i0 += kRouteThreads * U) {
            int e[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * kRouteThreads;
                e[u] = i < p.n_pred ? p.pred_idx[i] : -1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (e[u] >= 0 && e[u] < E) atomicAdd(&bins[e[u]], 1);
        }
        __syncthreads();
        if (tid < E) p.hist_plan[tid] = bins[tid];
        hist = bins;
    }
    if (threadIdx.x < kWave)
        plan_regs<S, 2>(p.mode, hist, E, p.G, S, p.c_max, host_of, p.slot_expert, p.slot_quota, p.rank_load_pred, p.n_iters);
}

static int route_and_plan(const PlanJob& p, const float* logits, int T, int k, int32_t* topk_idx, float* topk_w,
                          hipStream_t st) {
    const int grid = 1 + route_blocks(T, p.E);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kRouteThreads), (size_t)p.E * kWave, st, p, logits, T, k, topk_idx, topk_w);
        return check_launch();
    };
    switch (p.S) {
        case 1: return go(route_plan_kernel<1>);
        case 2: return go(route_plan_kernel<2>);
        case 3: return go(route_plan_kernel<3>);
        case 4: return go(route_plan_kernel<4>);
        case 5: return go(route_plan_kernel<5>);
        case 6: return go(route_plan_kernel<6>);
        case 7: return go(route_plan_kernel<7>);
        case 8: return go(route_plan_kernel<8>);
        case 9: return go(route_plan_kernel<9>);
        default: return go(route_plan_kernel<kPlanMaxSlots>);
    }
}

}  // namespace moegps

extern "C" int moe_layer_step(const moe_layer_step_args* a, void* stream) {
    using namespace moegps;
    if (!a) return MOE_ERR_INVALID_ARG;
    const int mode = a->mode, T = a->T, E = a->E, k = a->k, G = a->G, S = a->S;
    // what the calls of the single steps would refuse, before the first launch
    if (mode < MOE_MODE_NONE || mode > MOE_MODE_TOKEN) return MOE_ERR_INVALID_ARG;
    if (a->dtype != MOE_DTYPE_F32 && a->dtype != MOE_DTYPE_BF16) return MOE_ERR_INVALID_ARG;
    if (T < 0 || a->d < 1 || a->ffn < 1 || E < 1 || k < 1 || k > E || G < 1 || S < 1 || a->c_max < 1)
        return MOE_ERR_INVALID_ARG;
    if (E > MOE_MAX_EXPERTS || k > MOE_MAX_TOPK || G > MOE_MAX_RANKS || S > MOE_MAX_SLOTS || G * S > MOE_MAX_SEGMENTS)
        return MOE_ERR_UNSUPPORTED;
    if (ceil_div(E, G) > S) return MOE_ERR_INVALID_ARG;
    if ((int64_t)T * k >= (1ll << 31) || route_blocks(T, E) >= kRouteMaxBlocks) return MOE_ERR_UNSUPPORTED;
    if (((size_t)a->d * dtype_size(a->dtype)) % 16 != 0) return MOE_ERR_UNSUPPORTED;
    if (a->relu && !a->x_perm) return MOE_ERR_UNSUPPORTED;  // the row gather is built for the SwiGLU form only
    if (T == 0) return MOE_OK;
    if (!a->logits || !a->x || !a->packed || !a->topk_idx || !a->topk_w || !a->hist || !a->slot_expert ||
        !a->slot_quota || !a->rank_load_pred || !a->n_iters || !a->seg_offsets || !a->row_of_assign ||
        !a->assign_of_row || !a->rank_load || !a->y_perm || !a->out || !a->workspace_perm || !a->workspace_ffn)
        return MOE_ERR_INVALID_ARG;
    if (mode == MOE_MODE_DISTRIBUTION && !a->hist_pred) return MOE_ERR_INVALID_ARG;
    if (mode == MOE_MODE_TOKEN && (!a->pred_idx || !a->hist_plan)) return MOE_ERR_INVALID_ARG;
    if (!a->x_perm && (int64_t)T * a->d >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;  // 32-bit element offsets into x
    const int64_t A = (int64_t)T * k;
    if (a->workspace_perm_bytes < moe_permute_workspace_bytes(T, E, k, G, S)) return MOE_ERR_WORKSPACE_TOO_SMALL;
    if (a->x_perm && a->dtype == MOE_DTYPE_BF16 && A * a->d >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;  // as moe_grouped_ffn
    hipStream_t st = (hipStream_t)stream;
    int rc;
    const int32_t* hp = mode == MOE_MODE_TOKEN ? a->hist_plan : mode == MOE_MODE_DISTRIBUTION ? a->hist_pred : a->hist;
    // The prediction may be one of the step's own outputs (topk_idx as predicted ids, hist as predicted counts): it
    // then is what this step writes there, and nothing may run ahead of that or beside it.
    const size_t ids = (size_t)A * sizeof(int32_t), counts = (size_t)E * sizeof(int32_t);
    const void* pred = mode == MOE_MODE_TOKEN ? a->pred_idx : mode == MOE_MODE_DISTRIBUTION ? a->hist_pred : nullptr;
    const size_t n_pred = mode == MOE_MODE_TOKEN ? ids : counts;
    const bool own_pred = pred && (share_bytes(pred, n_pred, a->topk_idx, ids) || share_bytes(pred, n_pred, a->topk_w, ids) ||
                                   share_bytes(pred, n_pred, a->hist, counts));
    // x may lie in the FFN's scratch, being done with once its rows have been copied: then they are, before the FFN.
    const size_t tokens_bytes = (size_t)T * a->d * dtype_size(a->dtype);
    const bool copy_first = a->x_perm && share_bytes(a->x, tokens_bytes, a->workspace_ffn, a->workspace_ffn_bytes);
    const bool small = !own_pred && !copy_first && permute_in_one_workgroup(mode, A, E, G * S);
    // What the first workgroup of the routing launch writes, the plan and a cleared histogram, may lie in the logits, which the
    // others still read: then that is left to later launches.
    const size_t slots = (size_t)G * S * sizeof(int32_t), loads = (size_t)G * sizeof(int32_t);
    auto in_logits = [&](const void* p, size_t n) { return share_bytes(p, n, a->logits, (size_t)T * E * sizeof(float)); };
    const bool plan_in_logits = (mode == MOE_MODE_TOKEN && in_logits(a->hist_plan, counts)) || in_logits(a->slot_expert, slots) ||
                                in_logits(a->slot_quota, slots) || in_logits(a->rank_load_pred, loads) ||
                                in_logits(a->n_iters, sizeof(int32_t));
    const bool shared = !own_pred && (mode == MOE_MODE_NONE || !plan_in_logits) && E <= kPlanMaxExperts &&
                        S <= kPlanMaxSlots && G <= 32;
    // several workgroups permute and add up the histogram, which the first launch clears (and then counts predicted ids)
    const bool own_counts = mode == MOE_MODE_TOKEN && share_bytes(a->hist_plan, counts, a->hist, counts);
    const bool wide =
        shared && !small && !copy_first && !own_counts && !in_logits(a->hist, counts) && permute_counts(T, E, k, G, S);
    const bool together = shared && (wide || mode != MOE_MODE_NONE);
    auto plan = [&] {
        return moe_plan_duplicates(mode, hp, E, G, S, a->c_max, a->slot_expert, a->slot_quota, a->rank_load_pred,
                                   a->n_iters, stream);
    };
    const float* gate = a->x_perm ? nullptr : a->gate_in_ffn ? a->topk_w : nullptr;
    // The permuted rows are for the caller: the first product reads the rows of x, and they are copied beside it.
    const RowCopy copy = a->x_perm && !copy_first ? row_copy(a->x, a->dtype, T, a->d, k, a->row_of_assign, a->x_perm) : RowCopy{};
    // The permutation's scratch, done with by then, takes the list of the rows' tokens (it is larger than A ints), unless the caller
    // has it share memory with what the launch of the first product writes.
    const size_t rows = (size_t)A * a->d * dtype_size(a->dtype);
    const bool scratch_free = !share_bytes(a->workspace_perm, ids, a->workspace_ffn, a->workspace_ffn_bytes) &&
                              !share_bytes(a->workspace_perm, ids, a->y_perm, rows) &&
                              !share_bytes(a->workspace_perm, ids, a->x, tokens_bytes) &&
                              !(a->x_perm && share_bytes(a->workspace_perm, ids, a->x_perm, rows));
    int32_t* const tokens = scratch_free ? (int32_t*)a->workspace_perm : nullptr;
    const FfnOptions opt = ffn_options();  // (once: the job and the products go by the same)
    auto ffn = [&](FfnStage stage, TableJob* job) {
        if (copy_first)
            return grouped_ffn_call(a->relu, a->x_perm, A, nullptr, 1, nullptr, nullptr, a->dtype, A, a->d, a->ffn, E,
                                    a->seg_offsets, a->slot_expert, G * S, 0, G * S, a->packed, a->y_perm, a->workspace_ffn,
                                    a->workspace_ffn_bytes, stream, opt, stage, job);
        return grouped_ffn_call(a->relu, a->x, T, a->assign_of_row, k, gate ? a->assign_of_row : nullptr, gate, a->dtype, A,
                                a->d, a->ffn, E, a->seg_offsets, a->slot_expert, G * S, 0, G * S, a->packed, a->y_perm,
                                a->workspace_ffn, a->workspace_ffn_bytes, stream, opt, stage, job, copy, tokens);
    };
    TableJob job{};
    if ((rc = ffn(kFfnJobOnly, &job)) != MOE_OK) return rc;  // (checks its arguments, launches nothing)
    // The workgroup that permutes builds the tables too where their tile heights are given: one token on 128
    // experts 15.0 us against 8.9 and 6.9, 128 tokens 17.9 against 10.9 and 7.9, and a launch less.  Where it would
    // have to choose them first, a launch of its own is ahead (1001 tokens, 8 experts 28.7 against 13.9 and 9.7).
    const bool tables_too = small && job.t1.bm != 0 && (!job.t2.tiles || job.t2.bm != 0);
    if (!tables_too) job = TableJob{};
    if (together) {
        const bool count = mode == MOE_MODE_TOKEN && A <= kPlanCountMax;
        if (mode == MOE_MODE_TOKEN && !count && (rc = moe_histogram(a->pred_idx, A, E, a->hist_plan, stream)) != MOE_OK)
            return rc;
        const PlanJob p{mode, E, G, S, a->c_max, count ? nullptr : hp, a->pred_idx, (int)A, a->hist_plan,
                        a->slot_expert, a->slot_quota, a->rank_load_pred, a->n_iters, wide ? a->hist : nullptr};
        if ((rc = route_and_plan(p, a->logits, T, k, a->topk_idx, a->topk_w, st)) != MOE_OK) return rc;
    } else {
        if ((rc = moe_route_topk(a->logits, T, E, k, a->topk_idx, a->topk_w, stream)) != MOE_OK) return rc;
        if (own_pred && (rc = moe_histogram(a->topk_idx, A, E, a->hist, stream)) != MOE_OK) return rc;
        if (mode == MOE_MODE_TOKEN && (rc = moe_histogram(a->pred_idx, A, E, a->hist_plan, stream)) != MOE_OK) return rc;
        if (mode != MOE_MODE_NONE && (rc = plan()) != MOE_OK) return rc;
    }
    if (small) {
        const HomePlan home{a->slot_expert, a->slot_quota, a->rank_load_pred, a->n_iters};
        rc = permute_and_count(mode, T, k, E, G, S, a->topk_idx, a->pred_idx, hp, a->slot_expert, a->slot_quota,
                               a->seg_offsets, a->row_of_assign, a->assign_of_row, a->rank_load, a->hist, home, job, st);
    } else if (wide) {
        const HomePlan home{a->slot_expert, a->slot_quota, a->rank_load_pred, a->n_iters};
        rc = permute_and_count_wide(mode, T, k, E, G, S, a->topk_idx, a->pred_idx, hp, a->slot_expert, a->slot_quota,
                                    a->seg_offsets, a->row_of_assign, a->assign_of_row, a->rank_load, a->hist, home,
                                    a->workspace_perm, st);
    } else {
        if (!own_pred && (rc = moe_histogram(a->topk_idx, A, E, a->hist, stream)) != MOE_OK) return rc;
        if (mode == MOE_MODE_NONE && (rc = plan()) != MOE_OK) return rc;
        rc = moe_permute(mode, copy_first ? a->x : nullptr, a->dtype, T, a->d, E, k, G, S, a->topk_idx,
                         mode == MOE_MODE_TOKEN ? a->pred_idx : nullptr, a->hist, hp, a->slot_expert, a->slot_quota,
                         a->seg_offsets, a->row_of_assign, a->assign_of_row, copy_first ? a->x_perm : nullptr,
                         a->rank_load, a->workspace_perm, a->workspace_perm_bytes, stream);
    }
    if (rc != MOE_OK) return rc;
    if ((rc = ffn(tables_too ? kFfnTablesBuilt : kFfnAll, nullptr)) != MOE_OK) return rc;
    return moe_combine(a->y_perm, a->dtype, T, a->d, k, a->row_of_assign, gate ? nullptr : a->topk_w, a->out, stream);
}
