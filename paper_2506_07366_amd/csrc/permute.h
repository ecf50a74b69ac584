// Parts of the permutation that the whole-layer call launches on its own (permute.hip).
#pragma once
#include "ffn_tables.h"

namespace moegps {

// Outputs of the duplication plan, for mode 0, whose plan is the home placement of the batch's own counts.
struct HomePlan {
    int32_t *slot_expert, *slot_quota, *rank_load_pred, *n_iters;
};

// Whether moe_permute does the index steps of A assignments in one workgroup.
bool permute_in_one_workgroup(int mode, int64_t A, int E, int nseg);

// These index steps, with the histogram of topk_idx as an output (and in mode 0 the plan, `home`), and
// the tables of the grouped FFN behind them if `job` has a row list.
int permute_and_count(int mode, int T, int k, int E, int G, int S, const int32_t* topk_idx, const int32_t* pred_idx,
                      const int32_t* hist_pred, const int32_t* slot_expert, const int32_t* slot_quota,
                      int32_t* seg_offsets, int32_t* row_of_assign, int32_t* assign_of_row, int32_t* rank_load,
                      int32_t* hist_out, const HomePlan& home, const TableJob& job, hipStream_t st);

// The same by many workgroups, for batches that permute_counts() says they count; hist_out is zero before.  (The tables are
// a launch of their own.)
bool permute_counts(int T, int E, int k, int G, int S);
int permute_and_count_wide(int mode, int T, int k, int E, int G, int S, const int32_t* topk_idx, const int32_t* pred_idx,
                           const int32_t* hist_pred, const int32_t* slot_expert, const int32_t* slot_quota,
                           int32_t* seg_offsets, int32_t* row_of_assign, int32_t* assign_of_row, int32_t* rank_load,
                           int32_t* hist_out, const HomePlan& home, void* workspace, hipStream_t st);

}  // namespace moegps
