// Gate top-k as a call of its own (route_tokens.h holds the kernel's body).
#include "route_tokens.h"

namespace moegps {

template <int LPT, int VPL>
__global__ __launch_bounds__(kRouteThreads) void route_topk_kernel(const float* __restrict__ logits, int T, int E,
                                                                    int k, int32_t* __restrict__ topk_idx,
                                                                    float* __restrict__ topk_w) {
    route_tokens<LPT, VPL>(blockIdx.x, logits, T, E, k, topk_idx, topk_w);
}

template <int LPT, int VPL>
static int launch_route(const float* logits, int T, int E, int k, int32_t* idx, float* w, hipStream_t st) {
    hipLaunchKernelGGL((route_topk_kernel<LPT, VPL>), dim3(ceil_div(T, kRouteThreads / LPT)), dim3(kRouteThreads), 0, st,
                       logits, T, E, k, idx, w);
    return check_launch();
}

}  // namespace moegps

extern "C" int moe_route_topk(const float* logits, int T, int E, int k, int32_t* topk_idx, float* topk_w,
                              void* stream) {
    using namespace moegps;
    if (T < 0 || E < 1 || k < 1 || k > E) return MOE_ERR_INVALID_ARG;
    if (E > MOE_MAX_EXPERTS || k > MOE_MAX_TOPK) return MOE_ERR_UNSUPPORTED;
    if (route_blocks(T, E) > kRouteMaxBlocks) return MOE_ERR_UNSUPPORTED;
    if (T == 0) return MOE_OK;
    if (!logits || !topk_idx || !topk_w) return MOE_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    // lanes per token as route_lanes has them
    if (E <= 2) return launch_route<2, 1>(logits, T, E, k, topk_idx, topk_w, st);
    if (E <= 4) return launch_route<4, 1>(logits, T, E, k, topk_idx, topk_w, st);
    if (E <= 8) return launch_route<8, 1>(logits, T, E, k, topk_idx, topk_w, st);
    if (E <= 16) return launch_route<16, 1>(logits, T, E, k, topk_idx, topk_w, st);
    if (E <= 32) return launch_route<16, 2>(logits, T, E, k, topk_idx, topk_w, st);
    if (E <= 64) return launch_route<16, 4>(logits, T, E, k, topk_idx, topk_w, st);
    if (E <= 128) return launch_route<16, 8>(logits, T, E, k, topk_idx, topk_w, st);
    if (E <= 256) return launch_route<16, 16>(logits, T, E, k, topk_idx, topk_w, st);
    if (E <= 512) return launch_route<16, 32>(logits, T, E, k, topk_idx, topk_w, st);
    return launch_route<32, 32>(logits, T, E, k, topk_idx, topk_w, st);
}
