// bf16 GEMM instantiations for the weight-gradient layout dW = X^T dY: A(m,k) = X[k,m] (m-contiguous) and
// B(k,n) = dY[k,n] (n-contiguous); k runs over tokens.
#include "gemm_bf16_v2.h"

namespace mlm {

hipError_t launch_gemm_bf16_wgrad(const GemmArgs& a, hipStream_t st) {
  if (a.epi != EPI_STORE) return hipErrorInvalidValue;
  return launch_gemm_bf16_v2<false, false, EPI_STORE>(a, a.splitk_ws, st);
}

// The weight gradients of a layer shard (same operand layout, same k = tokens).  One grouped launch, in the tile size that
// fills the chip better, when the cost model says the shared last round beats the separate launches with their
// k-splits (v2_group_split: large tiles with that round split along k); separate launches otherwise.
hipError_t launch_gemm_bf16_wgrad_group(const GemmArgs* probs, int n, float* splitk_ws, hipStream_t st) {
  bool groupable = n >= 2 && n <= kMaxGroup;
  double alone = 0.0;
  for (int q = 0; q < n && groupable; ++q) {
    groupable = probs[q].epi == EPI_STORE && probs[q].bias == nullptr && probs[q].K == probs[0].K;
    const int M = probs[q].M, N = probs[q].N, K = probs[q].K;
    alone += v2_plan(M, N, K, true, v2_pick_bn<false, false, EPI_STORE>(M, N, K, true)).cost + 2.0;   // + launch and drain
  }
  if (groupable) {
    const double big = v2_group_cost(probs, n, V2_B), small = v2_group_cost(probs, n, V2_SMALL);
    const int forced = gemm_v2_forced_bn();
    const bool use_small = forced ? forced == V2_SMALL : small < big;
    if (!gemm_v2_group_off() && !forced && splitk_ws) {
      const V2GroupSplit sp = v2_group_split(probs, n);
      const double whole = use_small ? v2_group_cost(probs, n, V2_SMALL, true) : big;
      if (sp.split && sp.cost < 0.97 * whole && sp.cost + 2.0 < alone)
        return launch_gemm_bf16_v2_group<false, false, V2_B, false, true>(probs, n, st, sp, splitk_ws);
    }
    if (!gemm_v2_group_off() && (use_small ? small : big) + 2.0 < alone) {
      int tiles = 0;
      for (int q = 0; q < n; ++q) tiles += v2_tiles(probs[q], V2_SMALL, V2_SMALL);
      if (!use_small) return launch_gemm_bf16_v2_group<false, false, V2_B, false>(probs, n, st);
      return tiles <= gemm_cu_count() ? launch_gemm_bf16_v2_group<false, false, V2_SMALL, true>(probs, n, st)
                                      : launch_gemm_bf16_v2_group<false, false, V2_SMALL, false>(probs, n, st);
    }
  }
  for (int q = 0; q < n; ++q) {
    GemmArgs a = probs[q];
    a.splitk_ws = splitk_ws;
    hipError_t e = launch_gemm_bf16_wgrad(a, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mlm
