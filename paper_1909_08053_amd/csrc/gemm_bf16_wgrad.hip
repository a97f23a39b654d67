// bf16 GEMM instantiations for the weight-gradient layout dW = X^T dY: A(m,k) = X[k,m] (m-contiguous) and
// B(k,n) = dY[k,n] (n-contiguous); k runs over tokens.
#include "gemm_bf16_v2.h"

namespace mlm {

hipError_t launch_gemm_bf16_wgrad(const GemmArgs& a, hipStream_t st) {
  if (a.epi != EPI_STORE) return hipErrorInvalidValue;
  return launch_gemm_bf16_v2<false, false, EPI_STORE>(a, a.splitk_ws, st);
}

// The weight gradients of a layer shard (same operand layout, same k = tokens), as v2_group_plan says.
hipError_t launch_gemm_bf16_wgrad_group(const GemmArgs* probs, int n, float* splitk_ws, hipStream_t st) {
  const V2GroupPlan p = v2_group_plan(probs, n, splitk_ws != nullptr);
  if (p.split.split) return launch_gemm_bf16_v2_group<false, false, V2_B, false, true>(probs, n, st, p.split, splitk_ws);
  if (p.bn == V2_B) return launch_gemm_bf16_v2_group<false, false, V2_B, false>(probs, n, st);
  if (p.bn == V2_SMALL) {
    int tiles = 0;
    for (int q = 0; q < n; ++q) tiles += v2_tiles(probs[q], V2_SMALL, V2_SMALL);
    return tiles <= gemm_cu_count() ? launch_gemm_bf16_v2_group<false, false, V2_SMALL, true>(probs, n, st)
                                    : launch_gemm_bf16_v2_group<false, false, V2_SMALL, false>(probs, n, st);
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
