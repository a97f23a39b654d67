// bf16 GEMM instantiations for the weight-gradient layout dW = X^T dY: A(m,k) = X[k,m] (m-contiguous) and
// B(k,n) = dY[k,n] (n-contiguous); k runs over tokens.
#include "gemm_bf16_split.h"

namespace mlm {

hipError_t launch_gemm_bf16_wgrad(const GemmArgs& a, hipStream_t st) {
  if (a.epi != EPI_STORE) return hipErrorInvalidValue;
  return launch_gemm_bf16_any<false, false, EPI_STORE>(a, st);
}

template <int TM, int TN>
static hipError_t launch_split_group(const GemmArgs* probs, int n, int form, hipStream_t st) {
  SplitGroup g;
  memset(&g, 0, sizeof(g));
  int total = 0;
  for (int q = 0; q < n; ++q) {
    g.args[q] = probs[q];
    g.tile_begin[q] = total;
    total += split_tiles(form, probs[q].M, probs[q].N);
  }
  for (int q = n; q < kMaxGroup; ++q) g.tile_begin[q] = total;
  static LdsAttrOnce attr;
  return launch_split(&attr, gemm_bf16_split_group_kernel<TM, TN>, split_lds_bytes<TM, TN>(), total, st, g);
}

// The weight gradients of a layer shard (same operand layout, same k = tokens), as v2_group_middle, split_group_pick and v2_group_plan say.
hipError_t launch_gemm_bf16_wgrad_group(const GemmArgs* probs, int n, float* splitk_ws, hipStream_t st) {
  const V2GroupPlan p = v2_group_plan(probs, n, splitk_ws != nullptr);
  if (v2_group_middle(probs, n, p)) return launch_gemm_bf16_v2_group<false, false, 192, true>(probs, n, st);
  switch (split_group_pick(probs, n, p)) {
    case SPLIT_64: return launch_split_group<64, 64>(probs, n, SPLIT_64, st);
    case SPLIT_32X64: return launch_split_group<32, 64>(probs, n, SPLIT_32X64, st);
    case SPLIT_32: return launch_split_group<32, 32>(probs, n, SPLIT_32, st);
    default: break;
  }
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
