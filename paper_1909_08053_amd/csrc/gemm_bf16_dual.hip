// The two gradients of the vocabulary-parallel logits in one launch: dE = hf^T dL (weight-gradient layout) and dhf = dL E^T
// (input-gradient layout).  Neither reads the other's result, and each alone leaves a partly filled last round of tiles that its
// launch pays for by idle compute units or by fp32 partial tiles and a fix-up pass.
#include "gemm_bf16_split.h"

namespace mlm {

// Work items 0 .. first - 1 are the tiles of a1 (first_is_1) or of a0, the rest the other one's.
template <int BN, int KE0, int KE1, bool DEEP>
__global__ __launch_bounds__((v2_nw<BN, DEEP>() * 64), 2) void gemm_bf16_v2_dual_kernel(GemmArgs a0, V2Plan p0, GemmArgs a1,
                                                                                        V2Plan p1, int first_is_1) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int id = blockIdx.x, first = first_is_1 ? p1.full_tiles : p0.full_tiles;
  const int at = id < first ? id : id - first;
  if ((id < first) == (first_is_1 != 0)) {
    const int pid = p1.strip ? v2_xcd_order(at, p1.full_tiles, p1.window) : at;
    gemm_v2_work_item<true, true, EPI_STORE, BN, KE1, DEEP, false>(a1, p1, nullptr, pid, lds_raw);
  } else {
    const int pid = p0.strip ? v2_xcd_order(at, p0.full_tiles, p0.window) : at;
    gemm_v2_work_item<false, false, EPI_STORE, BN, KE0, DEEP, false>(a0, p0, nullptr, pid, lds_raw);
  }
}

template <int BN, int KE0, int KE1, bool DEEP>
static hipError_t launch_dual(const GemmArgs& a0, const GemmArgs& a1, bool first_is_1, hipStream_t st) {
  auto kern = gemm_bf16_v2_dual_kernel<BN, KE0, KE1, DEEP>;
  constexpr size_t k0 = v2_lds_bytes<false, false, BN, DEEP>(), k1 = v2_lds_bytes<true, true, BN, DEEP>(), kLds = k0 > k1 ? k0 : k1;
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
  V2Plan p0 = v2_plan(a0.M, a0.N, a0.K, false, BN), p1 = v2_plan(a1.M, a1.N, a1.K, false, BN);
  v2_set_walk(&p0, v2_window<BN, DEEP>(), a0.K);
  v2_set_walk(&p1, v2_window<BN, DEEP>(), a1.K);
  hipLaunchKernelGGL(kern, dim3((unsigned)(p0.full_tiles + p1.full_tiles)), dim3(v2_nw<BN, DEEP>() * 64), kLds, st, a0, p0, a1, p1,
                     first_is_1 ? 1 : 0);
  return hipGetLastError();
}

template <int TM, int TN>
static hipError_t launch_split_dual(const GemmArgs& a0, const GemmArgs& a1, int form, hipStream_t st) {
  static LdsAttrOnce attr;
  const int n0 = split_tiles(form, a0.M, a0.N), n1 = split_tiles(form, a1.M, a1.N);
  return launch_split(&attr, gemm_bf16_split_dual_kernel<TM, TN>, split_lds_bytes<TM, TN>(), n0 + n1, st, a0, a1, a1.K > a0.K ? n1 : n0);
}

hipError_t launch_gemm_bf16_dual(const GemmArgs& a0, const GemmArgs& a1, float* splitk_ws, hipStream_t st) {
  const V2Dual d = v2_dual(a0, a1);
  switch (split_dual_pick(a0, a1, d)) {
    case SPLIT_64: return launch_split_dual<64, 64>(a0, a1, SPLIT_64, st);
    case SPLIT_32X64: return launch_split_dual<32, 64>(a0, a1, SPLIT_32X64, st);
    case SPLIT_32: return launch_split_dual<32, 32>(a0, a1, SPLIT_32, st);
    default: break;
  }
  if (d.bn == V2_SMALL) return launch_dual<V2_SMALL, KE_ANY, KE_ANY, true>(a0, a1, d.first_is_1, st);
  if (d.bn == V2_B)
    return v2_k_end<V2_B>(a1.K) == KE_PAIR ? launch_dual<V2_B, KE_PAIR, KE_PAIR, false>(a0, a1, d.first_is_1, st)
                                           : launch_dual<V2_B, KE_PAIR, KE_SLICE, false>(a0, a1, d.first_is_1, st);
  GemmArgs a = a0;
  a.splitk_ws = splitk_ws;
  if (hipError_t e = launch_gemm_bf16_wgrad(a, st); e != hipSuccess) return e;
  a = a1;
  a.splitk_ws = splitk_ws;
  return launch_gemm_bf16_dgrad(a, st);
}

}  // namespace mlm
