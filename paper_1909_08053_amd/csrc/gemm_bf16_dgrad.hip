// bf16 GEMM instantiations for the input-gradient layout dX = dY W^T: A [M,K] k-contiguous (dY), B(k,n) = W[n,k]
// with W stored [in,out] = [N,K], i.e. k-contiguous as well.  Epilogues: plain store, GeLU' (fused dG = dY o GeLU'(G)).
#include "gemm_bf16_split.h"

namespace mlm {

hipError_t launch_gemm_bf16_dgrad(const GemmArgs& a, hipStream_t st) {
  switch (a.epi) {
    case EPI_STORE: return launch_gemm_bf16_any<true, true, EPI_STORE>(a, st);
    case EPI_DGELU: return launch_gemm_bf16_any<true, true, EPI_DGELU>(a, st);
    default: return hipErrorInvalidValue;
  }
}

template <int TM, int TN>
static hipError_t launch_split_colsum(const GemmArgs& a, const ColsumJob& j, int form, hipStream_t st) {
  constexpr size_t kTile = split_lds_bytes<TM, TN>(), kSums = colsum_lds_floats<bf16, 64 * kSplitWaves>() * sizeof(float);
  static LdsAttrOnce attr;
  const int tiles = split_tiles(form, a.M, a.N);
  return launch_split(&attr, gemm_bf16_split_colsum_kernel<TM, TN>, kTile > kSums ? kTile : kSums, tiles + j.blocks, st, a, j, tiles);
}

hipError_t launch_gemm_bf16_dgrad_colsum(const GemmArgs& a, const ColsumJob& j, hipStream_t st) {
  switch (split_pick_alone<true, true, EPI_STORE>(a.M, a.N, a.K, a.splitk_ws != nullptr).form) {
    case SPLIT_64: return launch_split_colsum<64, 64>(a, j, SPLIT_64, st);
    case SPLIT_32X64: return launch_split_colsum<32, 64>(a, j, SPLIT_32X64, st);
    case SPLIT_32: return launch_split_colsum<32, 32>(a, j, SPLIT_32, st);
    default: return launch_gemm_bf16_v2<true, true, EPI_STORE, true>(a, a.splitk_ws, st, &j);
  }
}

}  // namespace mlm
