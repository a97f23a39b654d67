// Dispatcher of the bf16 MFMA GEMM: operand layout -> translation unit.
#include <stdlib.h>
#include "gemm_bf16_split.h"

namespace mlm {

int gemm_v2_forced_bn() {
  static int forced = -1;
  if (forced < 0) {
    const char* e = getenv("MLM_GEMM_BN");
    const int v = e ? atoi(e) : 0;
    forced = (v == 128 || v == 192 || v == 256) ? v : 0;
  }
  return forced;
}

bool gemm_v2_group_off() {
  static const bool off = [] { const char* e = getenv("MLM_GEMM_GROUP"); return e && atoi(e) == 0; }();
  return off;
}

// Compute units of the current device, capped at the tail-split workspace's bound; one query per device.
int gemm_cu_count() {
  constexpr int kMaxDevices = 64, kCap = 256;
  static int cached[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return kCap;
  int n = __atomic_load_n(&cached[dev], __ATOMIC_RELAXED);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = kCap;
    if (n > kCap) n = kCap;
    __atomic_store_n(&cached[dev], n, __ATOMIC_RELAXED);
  }
  return n;
}

// (the cross-entropy GEMM always gets split-k scratch)
int gemm_bf16_ce_col_tiles(int M, int N, int K) {
  if (split_pick_alone<true, false, EPI_CE>(M, N, K, true).form) return (N + 63) / 64;      // (its forms are 64 columns wide)
  const int bn = v2_pick_bn<true, false, EPI_CE>(M, N, K, true);
  return (N + bn - 1) / bn;
}

hipError_t launch_gemm_bf16(const GemmArgs& a, hipStream_t st) {
  if (a.a_kc && !a.b_kc) return launch_gemm_bf16_fwd(a, st);
  if (a.a_kc && a.b_kc) return launch_gemm_bf16_dgrad(a, st);
  if (!a.a_kc && !a.b_kc) return launch_gemm_bf16_wgrad(a, st);
  return hipErrorInvalidValue;
}

}  // namespace mlm
