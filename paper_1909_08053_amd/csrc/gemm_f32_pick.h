// Which of the three fp32 GEMM kernels (gemm_f32.hip) a problem takes.  Host arithmetic only.
#pragma once

namespace mlm {

int gemm_cu_count();                    // compute units of the current device, at most 256

// Which kernel: the smallest of three time estimates in microseconds, fitted to measured calls of the three on MI355X
// (2048^3 and 4096^3, 1024 x {1024 .. 8192} x {1024 .. 8192}, 512 x 1536 x 512, 256 x 256 x {128 .. 512}, 800 x 1152 x 288).
//   * split kernel: a start-up, the serial eighth of k, and 52 TFLOP/s once the chip is full (its operands come through
//     the caches once per 32 x 32 tile);
//   * tile kernels: start-up plus rounds of two workgroups per CU; a last round with at most one workgroup per CU costs
//     a little more than half.  64 x 64: 31.5 us per round and 1024 k, 17.3 us with one workgroup per CU; 128 x 128: 119 / 63.
// 1024^3: 48 us (split), 23 us (64); 4096^3: 2540 (split), 985-1000 us (128: 139 TFLOP/s, the matrix cores' peak is 157);
// 256 x 256 x 512: < 10 us (split).  (One 64 x 64-tile kernel on the vector ALUs, 15.7 TFLOP/s at most, took
// 200 us for 1024^3 and 60 us for 256 x 256 x 512 before.)
// (A tile's lane offsets are 32-bit byte counts: 127 rows of a k-contiguous operand stay below 4 GiB up to this K, 63 rows up
// to the 2^24 that mlm_gemm accepts.)
constexpr int kF32MaxK128 = 1 << 23;
inline int f32_pick(int M, int N, int K) {
  auto tiles = [&](int b) { return (double)((M + b - 1) / b) * ((N + b - 1) / b); };
  const int cus = gemm_cu_count();
  auto rounds = [&](int b, double two, double one) {
    const double t = tiles(b), full = (double)(long)(t / (2 * cus)), rem = t - full * 2 * cus;
    return full * two + (rem > cus ? two : rem > 0 ? one : 0.0);
  };
  const double k = K / 1024.0;
  const double split = 3.0 + 6.0 * k + 2.0 * M * N * K / 52e6;
  const double t64 = 4.0 + rounds(64, 31.5, 17.3) * k, t128 = 3.0 + rounds(128, 119.0, 63.0) * k;
  if (split <= t64 && split <= t128) return 32;
  if (K > kF32MaxK128) return 64;
  return t64 <= t128 ? 64 : 128;
}

}  // namespace mlm
