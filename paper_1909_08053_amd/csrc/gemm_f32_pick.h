// Which of the three fp32 GEMM kernels (gemm_f32.hip) a problem takes.  Host arithmetic only.
#pragma once
#include "schedule.h"

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
inline double f32_tiles(int b, int M, int N) { return (double)((M + b - 1) / b) * ((N + b - 1) / b); }
// t tiles of b x b (64 or 128) in one launch of a tile kernel
inline double f32_tile_us(int b, double t, int K) {
  const int cus = gemm_cu_count();
  const double two = b == 64 ? 31.5 : 119.0, one = b == 64 ? 17.3 : 63.0;
  const double full = (double)(long)(t / (2 * cus)), rem = t - full * 2 * cus;
  return (b == 64 ? 4.0 : 3.0) + (full * two + (rem > cus ? two : rem > 0 ? one : 0.0)) * (K / 1024.0);
}
inline double f32_split_us(int M, int N, int K) { return 3.0 + 6.0 * (K / 1024.0) + 2.0 * M * N * K / 52e6; }
inline int f32_pick(int M, int N, int K) {
  const double split = f32_split_us(M, N, K);
  const double t64 = f32_tile_us(64, f32_tiles(64, M, N), K), t128 = f32_tile_us(128, f32_tiles(128, M, N), K);
  if (split <= t64 && split <= t128) return 32;
  if (K > kF32MaxK128) return 64;
  return t64 <= t128 ? 64 : 128;
}

inline double f32_us(int M, int N, int K) {
  const int b = f32_pick(M, N, K);
  return b == 32 ? f32_split_us(M, N, K) : f32_tile_us(b, f32_tiles(b, M, N), K);
}

// A weight gradient (0) and an input gradient (1) that do not depend on each other: the tile of one launch for both, or 0 for two
// launches.  32 where both take the split kernel; 64 where tiles of that size, those of longer k first, end a twentieth earlier than
// the two.  Tokens x width x vocabulary, the pass that forms dL included, two launches / one: 512 x 1024 x 4096 115 / 93 us,
// 600 x 768 x 6000 167 / 129, 1000 x 1536 x 3200 202 / 182, 700 x 1920 x 2560 156 / 128, 1024 x 640 x 16384 467 / 387, 900 x 384 x
// 30592 716 / 613, 333 x 960 x 1032 36 / 33; but 1024 x 1024 x 8192, whose longer tiles are one per unit, 287 / 296.
inline int f32_dual_pick(int M0, int N0, int K0, int M1, int N1, int K1) {
  if (f32_pick(M0, N0, K0) == 32 && f32_pick(M1, N1, K1) == 32) return 32;
  const bool swap = K1 > K0;                                   // l: the longer tiles, s: the others
  const int cus = gemm_cu_count(), t0 = (int)f32_tiles(64, M0, N0), t1 = (int)f32_tiles(64, M1, N1);
  const int nl = swap ? t1 : t0, ns = swap ? t0 : t1;
  const double kl = (swap ? K1 : K0) / 1024.0, ks = (swap ? K0 : K1) / 1024.0;
  const double beside = nl <= cus ? ns * ks / (2 * cus - nl) + 0.5 * ks : kl;      // k that a longer tile does with others beside it
  const double both = 4.0 + (nl + ns <= cus ? 17.3 * kl
                             : beside < kl  ? 31.5 * beside + 17.3 * (kl - beside)
                                            : two_batches(2 * cus, nl, 31.5 * kl, ns, 31.5 * ks));
  return both < 0.95 * (2.0 + f32_us(M0, N0, K0) + f32_us(M1, N1, K1)) ? 64 : 0;
}

// n weight gradients of the same K that do not depend on each other: the tile of one launch for all of them, or 0 for a launch
// each.  32 where each of them takes the split kernel; else the tiles of all share their partly filled last round.  The four of a
// layer shard, apart / together (tokens, width, FFN width, split): 1024, 1024, 4096, 1 225 / 208 us; the same split four ways 73 / 57;
// 333, 768, 3072, 1 77 / 53; 900, 640, 2560, 1 126 / 85; 2048, 768, 3072, 1 315 / 240; 4096, 1024, 4096, 1 806 / 753; 33, 2048, 8192, 1
// 92 / 77; of 21 measured none slower.
inline int f32_group_pick(const int* M, const int* N, int n, int K) {
  double apart = 0.0, t64 = 0.0, t128 = 0.0;
  bool split = true;
  for (int q = 0; q < n; ++q) {
    split = split && f32_pick(M[q], N[q], K) == 32;
    apart += 2.0 + f32_us(M[q], N[q], K);
    t64 += f32_tiles(64, M[q], N[q]);
    t128 += f32_tiles(128, M[q], N[q]);
  }
  if (split) return 32;
  const double us64 = 2.0 + f32_tile_us(64, t64, K), us128 = K > kF32MaxK128 ? 1e30 : 2.0 + f32_tile_us(128, t128, K);
  if (us64 >= apart && us128 >= apart) return 0;
  return us64 <= us128 ? 64 : 128;
}

}  // namespace mlm
