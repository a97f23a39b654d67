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
// Tile of the split kernel.  The matrix operations of a 32 x 32 tile take one compute unit 3.7 us per 1024 k, and few such tiles leave units
// idle: 16 x 16 where those find a unit each (256 x 256, 32 / 16: K = 128 4.0 / 3.6 us, 1024 6.7 / 4.2; below 128 k nothing to
// gain), or, at longer k, two a unit (256 x 512: K = 512 7.2 / 5.7 us, 1024 11.5 / 9.0, 2048 19.8 / 15.6, but 256 4.7 / 5.3: twice the
// operands are fetched).  A 16 x 16 tile sums in chunks of 16 k, in eight chains like the other; short k only where they are of one
// length (a longest chain of 32 k in place of 24 at K = 192 is 4 % further off; from 512 k on uneven ones differ by 0.4 % at most).
inline int f32_split_tile_of(int M, int N, int K) {
  const double t16 = f32_tiles(16, M, N);
  return (K % 128 == 0 && K > 0 && t16 <= gemm_cu_count()) || (K % 16 == 0 && K >= 512 && t16 <= 2 * gemm_cu_count()) ? 16 : 32;
}
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

// Microseconds of one launch with t tiles of b x b in it, b = 64 or 128: per round of two tiles a unit, and per k tile of it.  (Fitted to
// the four weight gradients of 103 layer shards of 12 .. 2726 tokens and 320 .. 2048 wide: within 6 % and, 128-wide, 2 %.  At short k
// the stores decide, which f32_tile_us leaves out.)
inline double f32_launch_us(int b, int chains, double t, int K) {
  const int cus = gemm_cu_count(), nk = (K + (b == 64 ? 63 : 31)) / (b == 64 ? 64 : 32);
  const double full = (double)(long)(t / (2 * cus)), rem = t - full * 2 * cus;
  const double two = b == 128 ? 5.1 + 3.8 * nk : chains == 8 ? 3.5 + 2.2 * nk : 1.9 + 2.1 * nk;
  const double one = b == 128 ? 2.9 + 2.0 * nk : chains == 8 ? 2.5 + 1.0 * nk : 1.6 + 1.04 * nk;
  return (b == 128 ? 4.2 : 3.6) + (full + (rem > cus)) * two + (rem > 0 && rem <= cus ? one : 0.0);
}

// Products in pieces on the bf16 matrix cores (gemm_f32_pieces.hip), in 128-wide tiles (two a compute unit) or 64-wide ones (one, its
// k in four chains), against the kernels above: microseconds of t tiles in one launch.  A round of 64-wide tiles, or of at most one
// 128-wide tile a unit, takes little less where units stay idle; more 128-wide tiles share the chip's power and take their share of it.
// Three layouts, plain stores, kernels above / 128 / 64: 1024 x 1024 x 4096 75 / 147 / 65 us, 768 x 2048 x 4096 135 / 149 / 117,
// 1024 x 3072 x 1024 54 / 45 / 56, 1024 x 4096 x 512 39 / 29 / 45, x 1024 71 / 52 / 74, 1536 x 4096 x 1024 105 / 82 / 107,
// 2048 x 6144 x 1024 194 / 142 / 222, 4096^3 980 / 665 / 950; but 1024 x 1024 x 256 8.4 / 15 / 9.5, 256 x 1024 x 4096 36 / 148 / 57
// (the split kernel's workgroups find a unit each: those sizes stay with it).
inline double f32_pieces_us(int bt, double t, int K) {
  const int cus = gemm_cu_count();
  const double f = t / cus;
  if (bt == 128) {
    const double step = f <= 1.0 ? 0.55 + (f > 0.5 ? 0.28 * (f - 0.5) : 0.0) : 0.67 * f > 1.05 ? 0.67 * f : 1.05;   // per 16 k
    return 5.5 + 2.0 * f + step * ((K + 15) / 16);
  }
  const double full = (double)(long)f, rem = f - full;
  return 2.0 + 4.2 * (full + (rem > 0.0)) + (0.925 * full + (rem > 0.0 ? 0.74 + 0.185 * rem : 0.0)) * ((K + 63) / 64);
}
// The tile of the product in pieces, or 0.  (At least a whole step of the 64-wide tile's: what is fetched ahead of the last step lies
// inside [0, K); and K up to where its 32-bit lane offsets reach.)
inline int f32_pieces_pick(int M, int N, int K) {
  const int b = f32_pick(M, N, K);
  if (b == 32 || K < 64 || K > kF32MaxK128) return 0;
  const double t128 = f32_pieces_us(128, f32_tiles(128, M, N), K), t64 = f32_pieces_us(64, f32_tiles(64, M, N), K);
  const double best = t128 < t64 ? t128 : t64;
  if (best >= 0.97 * f32_launch_us(b, b == 64 ? 2 : 1, f32_tiles(b, M, N), K)) return 0;
  return t128 < t64 ? 128 : 64;
}

// Launches that hold several problems.  No result gets further from the exact one by sharing a launch, so a tile's sums are at least
// as many chains over k as those of the kernel that its problem takes alone: eight in the split kernel, two in the 64-wide tiles, one
// in the 128-wide ones.  (Two chains in place of eight were up to 1.9 x further off, one in place of two 1.4 x: 55 tokens x 768 x 3072,
// 1.3e-7 against 7.5e-8.)  64-wide tiles can form eight; their workgroup then has a compute unit to itself.

// A weight gradient (0) and an input gradient (1) that do not depend on each other: the tile of one launch for both, or 0 for two
// launches, and the chains of its sums.  32 where both take the split kernel; 64 where tiles of that size, those of longer k first, end
// a twentieth earlier than the two.  Tokens x width x vocabulary, the pass that forms dL included, two launches / one: 512 x 1024 x 4096
// 115 / 94 us, 600 x 768 x 6000 167 / 131, 1000 x 1536 x 3200 202 / 182, 700 x 1920 x 2560 155 / 129, 1024 x 640 x 16384 469 / 394, 333 x
// 960 x 1032 36 / 33; but 1024 x 1024 x 8192, whose longer tiles are one per unit, 287 / 296.  Eight chains: 390 x 672 x 16032 421 / 278, 128 x
// 2232 x 21512 633 / 373, 4554 x 216 x 1168 124 / 90; not where the split kernel's workgroups find a unit each, which its price
// does not see: 805 x 200 x 3176 60 / 65, 6000 x 1024 x 256 90 / 109.
struct F32DualPick { int tile, chains; };
inline F32DualPick f32_dual_pick(int M0, int N0, int K0, int M1, int N1, int K1) {
  const int b0 = f32_pick(M0, N0, K0), b1 = f32_pick(M1, N1, K1), cus = gemm_cu_count();
  if (b0 == 32 && b1 == 32) return {32, 8};
  const bool split = b0 == 32 || b1 == 32;
  if (split && (b0 == 32 ? f32_tiles(32, M0, N0) : f32_tiles(32, M1, N1)) <= cus) return {0, 0};
  const bool swap = K1 > K0;                                   // l: the longer tiles, s: the others
  const int t0 = (int)f32_tiles(64, M0, N0), t1 = (int)f32_tiles(64, M1, N1);
  const int nl = swap ? t1 : t0, ns = swap ? t0 : t1;
  const double kl = (swap ? K1 : K0) / 1024.0, ks = (swap ? K0 : K1) / 1024.0;
  const double beside = nl <= cus ? ns * ks / (2 * cus - nl) + 0.5 * ks : kl;      // k that a longer tile does with others beside it
  const double both = 4.0 + (split || nl + ns <= cus ? two_batches(cus, nl, 17.3 * kl, ns, 17.3 * ks)
                             : beside < kl           ? 31.5 * beside + 17.3 * (kl - beside)
                                                     : two_batches(2 * cus, nl, 31.5 * kl, ns, 31.5 * ks));
  if (both >= 0.95 * (2.0 + f32_us(M0, N0, K0) + f32_us(M1, N1, K1))) return {0, 0};
  return {64, split ? 8 : 2};
}

// n weight gradients of the same K that do not depend on each other: how they are launched.  The four of a layer shard, a launch each /
// as planned (tokens, width, ways of the split): 333, 768, 1 77 / 55 us; 1024, 768, 1 167 / 129; 1024, 1024, 4 73 / 60; 40, 768, 1 33 / 23 (eight
// chains); 59, 736, 2 35 / 14; 33, 2048, 1 92 / 77 (128-wide); 372, 1912, 1 319 / 286 and 841, 984, 1 190 / 176 (128-wide ones in a launch of their
// own).  All in one launch of 128-wide tiles would be a little faster still (1024, 1024, 1 219 / 206, 197), and less exact.
struct F32GroupPlan {
  int tile;              // of one launch for all of them; 0: a launch each
  int chains;            // of the sums in 64-wide tiles
  bool wide_apart;       // those that take the 128-wide tile alone share a launch of their own; `tile` is the others'
  double us;
};
inline F32GroupPlan f32_group_plan(const int* M, const int* N, int n, int K) {
  double apart = 0.0, t64 = 0.0, t128 = 0.0;
  int n32 = 0, n128 = 0, rest = 0, rM[4], rN[4];
  for (int q = 0; q < n; ++q) {
    const int b = f32_pick(M[q], N[q], K);
    apart += b == 32 ? 2.0 + f32_split_us(M[q], N[q], K) : f32_launch_us(b, b == 64 ? 2 : 1, f32_tiles(b, M[q], N[q]), K);
    t64 += f32_tiles(64, M[q], N[q]);
    n32 += b == 32;
    n128 += b == 128;
    if (b == 128) t128 += f32_tiles(128, M[q], N[q]);
    else { rM[rest] = M[q]; rN[rest++] = N[q]; }
  }
  F32GroupPlan p = {0, 0, false, apart};
  if (n < 2) return p;
  if (n32 == n) return {32, 8, false, apart};
  const int chains = n32 ? 8 : 2;
  const double one = f32_launch_us(64, chains, t64, K), wide = f32_launch_us(128, 1, t128, K);
  if (one < p.us) p = {64, chains, false, one};
  if (n128 == n && wide < p.us) p = {128, 1, false, wide};
  if (n128 && n128 < n) {
    const F32GroupPlan r = f32_group_plan(rM, rN, rest, K);
    if (wide + r.us < p.us) p = {r.tile, r.chains, true, wide + r.us};
  }
  return p;
}

}  // namespace mlm
