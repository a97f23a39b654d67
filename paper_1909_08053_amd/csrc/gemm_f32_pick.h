// Which fp32 GEMM kernel a problem takes: in pieces on the bf16 matrix cores (gemm_f32_pieces.hip) or one of the three of gemm_f32.hip, and which
// problems share a launch.  Host arithmetic only.
#pragma once
#include "schedule.h"

namespace mlm {

int gemm_cu_count();                    // compute units of the current device, at most 256

// Which of the three kernels: the smallest of their time estimates in microseconds, fitted to measured calls of them on MI355X
// (2048^3 and 4096^3, 1024 x {1024 .. 8192} x {1024 .. 8192}, 512 x 1536 x 512, 256 x 256 x {128 .. 512}, 800 x 1152 x 288).
//   * split kernel: a start-up, the serial eighth of k, and 52 TFLOP/s once the chip is full (its operands come through
//     the caches once per 32 x 32 tile);
//   * tile kernels: start-up plus rounds of two workgroups per CU; a last round with at most one workgroup per CU costs
//     a little more than half.  64 x 64: 31.5 us per round and 1024 k, 17.3 us with one workgroup per CU; 128 x 128: 119 / 63.
// 1024^3: 48 us (split), 23 us (64); 4096^3: 2540 (split), 985-1000 us (128: 139 TFLOP/s, the matrix cores' peak is 157), both in pieces now;
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
// idle: 16 x 16 where those find a unit each (256 x 256, 32 / 16, us, A and B k-contiguous and k-major: K = 128 3.0 / 2.6 and 3.0 / 2.7, 1024 8.9 / 4.1 and 8.3 / 4.6;
// below 128 k nothing to gain), or, at longer k, two a unit (256 x 512: K = 512 5.4 / 4.2 and 5.6 / 4.5, 1024 9.4 / 6.9 and 8.6 / 8.4, 2048 15.8 / 11.8 and 13.6 / 14.6).
// A 16 x 16 tile sums in chunks of 16 k, in eight chains like the other; short k only where they are of one
// length (a longest chain of 32 k in place of 24 at K = 192 is 4 % further off; from 512 k on uneven ones differ by 0.4 % at most).  The line at
// 512 k is cautious (256 x 512 x 256 3.7 / 3.3).
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
// k in four chains), against the kernels above: microseconds of t tiles in one launch, fitted to 800 calls (within 7 %; 64-wide tiles at long k
// up to 8 % low).  A round of 64-wide tiles, or of at most one 128-wide tile a unit, takes little less where units stay idle; more 128-wide
// tiles share the chip's power and take their share of it.
// Plain stores, means of three layouts, kernels above / in pieces: 1024 x 1024 x 4096 74 / 67 us and 768 x 2048 x 4096 137 / 119 (64-wide), 1024 x
// 3072 x 1024 57 / 47, 1024 x 4096 x 512 41 / 32, x 1024 73 / 55, 1536 x 4096 x 1024 110 / 85, 2048 x 6144 x 1024 196 / 147, 4096^3 980 / 704
// (128-wide); the wrong one of the two takes 147 us at 1024 x 1024 x 4096, 222 at 2048 x 6144 x 1024.  Few tiles, 256 x 1024 x 4096 35 / 57: the
// split kernel's workgroups find a unit each, those sizes stay with it.
inline double f32_pieces_us(int bt, double t, int K) {
  const int cus = gemm_cu_count();
  const double f = t / cus;
  if (bt == 128) {                                                                  // an even number of steps of 16 k
    const double step = f <= 1.0 ? 0.55 + (f > 0.5 ? 0.28 * (f - 0.5) : 0.0) : 0.67 * f > 1.05 ? 0.67 * f : 1.05;
    const int steps = (K + 31) / 32 * 2;
    const double rem = f / 2 - (double)(long)(f / 2);
    const double last = f > 2.0 && rem > 0.0 && rem < 0.5 ? (1.0 - 2.0 * rem) * (2.5 + 0.4 * steps) : 0.0;    // a last round nearly empty
    return (f <= 1.0 ? 5.8 : 7.3) + 2.0 * f + last + 1.02 * step * steps;
  }
  const double full = (double)(long)f, rem = f - full;                              // ... of 64 k
  if (f <= 1.0) return 6.7 - 0.8 * f + (0.655 + 0.25 * f) * ((K + 127) / 128 * 2);
  return 2.2 + 4.3 * (full + (rem > 0.0)) + (0.88 * full + (rem > 0.0 ? 0.71 + 0.17 * rem : 0.0)) * ((K + 127) / 128 * 2);
}
// ... and of t 64-wide tiles of the kernels above in one round, for a single product (a fit to 140 calls, closer than f32_launch_us to few
// units at work)
inline double f32_round_us(double t, int K) { return 3.0 + 1.9 * t / gemm_cu_count() + 1.08 * ((K + 63) / 64); }
// The tile of the product in pieces, or 0.  (At least a whole step of the 64-wide tile's: what is fetched ahead of the last step lies
// inside [0, K); and K up to where its 32-bit lane offsets reach.)
inline int f32_pieces_pick(int M, int N, int K) {
  const int b = f32_pick(M, N, K);
  if (b == 32 || K < 64 || K > kF32MaxK128) return 0;
  const double t128 = f32_pieces_us(128, f32_tiles(128, M, N), K), t64 = f32_pieces_us(64, f32_tiles(64, M, N), K);
  const double best = t128 < t64 ? t128 : t64;
  // (Where the prices are close, kernels above / in pieces: 1896 x 248 x 440 11.6 / 12.4 us, 3744 x 104 x 400 11.4 / 12.1, 2488 x 208 x 232 8.4 /
  // 9.3, 1472 x 1184 x 72 9.5 / 10.5, 352 x 3888 x 200 13.7 / 14.3; but 640 x 800 x 624 14.9 / 13.9, 296 x 3120 x 904 21.5 / 19.5, 336 x 2384 x 608
  // 15.9 / 14.3.)
  const double t = f32_tiles(b, M, N), f = t / gemm_cu_count();
  const double now = b == 64 && f <= 1.0 ? f32_round_us(t, K) : 0.98 * f32_launch_us(b, b == 64 ? 2 : 1, t, K);
  if (best >= 0.99 * now) return 0;
  return t128 < t64 ? 128 : 64;
}

// Launches that hold several problems.  No result gets further from the exact one by sharing a launch, so a tile's sums are at least
// as many chains over k as those of the kernel that its problem takes alone: eight in the split kernel, two in the 64-wide tiles, one
// in the 128-wide ones.  (Two chains in place of eight were up to 1.9 x further off, one in place of two 1.4 x: 55 tokens x 768 x 3072,
// 1.3e-7 against 7.5e-8.)  64-wide tiles can form eight; their workgroup then has a compute unit to itself.

// A weight gradient (0) and an input gradient (1) that do not depend on each other: the tile of one launch for both, or 0 for two
// launches, and the chains of its sums.  Tokens x width x vocabulary, the pass that forms dL included.
//   * Both take the split kernel: 32.
//   * Neither alone is formed in pieces: 64 where tiles of that size, those of longer k first, end a twentieth earlier than the two.  Two launches /
//     one: 373 x 1992 x 448 27 / 24 us, 403 x 832 x 560 28 / 18.5, 761 x 2424 x 680 63 / 58, and of eight chains, where one takes the split kernel
//     alone, 245 x 1096 x 944 37 / 24, 99 x 2600 x 720 30 / 21.
//   * Either alone is formed in pieces: one launch of 64-wide tiles in pieces, which is no less exact than either (four chains each), or two
//     launches.  Kernels above, as they were launched / two launches, in pieces where that is faster / one in pieces: 390 x 672 x 16032 278 / 358 /
//     198 us, 4554 x 216 x 1168 90 / 112 / 73, 1101 x 1032 x 1024 66 / 81 / 61, 469 x 760 x 648 21 / 30 / 20, 3646 x 304 x 1328 95 / 101 / 71; but 709 x
//     1928 x 2568 143 / 134 / 141, 1326 x 1640 x 1752 151 / 132 / 147.  (The kernels above were a little faster at 604 x 1824 x 200, 24 / 30 / 25,
//     128 x 2232 x 21512, 373 / 523 / 385, and 313 x 1392 x 3000, 71 / 77 / 75; in sums of two chains they are three times as far off.)
//   * The split kernel's workgroups find a unit each, which its price does not see: two launches (3792 x 192 x 248 28 / 72, 6000 x 1024 x 256
//     79 / 86).
struct F32DualPick { int tile, chains; bool pieces; };
// us of a product in a launch of its own
inline double f32_alone_us(int M, int N, int K) {
  const int bt = f32_pieces_pick(M, N, K), b = f32_pick(M, N, K);
  if (bt) return f32_pieces_us(bt, f32_tiles(bt, M, N), K);
  return b == 32 ? f32_split_us(M, N, K) : f32_launch_us(b, b == 64 ? 2 : 1, f32_tiles(b, M, N), K);
}
// us of one launch of nl longer and ns shorter 64-wide tiles in pieces
inline double f32_pieces_two_us(int nl, int Kl, int ns, int Ks) {
  const int cus = gemm_cu_count(), sl = (Kl + 127) / 128 * 2, ss = (Ks + 127) / 128 * 2;
  if (nl + ns <= cus) return f32_pieces_us(64, nl + ns, Kl);
  return 2.0 + two_batches(cus, nl, 4.2 + 0.91 * sl, ns, 4.2 + 0.91 * ss);
}
inline F32DualPick f32_dual_pick(int M0, int N0, int K0, int M1, int N1, int K1) {
  const int b0 = f32_pick(M0, N0, K0), b1 = f32_pick(M1, N1, K1), cus = gemm_cu_count();
  if (b0 == 32 && b1 == 32) return {32, 8, false};
  const bool split = b0 == 32 || b1 == 32;
  if (split && (b0 == 32 ? f32_tiles(32, M0, N0) : f32_tiles(32, M1, N1)) <= cus) return {0, 0, false};
  const bool swap = K1 > K0;                                   // l: the longer tiles, s: the others
  const int t0 = (int)f32_tiles(64, M0, N0), t1 = (int)f32_tiles(64, M1, N1);
  const int nl = swap ? t1 : t0, ns = swap ? t0 : t1;
  if (f32_pieces_pick(M0, N0, K0) || f32_pieces_pick(M1, N1, K1)) {
    const int lo = swap ? K0 : K1, hi = swap ? K1 : K0;
    const bool one = lo >= 64 && hi <= kF32MaxK128 &&
                     f32_pieces_two_us(nl, hi, ns, lo) < 0.97 * (1.5 + f32_alone_us(M0, N0, K0) + f32_alone_us(M1, N1, K1));
    return {one ? 64 : 0, one ? 4 : 0, one};
  }
  const double kl = (swap ? K1 : K0) / 1024.0, ks = (swap ? K0 : K1) / 1024.0;
  const double beside = nl <= cus ? ns * ks / (2 * cus - nl) + 0.5 * ks : kl;      // k that a longer tile does with others beside it
  const double both = 4.0 + (split || nl + ns <= cus ? two_batches(cus, nl, 17.3 * kl, ns, 17.3 * ks)
                             : beside < kl           ? 31.5 * beside + 17.3 * (kl - beside)
                                                     : two_batches(2 * cus, nl, 31.5 * kl, ns, 31.5 * ks));
  if (both >= 0.95 * (2.0 + f32_us(M0, N0, K0) + f32_us(M1, N1, K1))) return {0, 0, false};
  return {64, split ? 8 : 2, false};
}

// n weight gradients of the same K that do not depend on each other and are not formed in pieces: how they are launched.  The four of a layer
// shard, a launch each / as planned (tokens, width, ways of the split): 37, 832, 1 34 / 28 us and 61, 848, 2 23 / 18 (eight chains); 407, 1248, 4 70 / 46
// and 58, 2144, 4 46 / 34 (two); 22, 2720, 4 44 / 31 (128-wide); 44, 1376, 1 57 / 52 and 23, 904, 1 30 / 26 (128-wide ones in a launch of their own).  All
// in one launch of 128-wide tiles would be a little faster still at some sizes, and less exact.
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

// The same where some of them are formed in pieces: for each the tile, 128 or 64, or 0 for those that are launched as f32_group_plan says.  The
// 128-wide ones share a launch, and the 64-wide ones.  As each alone would be; or all in 64-wide tiles, or the others beside the ones that alone
// take these or the 128-wide ones, where that ends a twentieth earlier: no result gets further off by it.  (One sum of 128-wide tiles
// against the split kernel's eight chains: equal from 400 k on, 1.2 times as far off at 128.)  The four of a layer shard, kernels above / each in the tile
// it takes alone / all in 64-wide ones / the others in 64-wide, in 128-wide ones (tokens, width, ways of the split): 3264, 384, 2 59 / 95 / 52 / 52 /
// 168 us; 4096, 768, 8 73 / 114 / 63 / 66 / 206; 333, 768, 1 54 / 58 / 67 / 62 / 35; 769, 1088, 2 106 / 111 / 116 / 111 / 85; 651, 720, 1 90 / 96 /
// 103 / 96 / 71; 1024, 1024, 4 62 / 68 / 61 / 62 / 99; but 1024, 1024, 1 204 / 156 / 221 / 157 / 160, 2528, 800, 4 135 / 101 / 115 / 115 / 172.
struct F32GroupTiles { int tile[4]; };
inline F32GroupTiles f32_group_tiles(const int* M, const int* N, int n, int K) {
  F32GroupTiles best = {{0, 0, 0, 0}}, t = best;
  int rM[4], rN[4], rest = 0, split = 0, any = 0;
  for (int q = 0; q < n; ++q) {
    best.tile[q] = f32_pieces_pick(M[q], N[q], K);
    any += best.tile[q] != 0;
    if (best.tile[q]) continue;
    split += f32_pick(M[q], N[q], K) == 32;
    rM[rest] = M[q];
    rN[rest++] = N[q];
  }
  if (!any) return best;
  auto us = [&](const F32GroupTiles& g) {
    double t64 = 0.0, t128 = 0.0;
    for (int q = 0; q < n; ++q) (g.tile[q] == 128 ? t128 : t64) += g.tile[q] ? f32_tiles(g.tile[q], M[q], N[q]) : 0.0;
    return (t128 > 0.0 ? 1.5 + f32_pieces_us(128, t128, K) : 0.0) + (t64 > 0.0 ? 1.5 + f32_pieces_us(64, t64, K) : 0.0);
  };
  // (what the split kernel takes a round of tiles: f32_split_us does not see that few of them find a unit each)
  double t32 = 0.0;
  for (int q = 0; q < rest; ++q) t32 += f32_tiles(32, rM[q], rN[q]);
  const double rounds = (double)(long)((t32 + gemm_cu_count() - 1) / gemm_cu_count());
  double others = !rest ? 0.0 : 1.5 + (split == rest ? 3.2 + 3.7 * rounds * (K / 1024.0) : f32_group_plan(rM, rN, rest, K).us);
  if (rest == 1 && !split && f32_tiles(64, rM[0], rN[0]) <= gemm_cu_count()) others = 1.5 + f32_round_us(f32_tiles(64, rM[0], rN[0]), K);
  double least = 0.95 * (us(best) + others);
  const F32GroupTiles alone = best;
  for (int form = 0; form < 3; ++form) {             // all in 64-wide tiles; the rest in 64-wide ones; in 128-wide ones
    if (form == 2 && split && K < 400) break;
    for (int q = 0; q < n; ++q) t.tile[q] = form && alone.tile[q] ? alone.tile[q] : form == 2 ? 128 : 64;
    if (const double u = us(t); u < least) {
      least = u;
      best = t;
    }
  }
  return best;
}

}  // namespace mlm
