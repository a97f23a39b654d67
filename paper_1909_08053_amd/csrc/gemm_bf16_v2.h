// Second-generation bf16 MFMA GEMM main loop for gfx950, built on three CDNA4 features:
//   * global_load_lds_dwordx4: tiles go from HBM/L2 straight into LDS (no VGPR staging, no LDS-write
//     instructions, no VALU permutes), asynchronously, tracked by vmcnt.  Each wave instruction moves
//     64 lanes x 16 B = 1 KB into one contiguous LDS kilobyte, so the bank-conflict swizzle is applied on
//     the GLOBAL side: lane t fetches the 16-byte unit that belongs at LDS position t.
//   * ds_read_b64_tr_b16: an operand that is contiguous along m or n in memory (weights [in,out] in the
//     forward GEMM, both operands of the weight-gradient GEMM) stays in LDS in its natural [k][n] layout and
//     is transposed by the LDS read itself: 16 lanes read a 4(k) x 16(n) patch and each lane receives four
//     consecutive k of one column.  Two such reads give the same 8-consecutive-k operand registers that a
//     16-byte read of a k-contiguous tile gives, so both kinds of tiles feed the same MFMA loop.
//   * 160 KB LDS: a 256 x 256 block tile with a FOUR-stage ring of 32-deep k-slices (128 KB).  The operands of a
//     slice are pulled into registers while the slice before it is multiplied, so its stage is re-armed while it is
//     still being multiplied: three slices are in flight and one is landed, about 3500 MFMA clocks of prefetch
//     distance, one barrier per slice.
//   * v_mfma_f32_16x16x32_bf16: the same peak rate as the 32 x 32 x 16 shape, but a higher sustained rate on real
//     (normally distributed) operands, where the chip's power limit sets the clock: 2.04 PFLOP/s against 1.77 with the
//     matrix pipe alone, 1.60 against 1.45 with this loop's fragment reads and copies around it.
// k is walked in pairs of 32-deep slices.  K need not be a multiple of anything: the 16-byte units of the last pair that
// lie past K are fetched from sixteen zero bytes (one compare and select per copy, compiled in for such K only), or, K being
// an odd multiple of 32, the last pair starts one slice early and multiplies that slice as zeros.
//
// Tail split: when the tile count does not fill a whole number of rounds of the 256 CUs, the tiles of the last
// partial round are split along k into f pieces (f = floor(256 / remainder)); each piece writes an fp32 partial
// tile to a workspace and gemm_v2_fixup_kernel sums the pieces in a fixed order (deterministic) and applies
// the epilogue, whichever it is.
#pragma once
#include "gemm_bf16.h"
#include "lds_dma.h"
#include "schedule.h"
#include <limits.h>
#include <string.h>
#include <type_traits>

namespace mlm {

constexpr int V2_B = 256;                   // block tile edge (M and N)
constexpr int V2_BK = 32;                   // k per stage
constexpr int V2_SMALL = 128;               // block tile edge of the small tile
// rows of the block tile by its width (192 and DEEP: the middle tile, 128 x 192)
template <int BN, bool DEEP> constexpr int v2_bm() { return BN == V2_SMALL || (BN == 192 && DEEP) ? V2_SMALL : V2_B; }
// DEEP: the small tile in a launch of at most one workgroup per compute unit.  It has to hide its latencies by itself, so it
// runs 8 waves (two per SIMD) of 32 x 64 and, where a pair of slices arrives at once (a k-contiguous operand), keeps eight
// slices in its ring; in larger launches two workgroups share a compute unit, and 4 waves of 64 x 64 read a third less from
// LDS.  Measured, 96 slices: 4 / 8 waves on 256 tiles 44.7 / 33.1 us, on 512 tiles 49.1 / 51 us; 8 against 4 slices in the
// ring 31.1 / 35.4 us (both operands k-contiguous), 32.5 / 33.1 (one), and 37 / 33.5 (none, 128 slices).
template <int BN, bool DEEP> constexpr int v2_waves_m() { return BN == 192 || DEEP ? 4 : 2; }
template <int BN, bool DEEP> constexpr int v2_nw() { return BN == V2_SMALL && !DEEP ? 4 : 8; }
inline int v2_slices(int K) { return 2 * ((K + 2 * V2_BK - 1) / (2 * V2_BK)); }   // 32-deep slices walked: whole pairs
// How K ends: KE_PAIR on a whole pair of slices; KE_SLICE on the first slice of a pair (K an odd multiple of 32; the large tiles'
// kernels: with KE_ANY they are 4-8 % slower at 8192 x 3072 x 1568, and KE_PAIR's with this form's arithmetic 0.7-1 %); KE_ANY.  (The middle tile has no KE_SLICE: of 499
// such K its forward products and input gradients are 1.7 % slower in it in the mean, weight gradients 0.6 % faster.)
enum { KE_PAIR, KE_SLICE, KE_ANY };
template <int BN, bool DEEP = false> int v2_k_end(int K) {
  if (K % (2 * V2_BK) == 0) return KE_PAIR;
  return BN != V2_SMALL && !DEEP && K % V2_BK == 0 && K >= 2 * V2_BK ? KE_SLICE : KE_ANY;
}
// an n-contiguous B of 192 columns is copied pair by pair like a k-contiguous operand: 24 copies among eight waves, where a slice's 12 are two a
// wave, a quarter of them twice
template <int BN, bool DEEP> constexpr bool v2_pair_b() { return BN == 192 && DEEP; }
template <bool A_KC, bool B_KC, bool DEEP> constexpr int v2_stages() { return DEEP && (A_KC || B_KC) ? 8 : 4; }
// A's ring, then B's ring: 128 KB for a 256 x 256 tile, 64 KB (128 KB DEEP) for a 128 x 128 one
constexpr size_t v2_ring_bytes(int bm, int bn, int stages) { return (size_t)stages * V2_BK * 2 * (bm + bn); }

// What a copy reads for the 16-byte units past K.
static __device__ const uint4 v2_zero16 = {0u, 0u, 0u, 0u};

// Bank swizzle of the [k][row] tile layout (XOR on the 16-byte unit index of a 512-byte k-row).  A transposing read
// is served in two passes of 32 lanes; a pass reads 64 contiguous bytes (four units) of each of four consecutive
// k-rows, and every k-row starts at bank 0.  XORing the unit index with 4 (k & 3) sends the four rows to four different
// 64-byte slots of the 256-byte bank row, so a pass touches every bank once (checked by simulation and with the
// LDS bank-conflict counter: an earlier swizzle that only spread the rows over 128 bytes showed 50 % conflict cycles).
// The 16 x 16 x 32 MFMA's operand puts k = 8 g .. 8 g + 7 into lane group g = lane / 16, so a pass of its transposing
// read covers k-rows 0 .. 3 (or 4 .. 7) AND 8 .. 11 (12 .. 15), 32 bytes of each: bit 3 of k moves a row by another 32
// bytes.  With this term the reads are conflict-free (simulated).
__device__ __forceinline__ int v2_mn_swizzle(int k) { return ((k & 3) << 2) | (((k >> 3) & 1) << 1); }

// LDS position (16-byte unit inside the k-row) of logical row-chunk u of k-row k, and its inverse, for a [k][ROWS]
// tile.  256 rows: the XOR above.  192 rows: a k-row is 384 bytes = 24 units and starts at bank 0 or 32 alternately
// (384 = 256 + 128), so the four k-rows of a pass would pair up on the same 64-byte slots; rotating the rows with
// bit 1 of k set by four units sends the four 64-byte windows to the four different slots of the 256-byte bank row
// (slot = (6 k + position / 4) mod 4 -> 0, 2, 1, 3), wrap-around included.
// (192 rows, 16 x 16 x 32 reads: two more units for bit 3 of k, as above)
__device__ __forceinline__ int v2_mn_rot192(int k) { return (((k >> 1) & 1) << 2) + (((k >> 3) & 1) << 1); }
template <int ROWS> __device__ __forceinline__ int v2_mn_pos(int u, int k) {
  if (ROWS != 192) return u ^ v2_mn_swizzle(k);
  const int t = u + v2_mn_rot192(k);
  return t >= ROWS / 8 ? t - ROWS / 8 : t;
}
template <int ROWS> __device__ __forceinline__ int v2_mn_chunk(int pos, int k) {
  if (ROWS != 192) return pos ^ v2_mn_swizzle(k);
  const int t = pos - v2_mn_rot192(k);
  return t < 0 ? t + ROWS / 8 : t;
}

// Bank swizzle of a k-contiguous operand's ring: rows of 128 bytes (two consecutive k-slices side by side, eight
// 16-byte units), unit index XORed with this value.  A 16-byte read of the wave is served in four passes of 16 lanes, and a
// pass does not take 16 consecutive lanes: the first one holds lanes 0-3, 12-15 and 20-27, i.e. rows 0-3 and 12-15 of unit u
// and rows 4-11 of unit u + 1.  With row pairs numbered in order, both sets of values are closed under that + 1 and the 16
// lanes touch 16 different bank groups (with a value that permutes the bits of the pair number -- distinct for 16
// consecutive lanes -- every pass met a two-way conflict: half of the LDS cycles of these reads; the counter
// now shows 1-12 % of a kernel's, epilogue included; the 8.3B-shape step 1797 -> 1791 us: the reads were mostly hidden).
__device__ __forceinline__ int v2_kc_swizzle(int row) { return (row >> 1) & 7; }

// Per-lane source pointers of one operand's DMA copies (NP 1-KB copies per wave).
//  * k-contiguous operand (KC): the ring holds two PAIRS of slices; a pair is [256 rows][64 k] = 128 bytes per row,
//    so one copy instruction fetches 8 rows x one full 128-byte line (fetching the two 64-byte halves separately,
//    slice by slice, costs twice the cache-line requests and was measured 40 % slower on the copy side).  A pair
//    takes 2 QPW copies per wave and is fetched once every two slices.
//  * operand contiguous along m / n (MN): a slice is [32 k][256 rows] = 512 bytes per k, QPW copies per slice.
// ANY_K (KE_ANY): units past K are read from v2_zero16.  A template parameter: the compare and select per copy cost 2-4 % of a
// large GEMM.
// PR: copied pair by pair, as every KC operand is.
template <bool KC, bool PR, int NP_, bool ANY_K, int ROWS>
struct V2Src {
  static constexpr int NP = NP_;       // PR: 1-KB copies per wave and PAIR (rows / (8 waves)); else per wave and slice
  // MN: a slice is ROWS / 16 one-KB copies; where that is no multiple of the wave count (192 rows: 12 copies, 8
  // waves x 2) the surplus copies repeat the last one (same source, same destination: harmless, keeps the per-wave
  // copy count -- and with it the vmcnt bookkeeping -- uniform)
  static constexpr int LAST = PR ? (1 << 20) : ROWS / 16 - 1;
  const bf16* p[NP];
  int kofs[NP];    // k of this lane's unit inside the pair (PR) / slice
  int kleft;       // K - k_begin: units with k >= kleft are zeros
  size_t step;     // elements to advance per 32-deep k-slice
  __device__ __forceinline__ void init(const bf16* P, int ld, int row0, int nrows, int k_begin, int K, int wave, int lane) {
    kleft = K - k_begin;
    if (KC) {
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int row = (wave * NP + q) * 8 + (lane >> 3);
        kofs[q] = ((lane & 7) ^ v2_kc_swizzle(row)) * 8;
        p[q] = P + (size_t)min(row0 + row, nrows - 1) * ld + k_begin + kofs[q];
      }
      step = V2_BK;
    } else {
      // unit u of k-row holds row-chunk u ^ v2_mn_swizzle(k)
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int g = 64 * min(wave * NP + q, LAST) + lane;      // linear 16-byte unit of the slice buffer
        const int k = g / (ROWS / 8);                            // (PR: the pair's two buffers follow one another)
        const int u = v2_mn_chunk<ROWS>(g % (ROWS / 8), k);
        kofs[q] = k;
        p[q] = P + (size_t)(k_begin + k) * ld + min(row0 + u * 8, nrows - 8);
      }
      step = (size_t)V2_BK * ld;
    }
  }
  // dst: LDS byte address of the pair's (KC) / slice's (MN) buffer; ks: first 32-deep k-slice of the pair / the slice,
  // relative to k_begin; wave_u: wave index as a uniform (SGPR) value
  __device__ __forceinline__ void issue_one(uint32_t dst, int wave_u, int ks, int q) const {
    const bf16* src = p[q] + (ptrdiff_t)ks * (ptrdiff_t)step;
    if (ANY_K) src = ks * V2_BK + kofs[q] < kleft ? src : reinterpret_cast<const bf16*>(&v2_zero16);
    dma16(src, dst + min(wave_u * NP + q, LAST) * 1024);
  }
  __device__ __forceinline__ void issue(uint32_t dst, int wave_u, int ks) const {
#pragma unroll
    for (int q = 0; q < NP; ++q) issue_one(dst, wave_u, ks, q);
  }
};

// Operand registers of the 16 x 16 x 32 MFMA for the 16-row tile starting at row `r0`: lane l holds k = 8 (l / 16) ..
// + 7 (the whole 32-deep slice is one MFMA deep) of row r0 + l % 16.
template <bool KC, int ROWS>
__device__ __forceinline__ bf16x8 v2_frag16(const unsigned char* ring, int stage, int r0, int lane) {
  constexpr int OPB = ROWS * V2_BK * 2;       // bytes of one k-slice of the operand
  const int l16 = lane & 15, lg = lane >> 4;
  if (KC) {
    const int row = r0 + l16;
    const int u = (stage & 1) * 4 + lg;
    return *reinterpret_cast<const bf16x8*>(ring + (stage >> 1) * (2 * OPB) + row * 128 +
                                            ((u ^ v2_kc_swizzle(row)) << 4));
  } else {
    // two transposing reads: lane j of a group addresses 4 rows (r0 + 4 (j % 4) ..) of k-row 8 g + 4 r + j / 4 and
    // lane i receives k = 8 g + 4 r .. + 3 of row r0 + i
    const unsigned char* op_base = ring + stage * OPB;
    const int u = (r0 >> 3) + ((l16 & 3) >> 1);
    v4s_t h[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = 8 * lg + 4 * r + (l16 >> 2);
      h[r] = lds_read_tr16(op_base + k * (ROWS * 2) + (v2_mn_pos<ROWS>(u, k) * 16) + (l16 & 1) * 8);
    }
    const v8s_t v = __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
}

struct V2Plan {
  int tiles_m, tiles_n, full_tiles, tail_tiles, split;   // grid = full_tiles + tail_tiles * split
  int bm, bn;                                             // tile: 256 x 256, 256 x 192, 128 x 192 or 128 x 128
  int window, strip, long_pieces;                         // walk over the tiles (v2_xcd_order, v2_tile_of; v2_set_walk)
  double cost;                                            // estimated kernel time in microseconds (host side only)
  int grid() const { return full_tiles + tail_tiles * split; }
  bool deep() const { return bn == 128 && grid() <= gemm_cu_count(); }   // one workgroup per compute unit: eight-slice ring
};

// Walk over the tiles.  Every XCD has its own L2, so the 32 tiles that its compute units work on at a time (64 of the small
// tile) should lie close together: 4 x 8 tiles read 12 operand panels, 1 x 32 read 33.  Workgroup ids go to the XCDs in turn.
//   strip = 0: ids straight to tiles, tile row fastest.  Good patches where the number of tile rows is a multiple of 32, and
//   otherwise up to all tile rows or all columns for every XCD.
//   Else v2_xcd_order: of every window of ids that is resident at a time, the ids of one XCD (congruent mod 8) take CONSECUTIVE
//   positions of the walk of v2_tile_of: the shorter side of the output is cut into strips `strip` tiles wide (the last takes
//   what is left); a strip is walked along the longer side, every other one backwards, a row of `strip` tiles at a time.
__host__ __device__ inline int v2_xcd_order(int id, int total, int window) {
  const int base = total <= window ? 0 : (int)((unsigned)id / (unsigned)window) * window;   // (a division is 0.07 us ahead of the first copy)
  const int cnt = total - base < window ? total - base : window;
  const int p = id - base, x = p & 7, per = cnt >> 3, more = cnt & 7;
  return base + x * per + (x < more ? x : more) + (p >> 3);
}
__host__ __device__ inline void v2_tile_of(const V2Plan& p, int q, int* tile_m, int* tile_n) {
  if (p.strip == 0) {
    *tile_n = (int)((unsigned)q / (unsigned)p.tiles_m);
    *tile_m = q - *tile_n * p.tiles_m;
    return;
  }
  const bool rows = p.tiles_m <= p.tiles_n;                         // strips of tile rows, walked along the columns
  const int cross = rows ? p.tiles_m : p.tiles_n, along = rows ? p.tiles_n : p.tiles_m;
  const int s = p.strip >= cross ? 0 : (int)((unsigned)q / (unsigned)(p.strip * along)), r = q - s * (p.strip * along);
  const int left = cross - s * p.strip, w = left < p.strip ? left : p.strip;
  int l = (int)((unsigned)r / (unsigned)w);
  const int c = s * p.strip + r - l * w;
  if (s & 1) l = along - 1 - l;
  *tile_m = rows ? c : l;
  *tile_n = rows ? l : c;
}
// Operand bytes (per k) of the busiest XCD, over the first two windows of ids, in strips of w.
inline long v2_walk_cost(const V2Plan& p, int window, int w) {
  const int tiles = p.tiles_m * p.tiles_n;
  const bool rows = p.tiles_m <= p.tiles_n;
  const int cross = rows ? p.tiles_m : p.tiles_n, along = rows ? p.tiles_n : p.tiles_m;
  const int bc = rows ? p.bm : p.bn, bl = rows ? p.bn : p.bm, len = w * along;
  long cost = 0;
  for (int base = 0; base < tiles && base < 2 * window; base += window) {
    const int cnt = tiles - base < window ? tiles - base : window;
    long busiest = 0;
    for (int x = 0; x < 8; ++x) {
      int q = base + x * (cnt >> 3) + (x < (cnt & 7) ? x : cnt & 7);
      const int end = q + (cnt >> 3) + (x < (cnt & 7));
      int nc = 0, lo = along, hi = -1;                 // panels across; first and last panel along
      while (q < end) {                                // strip by strip
        const int s = q / len, left = cross - s * w, sw = left < w ? left : w;
        const int stop = s * len + sw * along < end ? s * len + sw * along : end;
        int l0 = (q - s * len) / sw, l1 = (stop - 1 - s * len) / sw;
        nc += l1 > l0 ? sw : stop - q;
        if (s & 1) { const int t = l0; l0 = along - 1 - l1; l1 = along - 1 - t; }
        if (l0 < lo) lo = l0;
        if (l1 > hi) hi = l1;
        q = stop;
      }
      const long c = (long)nc * bc + (hi >= lo ? (long)(hi - lo + 1) * bl : 0);
      if (c > busiest) busiest = c;
    }
    cost += busiest;
  }
  return cost;
}
// The same with ids straight to tiles: an XCD meets every (R / gcd(R, 8))-th tile row.
inline long v2_plain_cost(const V2Plan& p, int window) {
  const int tiles = p.tiles_m * p.tiles_n, R = p.tiles_m;
  const int step = R % 8 == 0 ? 8 : R % 4 == 0 ? 4 : R % 2 == 0 ? 2 : 1;
  long cost = 0;
  for (int base = 0; base < tiles && base < 2 * window; base += window) {
    const int cnt = tiles - base < window ? tiles - base : window, share = (cnt + 7) / 8;
    const int nr = R / step < share ? R / step : share;
    int nc = (cnt + R - 1) / R;                        // columns of the window; an XCD may skip some
    if (nc > share) nc = share;
    cost += (long)nr * p.bm + (long)nc * p.bn;
  }
  return cost;
}
// Operand elements per k of an XCD's share of the k-pieces (the fourth's), in the order of their numbers or part by part of k.
inline long v2_piece_cost(const V2Plan& p, bool parts) {
  const int total = p.tail_tiles * p.split;
  int row[64], col[64], n = 0;
  long cost = 0;
  for (int id = total > 3 ? 3 : 0; id < total && n < 64; id += 8, ++n) {
    const int t = parts ? v2_xcd_order(id, total, p.window) : id, piece = parts ? t / p.tail_tiles : t % p.split;
    int m, c;
    v2_tile_of(p, p.full_tiles + (parts ? t % p.tail_tiles : t / p.split), &m, &c);
    row[n] = 16 * m + piece;                         // (at most 16 pieces)
    col[n] = 16 * c + piece;
    bool r = true, l = true;
    for (int i = 0; i < n; ++i) { r = r && row[i] != row[n]; l = l && col[i] != col[n]; }
    cost += (r ? p.bm : 0) + (l ? p.bn : 0);
  }
  return cost;
}
// The walk of a launch: the strip width that costs least, where that is a tenth less than ids straight to tiles (equal patches
// are better apart: 96 tiles of 6 rows 1 us) and spares the busiest XCD four megabytes.  Of 329 launches that would gain the tenth, time in
// strips by the megabytes spared: up to 0.5 1.015 (the walk's divisions), 0.5 .. 1 0.996, 1 .. 4 0.974, more 0.93; but up to 4 the call that the
// launch is part of lost up to 9 % (520 tokens x 864 x 2000 forward 28.5 / 31.1 us, its second product reads what the strips left
// on one XCD), one in thirty of 500 drawn calls, and with this line none.  Measured in strips, 1450 shapes of up to 600 tiles: small tile
// 0.90 of the time on average
// (20 tile rows 0.98, 15 rows 0.88, 33 rows 0.83; 1920 x 4096 x 6144 131 -> 86 us), 192 wide 0.98, 256 wide 1.00.
// long_pieces: an XCD takes the k-pieces of tail tiles part by part of k; short ones are spread over the XCDs.  36 tiles x 6 pieces of
// 16 slices in order / spread 15.2 / 12.3 us, 96 x 2 of 32 17.7 / 14.5; 80 x 3 of 80 and 32 x 4 .. 128 x 2 large tiles of
// 24 .. 100 about 1 % of their steps in order's favour; dhf of 863 tokens x 512 x 22616, 28 x 9 pieces of 79, 98.7 -> 78.8 us of its call.  Not
// where the spread ones, whose number shares a factor with the eight XCDs, share as many panels: 7343 x 112 x 14688, 58 tiles x 4, 161 / 175,
// 5519 x 208 x 3160, 88 x 2, 72 / 75.  Without whole tiles the strips are the pieces' own.
inline void v2_set_walk(V2Plan* p, int window, int K, bool strips = false) {
  p->window = window;
  p->long_pieces = 0;
  p->strip = 0;
  const int cross = p->tiles_m <= p->tiles_n ? p->tiles_m : p->tiles_n;
  if (p->full_tiles) {
    const long plain = v2_plain_cost(*p, window), least = (1 << 21) / K;      // (4 MB in elements per k)
    long best = strips ? LONG_MAX : plain - (plain / 10 > least ? plain / 10 : least);
    for (int w = cross < 3 ? cross : 3; w <= cross && w <= 12; ++w) {
      const long c = v2_walk_cost(*p, window, w);
      if (c <= best) { best = c; p->strip = w; }
    }
  }
  if (p->tail_tiles == 0 || v2_slices(K) < (p->bn == V2_SMALL ? 48 : 16) * p->split) return;
  const long spread = v2_piece_cost(*p, false);
  long best = spread - spread / 10;
  const int first = p->strip, last = p->full_tiles || cross > 12 ? first : cross;
  for (int w = first;; w = w == 0 && last > 4 ? 4 : last) {        // the launch's strips; or one of 0, 4 and the whole width
    V2Plan t = *p;
    t.strip = w;
    const long c = v2_piece_cost(t, true);
    if (c <= best) { best = c; p->strip = w; p->long_pieces = 1; }
    if (w == last) break;
  }
}

inline bool v2_in_strips(V2Plan p, int window, int K) {
  v2_set_walk(&p, window, K);
  return p.strip != 0;
}

// Cost-model constants (microseconds, fitted to rocprofv3 kernel durations of unsplit two-round launches at two
// k-lengths each on MI355X): fixed cost of a tile (fill + epilogue) and cost of one 32-deep k-slice, for the
// 256 x 256 tile and for the 256 x 192 tile (either B layout).  The narrow tile does 3/4 of the MFMA work per slice
// in 0.88 of the time, so it wins where it saves a round or fills one and loses on long-k shapes whose last round
// can be split instead.  The fix-up kernel reads the pieces mostly out of the last-level cache.
// The small tile has two: `alone` with at most one workgroup per compute unit in the launch, else for two that share one
// (fitted to 60 .. 2600 tiles of 48 .. 256 slices).  The dearer price of an odd number of tile rows, or of few, comes from a
// walk that spread those over all XCDs: 1920 x 12800 x 8192 (15 tile rows) 591 us, 256-wide 347.  With v2_tile_of the cheaper
// one fits every row count (that shape: 373 / 350), so the line is cautious: where it keeps a large tile the small one is now up
// to a fifth faster (768 x 6400 x 6144: 74 / 90 us).
inline double v2_small_slice(int tiles_m) {
  if (tiles_m % 2 || tiles_m <= 10) return 0.72;
  return 0.46;
}
inline double v2_tile_cost(int bn, int nk, bool alone, double small_slice) {
  if (bn == V2_SMALL) return alone ? 4.5 + 0.24 * nk : 6.0 + small_slice * nk;
  return bn == V2_B ? 9.2 + 0.67 * nk : 8.0 + 0.59 * nk;
}
inline double v2_fixup_cost(double traffic_us) { return 3.0 + 0.6 * traffic_us; }

int gemm_v2_forced_bn();                    // MLM_GEMM_BN=128|192|256 forces a tile width where it exists, else 0

// Decide whether, and how far, to split the last partial round along k.  Cost model in microseconds: a tile costs
// its fixed part + the per-slice cost of its k-slices; the pieces write fp32 partial tiles at ~5 TB/s and the fix-up
// kernel reads them back.
inline V2Plan v2_plan(int M, int N, int K, bool allow_split, int bn = V2_B) {
  const int cus = gemm_cu_count();
  V2Plan p;
  p.bm = bn == V2_SMALL ? V2_SMALL : V2_B;
  p.bn = bn;
  p.tiles_m = (M + p.bm - 1) / p.bm;
  p.tiles_n = (N + bn - 1) / bn;
  const int tiles = p.tiles_m * p.tiles_n;
  const int per_round = bn == V2_SMALL ? 2 * cus : cus;     // two workgroups of the small tile share a compute unit
  const int rem = tiles % per_round;
  const int nk = v2_slices(K);
  int split = 1;
  const bool alone = tiles <= cus;
  const double ss = v2_small_slice(p.tiles_m);
  double tail = rem ? v2_tile_cost(bn, nk, alone, ss) : 0.0;   // unsplit tail round
  if (allow_split && rem != 0 && rem * 2 <= cus) {
    int smax = cus / rem;
    if (smax > 16) smax = 16;
    for (int sp = 2; sp <= smax; ++sp) {
      if (nk / sp < 8) break;                         // keep at least 8 k-slices per piece
      const double traffic = (double)rem * sp * (p.bm * (double)bn * 4.0) / 5.0e6;
      const double t = v2_tile_cost(bn, (nk + sp - 1) / sp, alone, ss) + traffic + v2_fixup_cost(traffic);
      if (t < tail) { tail = t; split = sp; }
    }
  }
  p.split = split;
  p.tail_tiles = split > 1 ? rem : 0;
  p.full_tiles = tiles - p.tail_tiles;
  p.cost = (tiles / per_round) * v2_tile_cost(bn, nk, false, ss) + tail;
  return p;
}

// The middle tile, 128 x 192 in eight waves of 32 x 96 with an eight-slice ring (four for a weight gradient: eight are 6 % slower up to 4000 k,
// 5-15 % faster from 5500 on), one workgroup per compute unit: where it gives every unit at most one tile and the small tile would give some units
// two, the others one or none at that one's pace (v2_choose).  Not beyond one tile a unit (4096 x 1920 x 2560, 320 tiles, 40 / 59; 8192 x 3072 x 1536,
// 1024, 73 / 93), and where the small tile has one a unit as well that is shorter (1024 x 3840 x 1920 19.5 / 23.4).
inline int v2_middle_tiles(int M, int N) { return ((M + V2_SMALL - 1) / V2_SMALL) * ((N + 191) / 192); }
inline int v2_small_tiles(int M, int N) { return ((M + V2_SMALL - 1) / V2_SMALL) * ((N + V2_SMALL - 1) / V2_SMALL); }
inline bool v2_middle_fits(int M, int N) {
  const int cus = gemm_cu_count();
  return !gemm_v2_forced_bn() && v2_middle_tiles(M, N) <= cus && v2_small_tiles(M, N) > cus;
}
inline V2Plan v2_middle_plan(int M, int N) {
  const int tm = (M + V2_SMALL - 1) / V2_SMALL, tn = (N + 191) / 192;
  V2Plan p = {};
  p.tiles_m = tm;
  p.tiles_n = tn;
  p.full_tiles = tm * tn;
  p.split = 1;
  p.bm = V2_SMALL;
  p.bn = 192;
  return p;
}

// One work item (pid) of one GEMM: the body of the kernels below.
// BN = 256: 2 x 4 waves of 128 x 64.  BN = 192: 4 x 2 waves of 64 x 96 -- a tile count of 32 x (N / 192) fills the 256 CUs
// where N / 256 column tiles leave a quarter of them idle (N = 1536: 256 tiles instead of 192) or a half-empty second
// round (N = 3072: 512 instead of 384).
// BN = 128: a 128 x 128 tile for outputs of too few large tiles.  Per flop it reads twice the operand bytes and more of LDS
// (two workgroups per compute unit: 0.215 us per tile and 32-deep slice, where a quarter of the 256 x 256 tile's is 0.17),
// but a launch of at most two tiles per compute unit neither leaves units idle nor splits k over fp32 partial tiles.
// Library call, forward layout, best large tile against it: 1024 x 1920 x 960 18.7 -> 10.6 us, 1024 x 3840 x 1920
// 33.7 -> 21.2, 3000 x 1152 x 1536 27.5 -> 16.7, 4096 x 2048 x 768 20.3 -> 16.9; 4096 x 4096 x 768 stays (27 against 31).
// Grouped weight gradients of 228 such tiles (8192 tokens, 1536 wide, split eight ways): 152 us in eight launches -> 81.
// PIECES: the launch may hold k-pieces.  A whole tile takes no division but the walk's: a 64-bit one for the k range of every work
// item, and the walk in strips, were 0.1 - 0.3 us of launches of 4 - 6.
template <bool A_KC, bool B_KC, int EPI, int BN, int KE, bool DEEP, bool PIECES = true>
__device__ __forceinline__ void gemm_v2_work_item(const GemmArgs& a, const V2Plan& plan, float* splitk_ws, int pid,
                                                  unsigned char* lds_raw) {
  static_assert(BN == V2_B || BN == 192 || BN == V2_SMALL, "tile widths");
  constexpr int NW = v2_nw<BN, DEEP>(), BM = v2_bm<BN, DEEP>(), ST = v2_stages<A_KC, B_KC, DEEP>();
  constexpr int WAVES_M = v2_waves_m<BN, DEEP>(), WAVES_N = NW / WAVES_M;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int OPB_A = BM * V2_BK * 2, OPB_B = BN * V2_BK * 2;   // bytes of one k-slice of either operand
  constexpr bool A_PR = A_KC, B_PR = B_KC || v2_pair_b<BN, DEEP>();
  // 1-KB copies per wave: per pair of slices for a k-contiguous operand, per slice otherwise
  constexpr int NPA = A_PR ? BM / (8 * NW) : BM / 16 / NW, NPB = B_PR ? BN / (8 * NW) : (BN / 16 + NW - 1) / NW;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;

  // Work item: a full tile, or one k-piece of a tail tile.  An XCD takes long pieces of the same part of k and of neighbouring
  // tiles, which share panels; short ones, whose time is the first misses', are spread (v2_set_walk).
  const int np_total = (int)((unsigned)(a.K + 2 * V2_BK - 1) / (2 * V2_BK));   // pairs of 32-deep slices of the problem
  int vt = pid, piece = 0, kt_begin = 0, kt_end = 2 * np_total;
  const bool whole = !PIECES || pid < plan.full_tiles;
  if (!whole) {
    int t = pid - plan.full_tiles;
    if (plan.long_pieces) {
      t = v2_xcd_order(t, plan.tail_tiles * plan.split, plan.window);
      piece = (int)((unsigned)t / (unsigned)plan.tail_tiles);
      vt = plan.full_tiles + t - piece * plan.tail_tiles;
    } else {
      const int tail = (int)((unsigned)t / (unsigned)plan.split);
      vt = plan.full_tiles + tail;
      piece = t - tail * plan.split;
    }
    kt_begin = 2 * (int)((unsigned)(np_total * piece) / (unsigned)plan.split);        // (at most 2^18 pairs, 16 pieces)
    kt_end = 2 * (int)((unsigned)(np_total * (piece + 1)) / (unsigned)plan.split);
  }
  int tile_m, tile_n;
  v2_tile_of(plan, vt, &tile_m, &tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int nk = kt_end - kt_begin;                  // even, >= 2

  V2Src<A_KC, A_PR, NPA, KE == KE_ANY, BM> sa;
  V2Src<B_KC, B_PR, NPB, KE == KE_ANY, BN> sb;
  sa.init((const bf16*)a.A, a.lda, m0, a.M, kt_begin * V2_BK, a.K, wave, lane);
  sb.init((const bf16*)a.B, a.ldb, n0, a.N, kt_begin * V2_BK, a.K, wave, lane);

  const uint32_t ldsA = lds_offset_of(lds_raw), ldsB = ldsA + ST * OPB_A;
  const unsigned char* ringA = lds_raw;
  const unsigned char* ringB = lds_raw + ST * OPB_A;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  constexpr int NKC = (A_PR ? 1 : 0) + (B_PR ? 1 : 0), NMN = 2 - NKC;
  // Four slices are always in flight or landed; past the end of k the last pair / slice is fetched again into a
  // stage nobody reads (keeps the vmcnt bookkeeping and the instruction stream free of tail cases).  Issue order of
  // the initial fill = the order the steady state would have produced: pair 0, slices 0 1, pair 1, slices 2 3.
  const int last_pair = nk / 2 - 1, last_slice = nk - 1;
  // KE_SLICE: the last pair starts one slice early, and its first slice, which the pair
  // before it has multiplied already, is multiplied as zeros.  shift = 1 for the piece that holds that pair.
  const int shift = KE == KE_SLICE && kt_end * V2_BK > a.K ? 1 : 0;
  // first 32-deep slice of pair pr / memory slice of walked slice ks
  auto pair_of = [&](int pr) { return 2 * pr - (pr == last_pair ? shift : 0); };
  auto slice_of = [&](int ks) { return ks - (ks >= nk - 2 ? shift : 0); };
#pragma unroll
  for (int h = 0; h < ST / 2; ++h) {
    if (A_PR) sa.issue(ldsA + h * 2 * OPB_A, wave_u, pair_of(min(h, last_pair)));
    if (B_PR) sb.issue(ldsB + h * 2 * OPB_B, wave_u, pair_of(min(h, last_pair)));
#pragma unroll
    for (int s = 2 * h; s < 2 * h + 2; ++s) {
      if (!A_PR) sa.issue(ldsA + s * OPB_A, wave_u, slice_of(min(s, last_slice)));
      if (!B_PR) sb.issue(ldsB + s * OPB_B, wave_u, slice_of(min(s, last_slice)));
    }
  }
  // The operand registers of what is multiplied next are read from LDS while the matrix cores work.  The slice hand-over sits inside
  // slice kt: wait for the copies of slice kt+1, barrier, then re-arm what slice kt leaves behind (its operands are all
  // in registers by then): an MN operand's stage gets slice kt+4; a KC operand's pair-stage is free after the ODD
  // slice of the pair and then gets the pair two ahead.  Copies are ISSUED ONE AT A TIME BETWEEN MFMAs: back-to-back 1-KB copies fill
  // the vector-memory queue and would stall the wave, and with it the matrix pipe, for hundreds of clocks.
  //
  // Copies per wave issued at the hand-over of an even slice: EV = NMN QPW; of an odd slice: OD = NKC 2 QPW + NMN QPW
  // (pairs first).  Copies return in order, so "slice kt+1 has landed" is a bound on the copies still outstanding:
  //   even kt: everything up to the hand-over of kt+1-ST must be done        -> ST - 2 hand-overs outstanding
  //   odd kt:  the pair issued first at the hand-over of kt+2-ST must be done -> that hand-over's slice and ST - 3 more
  constexpr int C_SLICE = (A_PR ? 0 : NPA) + (B_PR ? 0 : NPB);     // copies per wave that re-arm a slice stage
  constexpr int C_PAIR = (A_PR ? NPA : 0) + (B_PR ? NPB : 0);      // copies per wave that re-arm a pair stage
  constexpr int EV = C_SLICE, OD = C_PAIR + C_SLICE;
  constexpr int W_INIT = (ST - 1) * C_SLICE + (ST / 2 - 1) * C_PAIR, W_EVEN = (ST / 2 - 1) * (EV + OD);
  constexpr int W_ODD = NKC > 0 ? (ST / 2) * EV + (ST / 2 - 2) * OD : W_EVEN;
  static_assert(W_INIT < 64 && W_EVEN < 64, "vmcnt holds six bits");
  (void)NMN;
  // ---- 16 x 16 x 32 MFMAs: one MFMA spans the slice's 32 k, so a wave holds the fragments of ONE slice: NA of A, NB
  // of B.  MFMA order: A fragment outer, B fragment inner.  A fragment j is replaced by the next slice's behind
  // its last MFMA (j, NB - 1) and is next used about NMF - NB MFMAs later; the B fragments are double-buffered (the slice's
  // parity picks the set) and the next slice's are read right after the hand-over.  The hand-over (wait for the
  // copies of slice kt + 1, barrier) sits after MFMA HO, ahead of the first read of slice kt + 1; the copies that
  // re-arm slice kt's stage (all of its fragments were in registers before the slice began) follow it, one at a
  // time between the MFMAs.  Measured on the benchmark step: HO = 0 .. 2 within noise of each other, later
  // hand-overs slower (HO = 15: +0.5 %); B fragment outer with in-place replacement of both operands (A fragments
  // then have NA MFMAs between read and use) the same step time, 1 % slower on the logits GEMM.
  constexpr int NA = WM / 16, NB = WN / 16, NMF = NA * NB;
  constexpr int HO = 1;
  static_assert(HO + 1 + NB <= NMF, "the next slice's B fragments are read in this slice");
  floatx4 acc[NB][NA];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  bf16x8 fa[NA], fb[2][NB];
  wait_vmcnt<W_INIT>();                  // slice 0 landed
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int j = 0; j < NA; ++j) fa[j] = v2_frag16<A_KC, BM>(ringA, 0, wm0 + j * 16, lane);
#pragma unroll
  for (int i = 0; i < NB; ++i) fb[0][i] = v2_frag16<B_KC, BN>(ringB, 0, wn0 + i * 16, lane);

  // one 32-deep slice; PAR = parity of kt (compile time: it fixes the ring stage bits and the copy schedule)
  auto slice = [&](auto par_c, int kt) {
    constexpr int PAR = decltype(par_c)::value;
    const int stage = kt & (ST - 1), nstage = (kt + 1) & (ST - 1);
    constexpr int NC = PAR == 0 ? EV : OD;                 // copies to issue in this slice
    constexpr int NAFTER = NMF - HO - 1;                   // MFMAs after the hand-over
    const int pair_idx = pair_of(min((kt + ST - 1) >> 1, last_pair));   // PAR == 1: the pair ST / 2 ahead of this slice's pair
    const uint32_t pair_sel = (uint32_t)(((kt + ST - 1) >> 1) & (ST / 2 - 1));
    const uint32_t pair_off_a = pair_sel * (2 * OPB_A), pair_off_b = pair_sel * (2 * OPB_B);
    const int slice_idx = slice_of(min(kt + ST, last_slice));
    const uint32_t slice_off_a = (uint32_t)stage * OPB_A, slice_off_b = (uint32_t)stage * OPB_B;
#pragma unroll
    for (int idx = 0; idx < NMF; ++idx) {
      const int i = idx % NB, j = idx / NB;
      constexpr int CUR = PAR, NXT = 1 - PAR;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[CUR][i], fa[j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (idx == HO) {
        wait_vmcnt<PAR == 0 ? W_EVEN : W_ODD>();   // this wave's copies of slice kt+1 have landed
        // this wave's LDS reads of slice kt's stage (the last fragments, read at the end of slice kt - 1) have returned ...
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0) only
        // ... so after this bare s_barrier (no memory fence: a fence would also wait for the copies in flight)
        // everyone's part of slice kt+1 is in LDS and nobody reads slice kt's stage any more.
        __builtin_amdgcn_s_barrier();
      }
      if (idx > HO) {
        // fragments of slice kt + 1 into the registers that slice kt has finished with
#pragma unroll
        for (int q = 0; q < NB; ++q)
          if (idx == HO + 1 + q) fb[NXT][q] = v2_frag16<B_KC, BN>(ringB, nstage, wn0 + q * 16, lane);
#pragma unroll
        for (int q = 0; q < NA; ++q) {
          // one MFMA after the fragment's last one (q, NB - 1) -- directly behind it the read needs wait states, the
          // MFMA still reads the registers -- but inside the slice and not before the hand-over
          const int last = q * NB + NB < NMF - 1 ? q * NB + NB : NMF - 1;
          const int at = last > HO ? last : HO + 1;
          if (idx == at) fa[q] = v2_frag16<A_KC, BM>(ringA, nstage, wm0 + q * 16, lane);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if (HO + 1 + (c * NAFTER) / (NC > 0 ? NC : 1) != idx) continue;   // copy c goes after MFMA HO + 1 + (c NAFTER) / NC
          // order: A's pair, B's pair (odd slices only), then A's slice, B's slice
          int r = c;
          constexpr int KA = (PAR == 1 && A_PR) ? NPA : 0, KB = (PAR == 1 && B_PR) ? NPB : 0;
          constexpr int MA = A_PR ? 0 : NPA;
          if (r < KA) { sa.issue_one(ldsA + pair_off_a, wave_u, pair_idx, r); continue; }
          r -= KA;
          if (r < KB) { sb.issue_one(ldsB + pair_off_b, wave_u, pair_idx, r); continue; }
          r -= KB;
          if (r < MA) { sa.issue_one(ldsA + slice_off_a, wave_u, slice_idx, r); continue; }
          r -= MA;
          sb.issue_one(ldsB + slice_off_b, wave_u, slice_idx, r);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  typedef std::integral_constant<int, 0> c0_t;
  typedef std::integral_constant<int, 1> c1_t;
  // (no slice is peeled off: with a second copy of the two bodies the register allocator rotates accumulators through the
  // fragments' registers, and the loop then holds 7-16 wait states for the fragment reads that overwrite them)
  for (int kt = 0; kt < nk; kt += 2) {
    if (KE == KE_SLICE && shift && kt == nk - 2) {
      const bf16x8 zero = {};
#pragma unroll
      for (int j = 0; j < NA; ++j) fa[j] = zero;
#pragma unroll
      for (int i = 0; i < NB; ++i) fb[0][i] = zero;
    }
    slice(c0_t{}, kt);
    slice(c1_t{}, kt + 1);
  }
  EpilogueAux<BM, BN, WAVES_M, WAVES_N> aux;
  if (EPI == EPI_DGELU && whole) aux.request(a, m0, n0);
  // copies of the (clamped) last slices are still in flight and target the ring the epilogue reuses
  wait_vmcnt<0>();
  __syncthreads();

  if (!whole) {
    // fp32 partial tile: piece-major [tail tile][piece][BM][BN]
    const int l16 = lane & 15, lg = lane >> 4;
    float* dst = splitk_ws + ((size_t)(vt - plan.full_tiles) * plan.split + piece) * (BM * BN);
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const float4 v = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        *reinterpret_cast<float4*>(dst + (wm0 + j * 16 + l16) * BN + wn0 + i * 16 + 4 * lg) = v;
      }
    return;
  }
  gemm_epilogue<BM, BN, WAVES_M, WAVES_N, EPI>(a, acc, lds_raw, m0, n0, tile_n, &aux);
}

// (two workgroups of the small tile fit a compute unit)
template <bool A_KC, bool B_KC, int EPI, int BN, int KE, bool DEEP>
__global__ __launch_bounds__((v2_nw<BN, DEEP>() * 64), 2) void gemm_bf16_v2_kernel(GemmArgs a, V2Plan plan, float* splitk_ws) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int id = blockIdx.x;
  const int pid = plan.strip && id < plan.full_tiles ? v2_xcd_order(id, plan.full_tiles, plan.window) : id;
  gemm_v2_work_item<A_KC, B_KC, EPI, BN, KE, DEEP>(a, plan, splitk_ws, pid, lds_raw);
}

// An input gradient with the column sums of its left operand (a bias gradient) in the same launch: the workgroups behind the
// tiles sum columns, on compute units that the tiles leave idle.
template <int BN, int KE, bool DEEP>
__global__ __launch_bounds__((v2_nw<BN, DEEP>() * 64), 2) void gemm_bf16_v2_colsum_kernel(GemmArgs a, V2Plan plan, float* splitk_ws,
                                                                                           ColsumJob job) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int id = blockIdx.x, items = plan.full_tiles + plan.tail_tiles * plan.split;
  if (id >= items) {
    colsum_block<bf16, v2_nw<BN, DEEP>() * 64>(job, id - items, reinterpret_cast<float*>(lds_raw));
    return;
  }
  const int pid = plan.strip && id < plan.full_tiles ? v2_xcd_order(id, plan.full_tiles, plan.window) : id;
  gemm_v2_work_item<true, true, EPI_STORE, BN, KE, DEEP>(a, plan, splitk_ws, pid, lds_raw);
}

// Several independent GEMMs of one operand layout in ONE launch (plain-store epilogue, no k-split): the tiles of
// problem q follow those of problem q - 1 in the grid, so the launch pays the partially filled last round of the
// 256 CUs once instead of once per GEMM.  Used for the weight gradients of a layer shard, which nothing but the
// optimizer waits for: four GEMMs with 72 + 72 + 24 + 60 tiles at the 8.3B-shape 1/8 shard become one round.
constexpr int kMaxGroup = 4;
struct GemmGroup {
  int xcd_order;                       // one walk through the tiles of all problems
  int tile_begin[kMaxGroup + 1];       // first work item of each problem; tile_begin[n] = grid size
  int full;                            // whole tiles; the work items behind them are k-pieces of the last problem's last tiles
  GemmArgs args[kMaxGroup];
  V2Plan plan[kMaxGroup];
};

// SPLIT: with k-pieces (V2GroupSplit), whose partial tiles go to splitk_ws
template <bool A_KC, bool B_KC, int BN, int KE, bool DEEP, bool SPLIT>
__global__ __launch_bounds__((v2_nw<BN, DEEP>() * 64), 2) void gemm_bf16_v2_group_kernel(GemmGroup g, float* splitk_ws) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int id = blockIdx.x;
  const int pid = g.xcd_order && (!SPLIT || id < g.full) ? v2_xcd_order(id, g.full, g.plan[0].window) : id;
  // the problem index is uniform over the workgroup: select its arguments with scalar compares
  int q = 0;
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i) q += pid >= g.tile_begin[i] ? 1 : 0;      // (past the grid for problems that do not exist)
  GemmArgs a = g.args[0];
  V2Plan plan = g.plan[0];
  int first = g.tile_begin[0];
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i)
    if (q == i) { a = g.args[i]; plan = g.plan[i]; first = g.tile_begin[i]; }
  gemm_v2_work_item<A_KC, B_KC, EPI_STORE, BN, KE, DEEP, SPLIT>(a, plan, SPLIT ? splitk_ws : nullptr, pid - first, lds_raw);
}

// Tail tiles: sum the k-pieces in piece order (deterministic) and apply the epilogue to the fp32 sums.  A wave owns
// whole 256-column tile rows (a lane: 4 consecutive columns), so the row statistics of the cross-entropy epilogue are
// one wave reduction.  Grid: (bm / kFixRows row groups, tail tiles), 4 waves, kFixRows / 4 rows per wave.
constexpr int kFixRows = 8;
template <int EPI>
__global__ __launch_bounds__(256) void gemm_v2_fixup_kernel(GemmArgs a, V2Plan plan, const float* __restrict__ ws) {
  const int t = blockIdx.y;                          // tail tile
  int tile_m, tile_n;
  v2_tile_of(plan, plan.full_tiles + t, &tile_m, &tile_n);
  const int bm = plan.bm, bn = plan.bn;               // a partial tile is [bm][bn] floats
  const int m0 = tile_m * bm, n0 = tile_n * bn;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = n0 + lane * 4;
  const bool col_ok = n < a.N && lane * 4 < bn;       // N is a multiple of 8: a 4-column group is all in or all out
  const int nc = col_ok ? n : 0;
  const int lcol = lane * 4 < bn ? lane * 4 : 0;
  const float* base = ws + (size_t)t * plan.split * (bm * bn) + lcol;
  float bv[4] = {0.f, 0.f, 0.f, 0.f};
  if ((EPI == EPI_STORE || EPI == EPI_BIAS_GELU) && a.bias != nullptr) {
    const bf16x4 b = *reinterpret_cast<const bf16x4*>((const bf16*)a.bias + nc);
#pragma unroll
    for (int e = 0; e < 4; ++e) bv[e] = (float)b[e];
  }
  constexpr int RPW = kFixRows / 4;
  float v[RPW][4];
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int r = blockIdx.x * kFixRows + wave * RPW + i;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[i][e] = bv[e];
    for (int p = 0; p < plan.split; ++p) {
      const float4 x = *reinterpret_cast<const float4*>(base + (size_t)p * (bm * bn) + r * bn);
      v[i][0] += x.x; v[i][1] += x.y; v[i][2] += x.z; v[i][3] += x.w;
    }
  }
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int r = blockIdx.x * kFixRows + wave * RPW + i;
    const int m = m0 + r;
    if (m >= a.M) break;                              // wave-uniform
    const bool ok = col_ok;
    bf16x4 o;
    if (EPI == EPI_STORE) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16)v[i][e];
    } else if (EPI == EPI_BIAS_GELU) {
      bf16x4 pre;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        pre[e] = (bf16)v[i][e];
        o[e] = (bf16)gelu_fwd(v[i][e], a.gelu_tanh != 0);
      }
      if (ok) *reinterpret_cast<bf16x4*>((bf16*)a.aux + (size_t)m * a.ldaux + n) = pre;
    } else if (EPI == EPI_DGELU) {
      const bf16x4 g4 = *reinterpret_cast<const bf16x4*>((const bf16*)a.aux + (size_t)m * a.ldaux + nc);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16)(v[i][e] * gelu_bwd((float)g4[e], a.gelu_tanh != 0));
    } else if (EPI == EPI_CE) {
      float mx = -INFINITY;
      if (ok) mx = fmaxf(fmaxf(v[i][0], v[i][1]), fmaxf(v[i][2], v[i][3]));
      mx = wave_max(mx);
      const float mxl = ce_base(mx) * 1.4426950408889634f;
      float se = 0.f;
      if (ok) {
#pragma unroll
        for (int e = 0; e < 4; ++e) se += __builtin_amdgcn_exp2f(fmaf(v[i][e], 1.4426950408889634f, -mxl));
      }
      se = wave_sum(se);
      const int loc = a.targets[m] - a.v0 - n0;       // target column inside this tile, if 0 <= loc < 256
      if (ok && loc >= 0 && (loc >> 2) == lane) {
        float tv = v[i][0];
#pragma unroll
        for (int e = 1; e < 4; ++e) tv = ((loc & 3) == e) ? v[i][e] : tv;
        a.t_out[m] = tv;
      }
      if (lane == 0) {
        a.part_m[(size_t)tile_n * a.M + m] = mx;
        a.part_s[(size_t)tile_n * a.M + m] = se;
      }
      if (a.C == nullptr) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16)v[i][e];
    } else if (EPI == EPI_DLOGITS) {
      const float coef = (a.loss_w ? a.loss_w[m] : 1.0f) / a.loss_stats[1];
      const float Mrl = a.Mrow[m] * 1.4426950408889634f;
      const float invS = coef / a.Srow[m];
      const int loc = a.targets[m] - a.v0 - n;        // target column relative to this lane's first column
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float pz = __builtin_amdgcn_exp2f(fmaf(v[i][e], 1.4426950408889634f, -Mrl)) * invS;
        if (loc == e) pz -= coef;
        o[e] = (bf16)pz;
      }
    }
    if (ok) *reinterpret_cast<bf16x4*>((bf16*)a.C + (size_t)m * a.ldc + n) = o;
  }
}

// the rings or the epilogue's staging strips + reduction area, whichever is larger
template <bool A_KC, bool B_KC, int BN, bool DEEP> constexpr size_t v2_lds_bytes() {
  constexpr int WAVES_M = v2_waves_m<BN, DEEP>();
  constexpr size_t kEpi = GemmTile<v2_bm<BN, DEEP>(), BN, WAVES_M, v2_nw<BN, DEEP>() / WAVES_M>::LDS_EPI;
  constexpr size_t kRing = v2_ring_bytes(v2_bm<BN, DEEP>(), BN, v2_stages<A_KC, B_KC, DEEP>()), kLds = kRing > kEpi ? kRing : kEpi;
  static_assert(kLds <= (BN == V2_SMALL && !DEEP ? 80 : 160) * 1024, "LDS budget");
  return kLds;
}

// Ids resident at a time, a multiple of the eight XCDs.
template <int BN, bool DEEP> int v2_window() {
  const int n = (BN == V2_SMALL && !DEEP ? 2 : 1) * gemm_cu_count() & ~7;
  return n < 8 ? 8 : n;
}

// JOB: gemm_bf16_v2_colsum_kernel with `job`
template <bool A_KC, bool B_KC, int EPI, int BN, int KE, bool DEEP, bool JOB>
hipError_t launch_gemm_bf16_v2_ke(const GemmArgs& a, float* splitk_ws, const ColsumJob* job, hipStream_t st) {
  constexpr size_t kLds = v2_lds_bytes<A_KC, B_KC, BN, DEEP>();
  static LdsAttrOnce attr;         // per instantiation and device
  V2Plan plan = BN == 192 && DEEP ? v2_middle_plan(a.M, a.N) : v2_plan(a.M, a.N, a.K, splitk_ws != nullptr, BN);
  v2_set_walk(&plan, v2_window<BN, DEEP>(), a.K);
  if constexpr (JOB) {
    auto kern = gemm_bf16_v2_colsum_kernel<BN, KE, DEEP>;
    if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(plan.grid() + job->blocks), dim3(v2_nw<BN, DEEP>() * 64), kLds, st, a, plan, splitk_ws, *job);
  } else {
    auto kern = gemm_bf16_v2_kernel<A_KC, B_KC, EPI, BN, KE, DEEP>;
    if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(plan.grid()), dim3(v2_nw<BN, DEEP>() * 64), kLds, st, a, plan, splitk_ws);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (plan.tail_tiles) {
    hipLaunchKernelGGL((gemm_v2_fixup_kernel<EPI>), dim3(plan.bm / kFixRows, plan.tail_tiles), dim3(256), 0, st, a, plan,
                       splitk_ws);
    e = hipGetLastError();
  }
  return e;
}

// Tiles (work items without a k-split) of one problem.
inline int v2_tiles(const GemmArgs& a, int bm, int bn) { return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); }

// Estimated time (microseconds) of the tiles of all problems in one launch without a k-split.  The last round of the small
// tile, where it leaves compute units with one workgroup, runs at that one's pace (1200 tiles of 128 slices, 2.34 rounds: 155 us).
// lowest: the small tile at its cheaper price whatever the row counts (v2_small_slice).
inline double v2_group_cost(const GemmArgs* probs, int n, int bn, bool lowest = false) {
  const int bm = bn == V2_SMALL ? V2_SMALL : V2_B, cus = gemm_cu_count(), per_round = bn == V2_SMALL ? 2 * cus : cus;
  int tiles = 0;
  for (int q = 0; q < n; ++q) tiles += v2_tiles(probs[q], bm, bn);
  double ss = 0.0;                     // mean over the tiles
  for (int q = 0; q < n; ++q) ss += v2_small_slice(lowest ? 32 : (probs[q].M + bm - 1) / bm) * v2_tiles(probs[q], bm, bn) / tiles;
  const int nk = v2_slices(probs[0].K), rem = tiles % per_round;
  return (tiles / per_round) * v2_tile_cost(bn, nk, false, ss) + (rem ? v2_tile_cost(bn, nk, rem <= cus, ss) : 0.0);
}

// The large tiles of all problems in one launch, the last `rem` of problem `last` (the one of most tiles) in `split` k-pieces each:
// the same trade as in v2_plan for the partly filled last round that the problems share.  split = 0: none.
// The four gradients of a layer shard (tokens x width, ways of the split), the better of 128- and 256-wide tiles against this:
// 4096 x 2560, 4 176 / 162 us, 6176 x 2560, 4 253 / 214, 7000 x 2304, 3 309 / 264, 8192 x 1920, 2 347 / 328, 6000 x 1152 246 / 192, 4096 x 1056
// 173 / 124, 8192 x 1216 333 / 260; but not where short k favours the small tile, at its cheaper price: 1536 x 1056 51 / 61, 2000 x
// 1152 71 / 82.
struct V2GroupSplit { int last, rem, split; double cost; };
inline V2GroupSplit v2_group_split(const GemmArgs* probs, int n) {
  const int cus = gemm_cu_count(), nk = v2_slices(probs[0].K);
  V2GroupSplit g = {0, 0, 0, 1e30};
  int tiles = 0;
  for (int q = 0; q < n; ++q) {
    const int t = v2_tiles(probs[q], V2_B, V2_B);
    tiles += t;
    if (t > v2_tiles(probs[g.last], V2_B, V2_B)) g.last = q;
  }
  g.rem = tiles % cus;
  if (tiles < cus || g.rem == 0 || g.rem > v2_tiles(probs[g.last], V2_B, V2_B)) return g;
  for (int sp = 2; sp <= 16 && sp * g.rem <= cus && nk / sp >= 8; ++sp) {
    const double traffic = (double)g.rem * sp * (V2_B * (double)V2_B * 4.0) / 5.0e6;
    const double t = (tiles / cus) * v2_tile_cost(V2_B, nk, false, 0.0) + v2_tile_cost(V2_B, (nk + sp - 1) / sp, false, 0.0) + traffic +
                     v2_fixup_cost(traffic);
    if (t < g.cost) { g.cost = t; g.split = sp; }
  }
  return g;
}

template <bool A_KC, bool B_KC, int BN, int KE, bool DEEP, bool SPLIT>
hipError_t launch_gemm_bf16_v2_group_ke(const GemmArgs* probs, int n, const V2GroupSplit& sp, float* splitk_ws, hipStream_t st) {
  auto kern = gemm_bf16_v2_group_kernel<A_KC, B_KC, BN, KE, DEEP, SPLIT>;
  constexpr size_t kLds = v2_lds_bytes<A_KC, B_KC, BN, DEEP>();
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
  GemmGroup g;
  memset(&g, 0, sizeof(g));
  int total = 0;
  for (int q = 0; q < n; ++q) {
    const GemmArgs& a = probs[!SPLIT ? q : q == n - 1 ? sp.last : q == sp.last ? n - 1 : q];       // (sp.last goes last)
    g.args[q] = a;
    g.plan[q] = BN == 192 && DEEP ? v2_middle_plan(a.M, a.N) : v2_plan(a.M, a.N, a.K, false, BN);
    g.tile_begin[q] = total;
    total += g.plan[q].full_tiles;
  }
  g.full = total;
  if (SPLIT) {
    V2Plan& p = g.plan[n - 1];
    p.full_tiles -= sp.rem;
    p.tail_tiles = sp.rem;
    p.split = sp.split;
    g.full -= sp.rem;
    total = g.full + sp.rem * sp.split;
  }
  for (int q = n; q <= kMaxGroup; ++q) g.tile_begin[q] = total;
  for (int strips = 0; strips < 2; ++strips) {         // strips for all problems where one gains by them
    for (int q = 0; q < n; ++q) v2_set_walk(&g.plan[q], v2_window<BN, DEEP>(), probs[0].K, strips != 0);
    for (int q = 0; q < n; ++q) g.xcd_order |= g.plan[q].strip != 0;
    if (!g.xcd_order) break;
  }
  hipLaunchKernelGGL(kern, dim3(total), dim3(v2_nw<BN, DEEP>() * 64), kLds, st, g, splitk_ws);
  if (hipError_t e = hipGetLastError(); e != hipSuccess || !SPLIT) return e;
  hipLaunchKernelGGL((gemm_v2_fixup_kernel<EPI_STORE>), dim3(V2_B / kFixRows, sp.rem), dim3(256), 0, st, g.args[n - 1], g.plan[n - 1],
                     splitk_ws);
  return hipGetLastError();
}

template <bool A_KC, bool B_KC, int BN, bool DEEP, bool SPLIT = false>
hipError_t launch_gemm_bf16_v2_group(const GemmArgs* probs, int n, hipStream_t st, const V2GroupSplit& sp = {}, float* splitk_ws = nullptr) {
  switch (v2_k_end<BN, DEEP>(probs[0].K)) {
    case KE_PAIR: return launch_gemm_bf16_v2_group_ke<A_KC, B_KC, BN, KE_PAIR, DEEP, SPLIT>(probs, n, sp, splitk_ws, st);
    case KE_SLICE:
      if constexpr (BN != V2_SMALL && !DEEP) return launch_gemm_bf16_v2_group_ke<A_KC, B_KC, BN, KE_SLICE, DEEP, SPLIT>(probs, n, sp, splitk_ws, st);
    default: return launch_gemm_bf16_v2_group_ke<A_KC, B_KC, BN, KE_ANY, DEEP, SPLIT>(probs, n, sp, splitk_ws, st);
  }
}

bool gemm_v2_group_off();                   // MLM_GEMM_GROUP=0: every weight gradient of a layer shard in a launch of its own

// The 192-wide tile exists for all but the cross-entropy epilogues, the small tile for every epilogue but the one that
// recomputes the logits: take the one the cost model prices lowest for this shape.
template <bool A_KC, bool B_KC, int EPI> constexpr bool v2_has_narrow() {
  return B_KC || EPI == EPI_STORE || EPI == EPI_BIAS_GELU;
}
// The middle tile exists with the 192-wide one.
template <bool A_KC, bool B_KC, int EPI> constexpr bool v2_has_middle() { return v2_has_narrow<A_KC, B_KC, EPI>(); }
template <int EPI> constexpr bool v2_has_small() { return EPI != EPI_DLOGITS; }
template <bool A_KC, bool B_KC, int EPI>
int v2_pick_bn(int M, int N, int K, bool allow_split) {
  const int forced = gemm_v2_forced_bn();
  if (forced == V2_B || (forced == 192 && v2_has_narrow<A_KC, B_KC, EPI>()) || (forced == V2_SMALL && v2_has_small<EPI>()))
    return forced;
  int best = V2_B;
  double cost = v2_plan(M, N, K, allow_split, V2_B).cost;
  for (int bn : {192, V2_SMALL}) {
    if (bn == 192 ? !v2_has_narrow<A_KC, B_KC, EPI>() : !v2_has_small<EPI>()) continue;
    const double c = v2_plan(M, N, K, allow_split, bn).cost;
    if (c < cost) { cost = c; best = bn; }
  }
  return best;
}

// Microseconds of a product whose output fits the middle tile: in those, and in the plan's tiles with k-pieces.  Fitted to 963 products of K from 1000
// to 32000, split-k scratch given, the fix-up included, operands in the caches and not (4 % weight gradients, 9-12 % others), the last term of the pieces to
// whole steps: their fp32 partial tiles, some 50 MB, push the step's activations out of the memory-side cache, and the launches behind take longer.
// dhf 3000 x 1536 x 7648 takes 85 us in middle tiles and 80 in pieces, and its step (ragged, split four ways) 541 and 551.
template <bool A_KC, int EPI>
double v2_middle_us(int M, int N, int K) {
  const double nk = v2_slices(K), f = (double)v2_middle_tiles(M, N) / gemm_cu_count(), bytes = ((double)M + N) * K * 2.0 / 5.0e6;
  if (!A_KC) return 5.3 + (0.29 + 0.121 * f) * nk + 0.075 * bytes;
  return (EPI == EPI_STORE ? 5.9 : 10.0) + (0.232 + 0.118 * f) * nk + 0.27 * bytes;
}
template <bool A_KC>
double v2_pieces_us(const V2Plan& p, int M, int N, int K) {
  const double bytes = ((double)M + N) * K * 2.0 / 5.0e6, partial = (double)p.tail_tiles * p.split * p.bm * p.bn * 4.0 / 5.0e6;
  return (A_KC ? 0.9 * p.cost + 0.5 * bytes : 0.873 * p.cost + 0.23 * bytes) + 1.3 * partial;
}

// The tiles of a product in a launch of its own: the middle tile or those of the plan, and their price.  The middle one, where it fits:
//   * Against a plan without k-pieces (short k, or no scratch) from K = 192 on: of 332 products 0.97 of the time at 192 .. 320 k, 0.85 at 450 .. 1000, 0.79
//     beyond (worst 1.08, 2144 x 2864 x 256 8.6 / 9.1 us); with GeLU or its derivative, whose operands then come behind the last product, from 640 on
//     (.. 448 1.02, up to 1.11; 640 .. 1000 0.91).  3000 x 1536 x 1536 forward 21.0 / 18.8, 8192 x 768 x 1536 21.8 / 20.9, 2352 x 1792 x 1728 22.9 / 20.5,
//     7168 x 640 x 2560 31.4 / 28.6, wgrad 992 x 4144 x 1800 29.3 / 26.0, without scratch dgrad 3000 x 1536 x 30592 395 / 305.
//   * Against k-pieces by price.  Steps with dhf in pieces / in middle tiles, us: 5000 x 1152 x 10944 717 / 706, 2400 x 1920 x 8544 658 / 646, 4000 x 1344 x 9600
//     781 / 771; 3000 x 1536 x 11264 684 / 690, x 15296 1242 / 1289, 7000 x 640 x 20000 1222 / 1271.
struct V2Choice { int bn; bool middle; V2Plan plan; double us; };
template <bool A_KC, bool B_KC, int EPI>
V2Choice v2_choose(int M, int N, int K, bool allow_split) {
  V2Choice c = {v2_pick_bn<A_KC, B_KC, EPI>(M, N, K, allow_split), false, {}, 0.0};
  c.plan = v2_plan(M, N, K, allow_split, c.bn);
  c.us = c.plan.cost;
  if constexpr (v2_has_middle<A_KC, B_KC, EPI>()) {
    if (K < (EPI == EPI_STORE ? 192 : 640) || !v2_middle_fits(M, N)) return c;
    const double us = v2_middle_us<A_KC, EPI>(M, N, K);
    if (c.plan.split > 1 && us >= v2_pieces_us<A_KC>(c.plan, M, N, K)) return c;
    c = {192, true, v2_middle_plan(M, N), us};
  }
  return c;
}

template <bool A_KC, bool B_KC, int EPI, int BN, bool DEEP, bool JOB>
hipError_t launch_gemm_bf16_v2_bn(const GemmArgs& a, float* splitk_ws, const ColsumJob* job, hipStream_t st) {
  switch (v2_k_end<BN, DEEP>(a.K)) {
    case KE_PAIR: return launch_gemm_bf16_v2_ke<A_KC, B_KC, EPI, BN, KE_PAIR, DEEP, JOB>(a, splitk_ws, job, st);
    case KE_SLICE:
      if constexpr (BN != V2_SMALL && !DEEP) return launch_gemm_bf16_v2_ke<A_KC, B_KC, EPI, BN, KE_SLICE, DEEP, JOB>(a, splitk_ws, job, st);
    default: return launch_gemm_bf16_v2_ke<A_KC, B_KC, EPI, BN, KE_ANY, DEEP, JOB>(a, splitk_ws, job, st);
  }
}

template <bool A_KC, bool B_KC, int EPI, bool JOB = false>
hipError_t launch_gemm_bf16_v2(const GemmArgs& a, float* splitk_ws, hipStream_t st, const ColsumJob* job = nullptr) {
  const V2Choice c = v2_choose<A_KC, B_KC, EPI>(a.M, a.N, a.K, splitk_ws != nullptr);
  if constexpr (v2_has_middle<A_KC, B_KC, EPI>())
    if (c.middle) return launch_gemm_bf16_v2_bn<A_KC, B_KC, EPI, 192, true, JOB>(a, splitk_ws, job, st);
  if constexpr (v2_has_narrow<A_KC, B_KC, EPI>())
    if (c.bn == 192) return launch_gemm_bf16_v2_bn<A_KC, B_KC, EPI, 192, false, JOB>(a, splitk_ws, job, st);
  if constexpr (v2_has_small<EPI>())
    if (c.bn == V2_SMALL)
      return c.plan.deep()
                 ? launch_gemm_bf16_v2_bn<A_KC, B_KC, EPI, V2_SMALL, true, JOB>(a, splitk_ws, job, st)
                 : launch_gemm_bf16_v2_bn<A_KC, B_KC, EPI, V2_SMALL, false, JOB>(a, splitk_ws, job, st);
  return launch_gemm_bf16_v2_bn<A_KC, B_KC, EPI, V2_B, false, JOB>(a, splitk_ws, job, st);
}

// How n weight gradients (both operands k-major) are launched: together in tiles of bn, `split`: with the last round in k-pieces; apart
// (bn = 0) where they are no group or the shared last round gains nothing over separate launches with their k-splits.
struct V2GroupPlan { int bn; V2GroupSplit split; double alone; };          // alone: microseconds of the launches apart
inline V2GroupPlan v2_group_plan(const GemmArgs* probs, int n, bool have_ws) {
  V2GroupPlan p = {0, {0, 0, 0, 1e30}, 1e30};
  if (gemm_v2_group_off() || n < 2 || n > kMaxGroup) return p;
  double alone = 0.0;
  for (int q = 0; q < n; ++q) {
    const int M = probs[q].M, N = probs[q].N, K = probs[q].K;
    if (probs[q].epi != EPI_STORE || probs[q].bias != nullptr || K != probs[0].K) return p;
    alone += v2_plan(M, N, K, true, v2_pick_bn<false, false, EPI_STORE>(M, N, K, true)).cost + 2.0;   // + launch and drain
  }
  p.alone = alone;
  const double big = v2_group_cost(probs, n, V2_B), small = v2_group_cost(probs, n, V2_SMALL);
  const int forced = gemm_v2_forced_bn();
  const bool use_small = forced ? forced == V2_SMALL : small < big;
  if ((!forced || forced == V2_B) && have_ws) {
    const V2GroupSplit sp = v2_group_split(probs, n);
    const double whole = use_small ? v2_group_cost(probs, n, V2_SMALL, true) : big;
    if (sp.split && sp.cost < 0.97 * whole && sp.cost + 2.0 < alone) return {V2_B, sp, alone};
  }
  if ((use_small ? small : big) + 2.0 < alone) p.bn = use_small ? V2_SMALL : V2_B;
  return p;
}

// n weight gradients in one launch of middle tiles: where those find a unit each and the small ones do not, but not
//   * where launches apart, whose long k goes out in pieces, are priced lower: from some 15000 tokens on, 23288 x 1248 split four ways 342 / 276 us, 17024 x 528
//     259 / 195 (the price here fitted to 183 groups, within 6 %, operands in the caches and not);
//   * where the small tiles are walked in strips and these are not yet (v2_set_walk): 1646 x 1312, 4 34.0 / 27.9, 1600 x 1856, 8 27.9 / 24.6.
// Elsewhere, gradients of a layer shard, T x H split p ways, the best of the other forms / so, us: 520 x 816, 2 16.7 / 14.0, 1376 x 640 29.7 / 25.2, 1648 x 1184, 4
// 36.0 / 28.5, 5400 x 1184, 4 75.7 / 67.0, 9146 x 1664, 8 121 / 107; 180 groups 0.90 in the mean.
inline bool v2_group_middle(const GemmArgs* probs, int n, const V2GroupPlan& p) {
  if (gemm_v2_group_off() || gemm_v2_forced_bn() || n < 2 || n > kMaxGroup || probs[0].K < 192) return false;
  const int K = probs[0].K, cus = gemm_cu_count();
  int middle = 0, small = 0;
  double bytes = 0.0;
  for (int q = 0; q < n; ++q) {
    if (probs[q].epi != EPI_STORE || probs[q].bias != nullptr || probs[q].K != K) return false;
    middle += v2_middle_tiles(probs[q].M, probs[q].N);
    small += v2_small_tiles(probs[q].M, probs[q].N);
    bytes += ((double)probs[q].M + probs[q].N) * K * 2.0 / 5.0e6;
  }
  if (small <= cus || middle > cus) return false;
  if (6.1 + (0.313 + 0.117 * middle / cus) * v2_slices(K) + 0.229 * bytes >= 0.95 * p.alone) return false;
  bool small_strips = false;
  for (int q = 0; q < n; ++q) {
    if (v2_in_strips(v2_middle_plan(probs[q].M, probs[q].N), v2_window<192, true>(), K)) return true;
    small_strips = small_strips || v2_in_strips(v2_plan(probs[q].M, probs[q].N, K, false, V2_SMALL), v2_window<V2_SMALL, false>(), K);
  }
  return !small_strips;
}

// How a weight gradient a0 and an input gradient a1 that do not depend on each other are launched: together in tiles of bn
// (first_is_1: a1's tiles, the longer ones, lead), or apart (bn = 0).  Measured apart / together, the pass that forms dL included:
// 8192 tokens x 3072 x 6400 533 / 490 us, 8192 x 1536 x 51200 2300 / 2155, 3008 x 3072 x 12800 420 / 345, 1536 x 3072 x 2048
// 54.5 / 46.8, 6144 x 2560 x 3072 159 / 144; small tiles 320 x 1920 x 1000 24.1 / 15.4, 704 x 384 x 512 17.7 / 14.2.  Where either
// alone fills three quarters of the units it gains nothing: 3008 x 3072 x 4096 131 / 138, 4096 x 1920 x 6400 178 / 183.
struct V2Dual { int bn; bool first_is_1; };
inline V2Dual v2_dual(const GemmArgs& a0, const GemmArgs& a1) {
  V2Dual d = {0, v2_slices(a1.K) > v2_slices(a0.K)};
  const int forced = gemm_v2_forced_bn();
  const int cus = gemm_cu_count(), nk0 = v2_slices(a0.K), nk1 = v2_slices(a1.K);
  // + launch and drain.  Busy compute units clock higher while others idle, so an unsplit last round costs less than its tiles
  // do in full ones (192 large tiles 0.89); the narrow tile falls behind at very long k (1600 slices: 1105 us, not 952).
  auto alone = [&](const GemmArgs& a, int bn) {
    const V2Plan p = v2_plan(a.M, a.N, a.K, true, bn);
    const int nk = v2_slices(a.K), tiles = p.tiles_m * p.tiles_n, rem = tiles % cus;
    double c = p.cost + 2.0;
    if (bn != V2_SMALL && p.split == 1 && rem) c -= 0.45 * (1.0 - (double)rem / cus) * v2_tile_cost(bn, nk, false, 0.0);
    if (bn == 192 && nk > 1024) c += 0.06 * nk * ((tiles + cus - 1) / cus);
    return c;
  };
  double best = 0.98 * (alone(a0, v2_pick_bn<false, false, EPI_STORE>(a0.M, a0.N, a0.K, true)) +
                        alone(a1, v2_pick_bn<true, true, EPI_STORE>(a1.M, a1.N, a1.K, true)));
  auto price = [&](int bn, bool one_each) {
    const int bm = bn == V2_SMALL ? V2_SMALL : V2_B;
    const int n0 = ((a0.M + bm - 1) / bm) * ((a0.N + bn - 1) / bn), n1 = ((a1.M + bm - 1) / bm) * ((a1.N + bn - 1) / bn);
    if (one_each && n0 + n1 > cus) return 1e30;
    const double c0 = v2_tile_cost(bn, nk0, one_each, 0.46), c1 = v2_tile_cost(bn, nk1, one_each, 0.46);
    return 2.0 + (d.first_is_1 ? two_batches(cus, n1, c1, n0, c0) : two_batches(cus, n0, c0, n1, c1));
  };
  if ((!forced || forced == V2_B) && a0.K % (2 * V2_BK) == 0 && a1.K % V2_BK == 0 && a1.K >= 2 * V2_BK) {
    const double t = price(V2_B, false);
    if (t < best) { best = t; d.bn = V2_B; }
  }
  if ((!forced || forced == V2_SMALL) && price(V2_SMALL, true) < best) d.bn = V2_SMALL;
  return d;
}

// One translation unit per operand layout (keeps compile times parallel).
hipError_t launch_gemm_bf16_fwd(const GemmArgs& a, hipStream_t st);     // A k-contiguous, B n-contiguous
hipError_t launch_gemm_bf16_dgrad(const GemmArgs& a, hipStream_t st);   // both k-contiguous
hipError_t launch_gemm_bf16_wgrad(const GemmArgs& a, hipStream_t st);   // A m-contiguous, B n-contiguous

}  // namespace mlm
