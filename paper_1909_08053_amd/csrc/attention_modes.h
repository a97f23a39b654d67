// How the bf16 attention kernels divide a launch into workgroups (the kernels: attention_bf16.hip).  Host arithmetic only.
#pragma once

namespace mlm {

int gemm_cu_count();                    // compute units of the current device, at most 256

// Forward and dQ: WIDE and PAIR take 128 rows of one (batch, head) pair per workgroup, SPLIT 64.
enum AttnMode { ATTN_WIDE, ATTN_PAIR, ATTN_SPLIT };

// All workgroups of a (batch, head) pair run on one XCD (an eighth of the compute units), and the eight XCDs take the pairs in
// turn: what decides is the number of 128-row workgroups of the busiest XCD next to their number overall.  Measured as WIDE,
// PAIR, SPLIT (us, forward + dQ, compute units 256, s x pairs):
//   SPLIT while its workgroups, twice as many, fit the compute units overall and on the XCD; causal ones, of which the short
//   ones make room for the long ones, up to two per unit there.  d = 96: 1024 x 8 causal 47, 44, 34; 3072 x 4 causal 120, 103,
//   77, but full 125, 110, 145; 4096 x 4 full 170, 152, 197; 768 x 20 full 39, 39, 57.  d = 128: 8192 x 1 causal 434, 328, 458.
//   PAIR up to one workgroup per compute unit: a causal chain of steps halved.  And beyond, causal, while the busiest XCD has
//   one or two pairs and two workgroups per unit, or three pairs and one and a half: its longest chain alone is then the
//   launch's time.  d = 96: 4096 x 16 causal 243, 180; 2048 x 24 causal 126, 107; 8192 x 8 causal 381, 324.
//   WIDE for the rest.  d = 96: 1024 x 64 causal 76, 91; 2048 x 32 causal 132, 135; 4096 x 20 causal 270, 300; full 1024 x 128
//   166, 193, 8192 x 8 570, 586.
// (PAIR does not exist for d = 192: WIDE in its place.)
inline AttnMode attn_mode(int s, int pairs, bool causal, int d) {
  const long cus = gemm_cu_count(), xcd_cus = cus / 8, blocks = (s + 127) / 128, wgs = blocks * pairs;
  const long xcd_pairs = (pairs + 7) / 8, xcd_wgs = xcd_pairs * blocks;
  if (2 * wgs <= cus && 2 * xcd_wgs <= (causal ? 2 : 1) * xcd_cus) return ATTN_SPLIT;
  if (d > 128) return ATTN_WIDE;
  if (wgs <= cus) return ATTN_PAIR;
  if (causal && (xcd_pairs <= 2 ? xcd_wgs <= 2 * xcd_cus : xcd_pairs == 3 && 2 * xcd_wgs <= 3 * xcd_cus)) return ATTN_PAIR;
  return ATTN_WIDE;
}

// Forward under a causal mask, PAIR and SPLIT: half a block of rows from either end of the sequence per workgroup, which all have the same
// work then, where every workgroup of the busiest XCD has a compute unit from the start and the longest one would be the launch's time
// (us, blocks / folded; s x pairs).  d = 96: 1024 x 32 23.6 / 21.3, with dropout 38.4 / 31.8; 1000 x 16 17.6 / 16.6, 512 x 64 16.2 / 15.5; d = 64:
// 1024 x 32 20.4 / 16.5; d = 128, dropout: 512 x 16 17.5 / 15.4.  Where workgroups queue, the short ones fill up behind the long ones by
// themselves, and half of a folded one's waves wait: d = 96 4096 x 16 91 / 101, 2048 x 24 53 / 57, 8192 x 8 161 / 184, d = 64 3072 x 4 31 / 42.
// Few tiles: d = 64 200 x 12 6.3 / 7.3, d = 96 320 x 6 11.4 / 12.0.  (Head size 192 has one group: its waves do not share a SIMD.)
inline bool attn_fwd_fold(AttnMode m, int s, int pairs) {
  const long rows = m == ATTN_SPLIT ? 64 : 128;
  return m != ATTN_WIDE && s >= 512 && (pairs + 7) / 8 * ((s + rows - 1) / rows) <= gemm_cu_count() / 8;
}

// dK / dV in a launch of its own (attn_bwd_mode), no mask, d = 64 or 96: 64-key workgroups (else 128-key ones) while twice as many fit
// the compute units overall and on the busiest XCD.  us, 128 / 64 keys: d = 96 1024 x 8 27 / 20, 64 1024 x 16 23 / 17; but 3072 x 4 74 / 91, 768 x
// 20 24 / 33.  (Under a causal mask and for larger heads launches that small are joint.)
inline bool attn_dkv_split(int s, int pairs) {
  const long cus = gemm_cu_count(), blocks = (s + 127) / 128;
  return 2 * blocks * pairs <= cus && 2 * blocks * ((pairs + 7) / 8) <= cus / 8;
}

// Backward: dQ and dK / dV as two launches (divided as above), or in one (attn_bwd_bf16_kernel), in 128-row workgroups or 64-row
// ones.  `parts` workgroups share a dK / dV block.  Of the busiest XCD's share of the 128-row workgroups of one kind, xcd_wgs:
//   64 rows while both kinds then find a compute unit each (and an eighth more); causal, d <= 96, from 6 blocks a sequence on, up
//   to two workgroups per unit: d = 96 1024 x 16 pairs 77 -> 70 us with the call's GEMMs, in 128 rows 72; 512 x 24 in 64 rows 53.3, 128 51.9.
//   Causal: 128 rows, however many, since the short blocks fill up behind the long ones: d = 96 1024 x 32 pairs 82 -> 71, 1024 x
//   64 153 -> 135, 2048 x 16 115 -> 92, 768 x 96 145 -> 140.  But not two pairs an XCD of more than one and a half blocks per
//   unit: 4096 x 12 246 -> 255.
//   No mask: only while the workgroups leave units idle, three quarters: d = 96 768 x 12 62 -> 56, but 2048 x 6 90 -> 98.
// (d = 192 has the joint launch in 128-row workgroups only: its blocks take a compute unit each, and two launches were 188 us against
// 118, 1024 x 16 causal, and 1616 against 1211, 2048 x 48 full; 64 rows equal up to 8 an XCD, above 316 / 262, 1024 x 48.)
enum AttnBwdMode { ATTN_BWD_TWO, ATTN_BWD_JOINT, ATTN_BWD_JOINT_SPLIT };
inline AttnBwdMode attn_bwd_mode(int s, int pairs, bool causal, int parts) {
  const long xcd_cus = gemm_cu_count() / 8, blocks = (s + 127) / 128, xcd_pairs = (pairs + 7) / 8, xcd_wgs = xcd_pairs * blocks;
  if (2 * (1 + parts) * xcd_wgs <= xcd_cus + xcd_cus / 8) return ATTN_BWD_JOINT_SPLIT;
  if (!causal) return 4 * (1 + parts) * xcd_wgs <= 3 * xcd_cus ? ATTN_BWD_JOINT : ATTN_BWD_TWO;
  if (parts == 1 && blocks >= 6 && 2 * xcd_wgs <= xcd_cus) return ATTN_BWD_JOINT_SPLIT;
  return xcd_pairs <= 2 && 2 * xcd_wgs > 3 * xcd_cus ? ATTN_BWD_TWO : ATTN_BWD_JOINT;
}

}  // namespace mlm
