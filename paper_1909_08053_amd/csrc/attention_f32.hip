// fp32 attention for dtype MLM_F32 on the fp32 matrix cores (v_mfma_f32_32x32x2_f32): streaming-softmax forward and a
// backward (dQ per query block, dK/dV per key block; one launch for both while their blocks find a compute unit each) that recomputes
// the probabilities from the saved log-sum-exp, so nothing of size s x s is ever stored and no atomics are needed (results are deterministic).
//
// A workgroup owns 32 rows (queries in forward and dQ, keys in dK/dV) of one (batch, head); its four waves take the
// 32-row tiles of the other sequence axis in turn (wave w: tiles w, w + 4, ...) and their partial results are merged
// through LDS in wave order: splitting the streamed axis over the waves shortens the serial chain, and a sequence of 128
// tokens, four tiles long, still keeps all four waves busy.  Bound by the matrix cores' fp32 rate and, below a few tiles
// per wave, by the chain of one tile.  Two sequences of 512 tokens, 16 heads of 64, causal: forward 26 us, dQ 36, dK/dV 47
// (739 / 721 + 7 for delta / 1134 with one thread per row on the vector ALUs); two of 128 tokens, 2 heads: 8 / 11 / 14 us
// (192 / 190 + 6 / 305).  A tile's values are requested in runs, the rows ahead of the scores and the columns ahead of the
// exponentials, in the registers that the rows leave; the next tile's rows ahead of the forward's second product.  Before, with the
// order left to the compiler -> now: 2048 tokens, 8 heads of 64: forward 83 -> 78, dQ 127 -> 115, dK/dV 140 -> 137; four sequences of
// 256, 8 heads of 80, no mask, dropout: 28.8 -> 15.3, 24.1 -> 23.4, 33 -> 26.4; 512, 8 heads of 128: 32 -> 29.7, both backward 81 -> 74; two
// of 128, 4 heads of 64: 9.0 -> 8.2, both 15.6 -> 14.6; two of 512, 8 heads of 96: 27.4 -> 25.0, dQ 35.9 -> 37.2 (the one loss).
//
// Scores are computed so that a lane's 16 accumulator values belong to ONE owned row, column l % 32 of the 32 x 32 tile,
// and to the streamed rows 8 (e / 4) + 4 (l / 32) + e % 4: row statistics are per-lane scalars plus one cross-half
// exchange, and value e is already the second product's operand for the pair of streamed rows {8 (e / 4) + e % 4, + 4} --
// the probabilities never leave their registers.  Operands come straight from the caches: 16-byte reads of a row where
// the head dimension is contracted (the order of a contraction is free, so the 8-deep chunk c feeds four MFMAs with
// elements 8 c + j / 8 c + 4 + j in the half-waves), 128-byte coalesced reads where the sequence is.
//
// Masking follows the integer predicate allowed(i,j) = (j < key_len[b]) && (!causal || j <= i);
// excluded keys contribute exactly zero.
// Dropout of the probabilities (a.drop.enabled): the forward kernel draws the keep decision of element
// ((batch, head, i), j) from the counter-based generator, saves it as one bit per key and uses p_ij keep / (1 - p) in
// C = P V; the row sum and the log-sum-exp stay those of the undropped scores.  The backward kernels read the bits.
#include "common.h"
#include "rng.h"

namespace mlm {

constexpr int AF_ROWS = 32;          // owned rows per workgroup and rows per streamed tile
constexpr int AF_WAVES = 4;

template <int D> struct AfShape {
  static constexpr int NC = D / 8;               // 8-deep chunks of the head dimension
  static constexpr int DT = (D + 31) / 32;       // 32-column tiles of it (the last one may hang over D)
};

// Workgroup id -> (block, head, batch).  With `pg` > 0 all blocks of a (batch, head) pair run on one XCD (ids go to the eight XCDs
// in turn), whose L2 then holds the rows they share; an XCD takes its pairs in groups of pg, and of a group first the first block
// of every pair, then the second, ..: the longest causal blocks of all pairs start first.  pg = 0: blocks of a pair in sequence,
// over all XCDs (af_pairs: when).  The backward call of 64 pairs of 512, d = 64, causal (its GEMMs included) 311 -> 234 us, 32
// pairs 204 -> 169, forward 147 -> 129; without a mask 2 % and nothing.
struct AfBlock { int xb, hd, bi; bool valid; };
__device__ __forceinline__ AfBlock af_block(int nb, int hl, int b, int pg) {
  const int id = blockIdx.x, pairs = hl * b;
  int xb, pair;                                        // (as few divisions as there are: 0.07 us each ahead of the first load)
  if (pg > 0) {
    const int npx = (pairs + 7) / 8;
    int r = id >> 3, first = 0, size = npx;
    if (pg < npx) {
      const int g = r / (pg * nb);
      r -= g * pg * nb;
      first = g * pg;
      size = min(pg, npx - first);
    }
    xb = r / size;
    pair = (first + r - xb * size) * 8 + (id & 7);
  } else {
    pair = id / nb;
    xb = id - pair * nb;
  }
  const int bi = pair / hl;
  return {xb, pair - bi * hl, bi, pair < pairs};
}
// Pairs of a group, and the grid.
static int af_pairs(const AttnArgs& a, int nb, unsigned* grid) {
  const int pairs = a.hl * a.b, npx = (pairs + 7) / 8, xcd_cus = gemm_cu_count() / 8;
  // whole pairs leave some XCDs with one more: not where that is a sixth of the work and more than a compute unit's
  if (npx * nb > xcd_cus && (8 * npx - pairs) * 6 > pairs) {
    *grid = (unsigned)(nb * pairs);
    return 0;
  }
  *grid = (unsigned)(8 * npx * nb);
  const int pg = (4 * xcd_cus + nb - 1) / nb;
  return pg < npx ? pg : npx;
}

// This lane's share (elements 8 c + 4 lh .. + 3 of every chunk c) of one row of the head.
template <int D>
__device__ __forceinline__ void af_load_row(const float* __restrict__ row, int lh, float (&f)[D / 2]) {
#pragma unroll
  for (int c = 0; c < D / 8; ++c) {
    const float4 v = *reinterpret_cast<const float4*>(row + 8 * c + 4 * lh);
    f[4 * c] = v.x; f[4 * c + 1] = v.y; f[4 * c + 2] = v.z; f[4 * c + 3] = v.w;
  }
}
// The streamed tile's rows from r0 on in the two forms that the products take, each as one run of requests ahead of what multiplies it
// (left to itself the compiler requests a value or two when the last ones have been used).  M: element (0, 0) of the matrix; rows
// beyond nrows - 1 repeat the last one (their weights are zero); r0 is wave-uniform, and a lane adds 32 bits to a scalar address.
template <int D>
__device__ __forceinline__ void af_tile_rows(const float* __restrict__ M, int ld, int r0, int nrows, int l32, int lh, float (&f)[D / 2]) {
  af_load_row<D>(M + (size_t)r0 * ld + (uint32_t)min(l32, nrows - 1 - r0) * (uint32_t)ld, lh, f);
}
template <int D>
__device__ __forceinline__ void af_tile_columns(const float* __restrict__ M, int ld, int r0, int nrows, int l32, int lh,
                                                float (&f)[16][AfShape<D>::DT]) {
  const char* tile = reinterpret_cast<const char*>(M + (size_t)r0 * ld);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const uint32_t r = 4u * (uint32_t)ld * (uint32_t)min(8 * (e >> 2) + 4 * lh + (e & 3), nrows - 1 - r0);
#pragma unroll
    for (int dt = 0; dt < AfShape<D>::DT; ++dt)          // (columns past the head's: its last one again, never stored)
      f[e][dt] = *reinterpret_cast<const float*>(tile + (r + 4u * (uint32_t)min(dt * 32 + l32, D - 1)));
  }
}
// acc[streamed row][owned row] = sum over the head dimension of streamed[row] . owned
template <int D>
__device__ __forceinline__ floatx16 af_scores(const float (&row)[D / 2], const float (&own)[D / 2]) {
  floatx16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
  for (int c = 0; c < D / 2; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(row[c], own[c], acc, 0, 0, 0);
  return acc;
}
// out[dt][head column][owned row] += sum over the tile's streamed rows of M[row][column] w[row][owned row]
template <int D>
__device__ __forceinline__ void af_accumulate(const float (&M)[16][AfShape<D>::DT], const floatx16& w, floatx16 (&out)[AfShape<D>::DT]) {
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int dt = 0; dt < AfShape<D>::DT; ++dt) out[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(M[e][dt], w[e], out[dt], 0, 0, 0);
}
// The waves' accumulators parked in LDS ([wave][value][lane]: conflict-free)
template <int NV> __device__ __forceinline__ float* af_park(float* lds, int wave, int lane) { return lds + (size_t)wave * NV * 64 + lane; }
// af_accumulate for a tile in which, if `edge`, some pairs are excluded (off(e): this lane's pair e is).  An excluded pair's weight is
// zero, but zero times Inf or NaN is NaN and the matrix cores multiply every pair: a tile that holds such a value is added pair by
// pair, the allowed ones only.  (Looking at the values costs nothing new now that the tile is in registers; looking at the sums
// behind the products, with a copy of what they were before, took 32 registers and as many moves at a head of 64.)
template <int D, typename Off>
__device__ __forceinline__ void af_accumulate_masked(const float* __restrict__ M, int ld, int r0, int lane,
                                                     const float (&columns)[16][AfShape<D>::DT], const floatx16& w, bool edge, Off off,
                                                     float* park, floatx16 (&out)[AfShape<D>::DT]) {
  bool finite = true;
  if (edge) {
    float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < AfShape<D>::DT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) x[e & 3] = fmaf(0.f, columns[e][dt], x[e & 3]);       // 0, or NaN
    const float xs = (x[0] + x[1]) + (x[2] + x[3]);
    finite = __builtin_amdgcn_ballot_w64(xs != xs) == 0;
  }
  if (__builtin_expect(finite, 1)) {
    af_accumulate<D>(columns, w, out);
    return;
  }
  // (the sums wait in this lane's own part of LDS, which nothing else uses before the end: in registers, this loop is what decides how
  // many the kernel takes)
#pragma unroll
  for (int dt = 0; dt < AfShape<D>::DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) park[(dt * 16 + e) * 64] = out[dt][e];
  uint32_t allow = 0;
#pragma unroll
  for (int e = 0; e < 16; ++e) allow |= off(e) ? 0u : 1u << e;
  const int l32 = lane & 31, lh = lane >> 5;
#pragma unroll 1
  for (int r = 0; r < AF_ROWS; ++r) {
    const int e = 4 * (r >> 3) + (r & 3), src = l32 + 32 * ((r >> 2) & 1);    // where the weight of streamed row r is
    float we = w[0];
#pragma unroll
    for (int q = 1; q < 16; ++q) we = q == e ? w[q] : we;
    we = __shfl(we, src, 64);
    const bool on = (__shfl(allow, src, 64) >> e) & 1u;
    if (!on) continue;                                 // (an allowed row lies inside the sequence)
    const float* p = M + (size_t)(r0 + r) * ld + 4 * lh;
#pragma unroll 1
    for (int g = 0; g < D / 8; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) park[(4 * g + i) * 64] = fmaf(p[8 * g + i], we, park[(4 * g + i) * 64]);
  }
#pragma unroll
  for (int dt = 0; dt < AfShape<D>::DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) out[dt][e] = park[(dt * 16 + e) * 64];
}

template <int D>
__global__ __launch_bounds__(64 * AF_WAVES, D <= 64 ? 2 : 1) void attn_fwd_f32_kernel(AttnArgs a, int pg) {
  constexpr int DT = AfShape<D>::DT, NV = DT * 16 + 2;
  extern __shared__ __attribute__((aligned(16))) float lds_af[];
  const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (a.s + AF_ROWS - 1) / AF_ROWS;
  const AfBlock blk = af_block(nb, a.hl, a.b, pg);
  if (!blk.valid) return;
  const int qb = nb - 1 - blk.xb;                        // longest (causal) blocks first
  const int hd = blk.hd, bi = blk.bi;
  const int ld = 3 * a.hl * D;
  const float* base = (const float*)a.qkv + (size_t)bi * a.s * ld;
  const int klen = attn_key_len(a.key_len, bi, a.s);
  const int q0 = qb * AF_ROWS, qi = q0 + l32;
  const float scale = 1.0f / sqrtf((float)D);
  float q[D / 2];
  af_load_row<D>(base + (size_t)min(qi, a.s - 1) * ld + hd * D, lh, q);
  floatx16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
  float m = -INFINITY, l = 0.f;                          // l: this half-wave's keys only
  int kv_end = klen;
  if (a.causal) kv_end = min(kv_end, min(a.s, q0 + AF_ROWS));
  const size_t prow = ((size_t)bi * a.hl + hd) * a.s + min(qi, a.s - 1);   // row of the [b, hl, s, s] probability tensor
  const float* K = base + (a.hl + hd) * D;
  const float* V = base + (2 * a.hl + hd) * D;
  float* park = af_park<NV>(lds_af, wave, lane);
  float kr[D / 2], vc[16][DT];
  if (wave * AF_ROWS < kv_end) af_tile_rows<D>(K, ld, wave * AF_ROWS, a.s, l32, lh, kr);
  for (int k0 = wave * AF_ROWS; k0 < kv_end; k0 += AF_WAVES * AF_ROWS) {
    floatx16 s = af_scores<D>(kr, q);
    af_tile_columns<D>(V, ld, k0, a.s, l32, lh, vc);      // (in the registers of K's rows)
    __builtin_amdgcn_sched_barrier(0);
    float mt = -INFINITY;
    auto off = [&](int e) {
      const int key = k0 + 8 * (e >> 2) + 4 * lh + (e & 3);
      return key >= klen || (a.causal && key > qi);
    };
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = off(e) ? -INFINITY : s[e] * scale;
      mt = fmaxf(mt, s[e]);
    }
    // key k0 is allowed for every query of the block (k0 < kv_end, and a causal tile never starts right of the block's
    // first query), so the maximum is finite
    const float mn = fmaxf(m, fmaxf(mt, __shfl_xor(mt, 32, 64)));
    const float corr = expf(m - mn);
    float ls = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s[e] = expf(s[e] - mn);
      ls += s[e];
    }
    l = l * corr + ls;
    m = mn;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dt][e] *= corr;
    if (a.drop.enabled) {
      uint32_t word = 0;                                 // this half-wave's 16 of the tile's 32 keep bits
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t k4 = drop_keep4(a.drop, (prow * a.s + k0 + 8 * g + 4 * lh) >> 2);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[4 * g + e] = ((k4 >> e) & 1u) ? s[4 * g + e] : 0.f;
        word |= k4 << (8 * g + 4 * lh);
      }
      word |= __shfl_xor(word, 32, 64);
      if (lh == 0 && qi < a.s) a.keep_bits[prow * a.keep_pitch + (k0 >> 5)] = word;
    }
    const bool edge = k0 + AF_ROWS > klen || (a.causal && k0 + AF_ROWS - 1 > q0);      // wave-uniform
    if (k0 + AF_WAVES * AF_ROWS < kv_end) af_tile_rows<D>(K, ld, k0 + AF_WAVES * AF_ROWS, a.s, l32, lh, kr);
    __builtin_amdgcn_sched_barrier(0);
    af_accumulate_masked<D>(V, ld, k0, lane, vc, s, edge, off, park, o);
  }
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) park[(dt * 16 + e) * 64] = o[dt][e];
  park[DT * 16 * 64] = m;
  park[(DT * 16 + 1) * 64] = l;
  __syncthreads();
  // every wave forms the merged statistics of all rows and finishes DT of the 4 DT groups of four head columns
  float M = -INFINITY, L = 0.f, c[AF_WAVES];
#pragma unroll
  for (int w = 0; w < AF_WAVES; ++w) M = fmaxf(M, af_park<NV>(lds_af, w, lane)[DT * 16 * 64]);   // wave 0 has tile 0: finite
#pragma unroll
  for (int w = 0; w < AF_WAVES; ++w) {
    c[w] = expf(af_park<NV>(lds_af, w, lane)[DT * 16 * 64] - M);
    L += c[w] * (af_park<NV>(lds_af, w, lane)[(DT * 16 + 1) * 64] + af_park<NV>(lds_af, w, lane ^ 32)[(DT * 16 + 1) * 64]);
  }
  if (qi >= a.s) return;
  const float inv = a.drop.scale / L;
  float* crow = (float*)a.ctx + ((size_t)bi * a.s + qi) * (a.hl * D) + hd * D;
#pragma unroll
  for (int i = 0; i < DT; ++i) {
    const int grp = wave * DT + i, dt = grp >> 2, g = grp & 3;
    const int col = dt * 32 + 8 * g + 4 * lh;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < AF_WAVES; ++w) {
      const float* p = af_park<NV>(lds_af, w, lane) + (dt * 16 + 4 * g) * 64;
      r.x += p[0] * c[w]; r.y += p[64] * c[w]; r.z += p[128] * c[w]; r.w += p[192] * c[w];
    }
    if (col < D) *reinterpret_cast<float4*>(crow + col) = make_float4(r.x * inv, r.y * inv, r.z * inv, r.w * inv);
  }
  if (wave == 0 && lh == 0) a.lse[((size_t)bi * a.hl + hd) * a.s + qi] = M + logf(L);
}

// dQ_i = scale * sum_j dS_ij K_j,  dS_ij = P_ij (dO_i . V_j - delta_i),  P_ij = exp(scale q_i.k_j - lse_i);
// delta_i = dO_i . O_i is formed here from rows the lanes hold and left in the workspace for the dK/dV kernel.
// (JOINT: part of attn_bwd_dkv_f32_kernel<D, true>, whose dK/dV blocks form delta themselves)
template <int D, bool JOINT>
__device__ __forceinline__ void attn_bwd_dq_f32_block(const AttnArgs a, const AfBlock blk) {
  constexpr int DT = AfShape<D>::DT, NV = DT * 16;
  extern __shared__ __attribute__((aligned(16))) float lds_af[];
  const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qb = (a.s + AF_ROWS - 1) / AF_ROWS - 1 - blk.xb;
  const int hd = blk.hd, bi = blk.bi;
  const int ld = 3 * a.hl * D, ldo = a.hl * D;
  const float* base = (const float*)a.qkv + (size_t)bi * a.s * ld;
  const int klen = attn_key_len(a.key_len, bi, a.s);
  const int q0 = qb * AF_ROWS, qi = q0 + l32, qc = min(qi, a.s - 1);
  const float scale = 1.0f / sqrtf((float)D);
  float q[D / 2], dov[D / 2];
  af_load_row<D>(base + (size_t)qc * ld + hd * D, lh, q);
  af_load_row<D>((const float*)a.dctx + ((size_t)bi * a.s + qc) * ldo + hd * D, lh, dov);
  float dl = 0.f;
  {
    float ov[D / 2];
    af_load_row<D>((const float*)a.ctx + ((size_t)bi * a.s + qc) * ldo + hd * D, lh, ov);
#pragma unroll
    for (int c = 0; c < D / 2; ++c) dl = fmaf(ov[c], dov[c], dl);
    dl += __shfl_xor(dl, 32, 64);
  }
  const size_t row = ((size_t)bi * a.hl + hd) * a.s + qc;
  const float lse = a.lse[row];
  if (!JOINT && wave == 0 && lh == 0 && qi < a.s) a.delta[row] = dl;
  floatx16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[dt][e] = 0.f;
  int kv_end = klen;
  if (a.causal) kv_end = min(kv_end, min(a.s, q0 + AF_ROWS));
  const float* K = base + (a.hl + hd) * D;
  const float* V = base + (2 * a.hl + hd) * D;
  float* park = af_park<NV>(lds_af, wave, lane);
  for (int k0 = wave * AF_ROWS; k0 < kv_end; k0 += AF_WAVES * AF_ROWS) {
    float kr[D / 2], vr[D / 2], kc[16][DT];
    af_tile_rows<D>(K, ld, k0, a.s, l32, lh, kr);
    af_tile_rows<D>(V, ld, k0, a.s, l32, lh, vr);
    const uint32_t bits = a.drop.enabled ? a.keep_bits[row * a.keep_pitch + (k0 >> 5)] >> (4 * lh) : 0xFFFFFFFFu;
    constexpr bool STAGED = D <= 80;
    if (STAGED) __builtin_amdgcn_sched_barrier(0);
    floatx16 s = af_scores<D>(kr, q);
    if (STAGED) {
      af_tile_columns<D>(K, ld, k0, a.s, l32, lh, kc);    // (in the registers of the rows)
      __builtin_amdgcn_sched_barrier(0);
    }
    const floatx16 dp = af_scores<D>(vr, dov);
    auto off = [&](int e) {
      const int key = k0 + 8 * (e >> 2) + 4 * lh + (e & 3);
      return key >= klen || (a.causal && key > qi);
    };
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = expf(s[e] * scale - lse);
      // gradient w.r.t. the undropped probability
      const float g = ((bits >> (8 * (e >> 2) + (e & 3))) & 1u) ? dp[e] * a.drop.scale : 0.f;
      const float ds = p * (g - dl);
      s[e] = off(e) ? 0.f : ds;
    }
    const bool edge = k0 + AF_ROWS > klen || (a.causal && k0 + AF_ROWS - 1 > q0);      // wave-uniform
    if (!STAGED) af_tile_columns<D>(K, ld, k0, a.s, l32, lh, kc);
    af_accumulate_masked<D>(K, ld, k0, lane, kc, s, edge, off, park, dq);
  }
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) park[(dt * 16 + e) * 64] = dq[dt][e];
  __syncthreads();
  if (qi >= a.s) return;
  float* orow = (float*)a.dqkv + ((size_t)bi * a.s + qi) * ld + hd * D;
#pragma unroll
  for (int i = 0; i < DT; ++i) {
    const int grp = wave * DT + i, dt = grp >> 2, g = grp & 3;
    const int col = dt * 32 + 8 * g + 4 * lh;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < AF_WAVES; ++w) {
      const float* p = af_park<NV>(lds_af, w, lane) + (dt * 16 + 4 * g) * 64;
      r.x += p[0]; r.y += p[64]; r.z += p[128]; r.w += p[192];
    }
    if (col < D) *reinterpret_cast<float4*>(orow + col) = make_float4(r.x * scale, r.y * scale, r.z * scale, r.w * scale);
  }
}

// dV_j = sum_i P_ij dO_i,  dK_j = scale * sum_i dS_ij Q_i
// JOINT: dQ's blocks follow in the same launch, for calls whose blocks all find a compute unit at once (else dQ runs two workgroups
// per unit in a launch of its own, and here only one).  Delta of a tile's queries is then formed here, from the rows of dO that
// the scores read anyway and those of O.  Two of 128 tokens, 2 heads of 64: 23 us
// in two launches, 14.5 in one (16.9 with O's rows requested behind the scores).
template <int D, bool JOINT>
__global__ __launch_bounds__(64 * AF_WAVES, 1) void attn_bwd_dkv_f32_kernel(AttnArgs a, int pg) {
  constexpr int DT = AfShape<D>::DT, NV = 2 * DT * 16;
  extern __shared__ __attribute__((aligned(16))) float lds_af[];
  const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  AfBlock blk;
  if (JOINT) {
    const int nb = (a.s + AF_ROWS - 1) / AF_ROWS, n = nb * a.hl * a.b, k = blockIdx.x;
    const int id = k < n ? k : k - n, pair = id / nb, pb = pair / a.hl;
    blk = {id - pair * nb, pair - pb * a.hl, pb, true};
    if (k >= n) {
      attn_bwd_dq_f32_block<D, true>(a, blk);
      return;
    }
  } else {
    blk = af_block((a.s + AF_ROWS - 1) / AF_ROWS, a.hl, a.b, pg);
    if (!blk.valid) return;
  }
  const int hd = blk.hd, bi = blk.bi;
  const int ld = 3 * a.hl * D, ldo = a.hl * D;
  const float* base = (const float*)a.qkv + (size_t)bi * a.s * ld;
  const float* dO = (const float*)a.dctx + (size_t)bi * a.s * ldo + hd * D;
  const float* Q = base + hd * D;
  const int klen = attn_key_len(a.key_len, bi, a.s);
  const int kb0 = blk.xb * AF_ROWS, kj = kb0 + l32, kc = min(kj, a.s - 1);
  const float scale = 1.0f / sqrtf((float)D);
  float kf[D / 2], vf[D / 2];
  af_load_row<D>(base + (size_t)kc * ld + (a.hl + hd) * D, lh, kf);
  af_load_row<D>(base + (size_t)kc * ld + (2 * a.hl + hd) * D, lh, vf);
  floatx16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dk[dt][e] = 0.f; dv[dt][e] = 0.f; }
  const size_t row0 = ((size_t)bi * a.hl + hd) * a.s;
  // key blocks of padding only get zeros; a causal block starts at its own first query
  const int q_begin = kb0 >= klen ? a.s : (a.causal ? kb0 : 0);
  float* park = af_park<NV>(lds_af, wave, lane);
  for (int q0 = q_begin + wave * AF_ROWS; q0 < a.s; q0 += AF_WAVES * AF_ROWS) {
    const int qr = min(q0 + l32, a.s - 1);
    // the tile's per-query values are requested ahead of the scores, and the mask selects the finished probability: with
    // the loads behind the mask they were taken one by one inside branches (fp32 layer step 1342 -> 1314 us)
    float lse[16], del[16];
    uint32_t bits[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int ic = min(q0 + 8 * (e >> 2) + 4 * lh + (e & 3), a.s - 1);
      lse[e] = a.lse[row0 + ic];
      if (!JOINT) del[e] = a.delta[row0 + ic];
    }
    // O's row of query q0 + l32, requested ahead of the scores too where there are registers for it
    constexpr bool EARLY = JOINT && D <= 80;
    const float* orow = (const float*)a.ctx + ((size_t)bi * a.s + qr) * ldo + hd * D + 4 * lh;
    float4 ov[EARLY ? D / 8 : 1];
    if (EARLY) {
#pragma unroll
      for (int c = 0; c < D / 8; ++c) ov[c] = *reinterpret_cast<const float4*>(orow + 8 * c);
    }
    if (a.drop.enabled) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        bits[e] = a.keep_bits[(row0 + min(q0 + 8 * (e >> 2) + 4 * lh + (e & 3), a.s - 1)) * a.keep_pitch + (kb0 >> 5)];
    }
    constexpr bool STAGED = D <= 96;                      // above, the rows do not fit beside four accumulators: taken as they are needed
    auto requested = [] {
      if (STAGED) __builtin_amdgcn_sched_barrier(0);
    };
    float qf[D / 2], gf[D / 2], qc[16][DT], gc[16][DT];
    af_tile_rows<D>(Q, ld, q0, a.s, l32, lh, qf);
    af_tile_rows<D>(dO, ldo, q0, a.s, l32, lh, gf);
    requested();
    floatx16 s = af_scores<D>(qf, kf);                    // [query][key]
    if (STAGED) af_tile_columns<D>(dO, ldo, q0, a.s, l32, lh, gc);       // (in the registers of Q's rows)
    requested();
    floatx16 dp = af_scores<D>(gf, vf);
    if (JOINT) {
      float dl = 0.f;                                     // of query q0 + l32, in the order of the dQ kernel
#pragma unroll
      for (int c = 0; c < D / 8; ++c) {
        const float4 o = EARLY ? ov[EARLY ? c : 0] : *reinterpret_cast<const float4*>(orow + 8 * c);
        dl = fmaf(o.x, gf[4 * c], dl); dl = fmaf(o.y, gf[4 * c + 1], dl); dl = fmaf(o.z, gf[4 * c + 2], dl); dl = fmaf(o.w, gf[4 * c + 3], dl);
      }
      dl += __shfl_xor(dl, 32, 64);
#pragma unroll
      for (int e = 0; e < 16; ++e) del[e] = __shfl(dl, 8 * (e >> 2) + 4 * lh + (e & 3), 64);
    }
    if (STAGED) af_tile_columns<D>(Q, ld, q0, a.s, l32, lh, qc);
    requested();
    auto off = [&](int e) {
      const int i = q0 + 8 * (e >> 2) + 4 * lh + (e & 3);
      return kj >= klen || i >= a.s || (a.causal && kj > i);
    };
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = expf(s[e] * scale - lse[e]);
      float keep = 1.0f;
      if (a.drop.enabled) keep = ((bits[e] >> l32) & 1u) ? a.drop.scale : 0.f;
      const float pd = p * keep, ds = p * (dp[e] * keep - del[e]);
      s[e] = off(e) ? 0.f : pd;
      dp[e] = off(e) ? 0.f : ds;
    }
    const bool edge = kb0 + AF_ROWS > klen || q0 + AF_ROWS > a.s || (a.causal && kb0 + AF_ROWS - 1 > q0);   // wave-uniform
    if (!STAGED) af_tile_columns<D>(dO, ldo, q0, a.s, l32, lh, gc);
    af_accumulate_masked<D>(dO, ldo, q0, lane, gc, s, edge, off, park, dv);
    if (!STAGED) af_tile_columns<D>(Q, ld, q0, a.s, l32, lh, qc);
    af_accumulate_masked<D>(Q, ld, q0, lane, qc, dp, edge, off, park, dk);
  }
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      park[(dt * 16 + e) * 64] = dk[dt][e] * scale;
      park[((DT + dt) * 16 + e) * 64] = dv[dt][e];
    }
  __syncthreads();
  if (kj >= a.s) return;
  float* krow = (float*)a.dqkv + ((size_t)bi * a.s + kj) * ld + (a.hl + hd) * D;
#pragma unroll
  for (int i = 0; i < 2 * DT; ++i) {
    const int grp = wave * 2 * DT + i, t = grp >> 2, g = grp & 3;     // t < DT: dK tile t, else dV tile t - DT
    const int col = (t % DT) * 32 + 8 * g + 4 * lh;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < AF_WAVES; ++w) {
      const float* p = af_park<NV>(lds_af, w, lane) + (t * 16 + 4 * g) * 64;
      r.x += p[0]; r.y += p[64]; r.z += p[128]; r.w += p[192];
    }
    if (col < D) *reinterpret_cast<float4*>(krow + (t < DT ? 0 : a.hl * D) + col) = r;
  }
}

template <int D>
__global__ __launch_bounds__(64 * AF_WAVES, D <= 64 ? 2 : 1) void attn_bwd_dq_f32_kernel(AttnArgs a, int pg) {
  const AfBlock blk = af_block((a.s + AF_ROWS - 1) / AF_ROWS, a.hl, a.b, pg);
  if (blk.valid) attn_bwd_dq_f32_block<D, false>(a, blk);
}
bool attn_f32_supported(int d) { return d > 0 && d % 16 == 0 && d <= 128; }

#define MLM_AF_SWITCH(MACRO)                                                                         \
  switch (a.d) {                                                                                     \
    case 16: MACRO(16) break; case 32: MACRO(32) break; case 48: MACRO(48) break;                    \
    case 64: MACRO(64) break; case 80: MACRO(80) break; case 96: MACRO(96) break;                    \
    case 112: MACRO(112) break; case 128: MACRO(128) break;                                          \
    default: return hipErrorInvalidValue;                                                            \
  }

// values per lane that a wave parks -> bytes of LDS of the workgroup
static constexpr size_t af_lds(int values) { return (size_t)AF_WAVES * values * 64 * sizeof(float); }

hipError_t launch_attn_fwd_f32(const AttnArgs& a, hipStream_t st) {
  unsigned ngrid;
  const int pg = af_pairs(a, (a.s + AF_ROWS - 1) / AF_ROWS, &ngrid);
  const dim3 grid(ngrid), block(64 * AF_WAVES);
#define MLM_AF_FWD(DD)                                                                               \
  {                                                                                                  \
    constexpr size_t lds = af_lds(AfShape<DD>::DT * 16 + 2);                                         \
    static LdsAttrOnce attr;                                                                         \
    if (hipError_t e = attr.ensure((const void*)attn_fwd_f32_kernel<DD>, (int)lds); e != hipSuccess) return e; \
    hipLaunchKernelGGL((attn_fwd_f32_kernel<DD>), grid, block, lds, st, a, pg);                      \
  }
  MLM_AF_SWITCH(MLM_AF_FWD)
#undef MLM_AF_FWD
  return hipGetLastError();
}

hipError_t launch_attn_bwd_f32(const AttnArgs& a, hipStream_t st) {
  const long joint = 2l * ((a.s + AF_ROWS - 1) / AF_ROWS) * a.hl * a.b;
  if (joint <= gemm_cu_count()) {
#define MLM_AF_JOINT(DD)                                                                             \
  {                                                                                                  \
    constexpr size_t lds = af_lds(2 * AfShape<DD>::DT * 16);                                         \
    static LdsAttrOnce attr;                                                                         \
    if (hipError_t e = attr.ensure((const void*)(attn_bwd_dkv_f32_kernel<DD, true>), (int)lds); e != hipSuccess) return e; \
    hipLaunchKernelGGL((attn_bwd_dkv_f32_kernel<DD, true>), dim3((unsigned)joint), dim3(64 * AF_WAVES), lds, st, a, 0); \
  }
    MLM_AF_SWITCH(MLM_AF_JOINT)
#undef MLM_AF_JOINT
    return hipGetLastError();
  }
  unsigned ngrid;
  const int pg = af_pairs(a, (a.s + AF_ROWS - 1) / AF_ROWS, &ngrid);
  const dim3 grid(ngrid), block(64 * AF_WAVES);
#define MLM_AF_BWD(DD)                                                                               \
  {                                                                                                  \
    constexpr size_t lds1 = af_lds(AfShape<DD>::DT * 16), lds2 = af_lds(2 * AfShape<DD>::DT * 16);   \
    static_assert(lds2 <= 160 * 1024, "LDS budget");                                                 \
    static LdsAttrOnce attr1, attr2;                                                                 \
    if (hipError_t e = attr1.ensure((const void*)attn_bwd_dq_f32_kernel<DD>, (int)lds1); e != hipSuccess) return e; \
    if (hipError_t e = attr2.ensure((const void*)(attn_bwd_dkv_f32_kernel<DD, false>), (int)lds2); e != hipSuccess) return e; \
    hipLaunchKernelGGL((attn_bwd_dq_f32_kernel<DD>), grid, block, lds1, st, a, pg);                  \
    hipLaunchKernelGGL((attn_bwd_dkv_f32_kernel<DD, false>), grid, block, lds2, st, a, pg);                 \
  }
  MLM_AF_SWITCH(MLM_AF_BWD)
#undef MLM_AF_BWD
  return hipGetLastError();
}

}  // namespace mlm
