// bf16 GEMM for outputs of few tiles (gfx950): C[m,n] = sum_k A(m,k) B(k,n) in tiles of 64 x 64, 32 x 64 or 32 x 32, whose
// k is dealt to the eight waves of a workgroup in 32-deep slices.
//   * Such a product is bound by latency, not by bytes or flops: the 128 x 128 tile leaves most compute units idle there, and
//     its ring of slices, its barriers and its epilogue are a chain of 5 us before anything is stored.  Here every wave loads
//     the fragments of its own slices straight into registers (no LDS, no barrier in the loop, two slices in flight a wave and
//     sixteen a compute unit), and the eight partial sums of an output meet once, in LDS.
//   * A k-contiguous operand is a fragment as it lies in memory: lane l takes the 16 bytes k = 8 (l / 16) .. + 7 of row l % 16.
//     An operand contiguous along m / n is transposed in registers: lane l loads four (two) neighbouring columns of the eight
//     k-rows 8 (l / 16) .. + 7 -- 16 lanes a full 128-byte line (half of one) -- and one byte permute per register pairs two
//     k-rows; its 16 x 16 tiles then hold columns 4 c + f (2 c + f), f the tile's number, and the store undoes that order for nothing.
//   * Sums: eight chains over k, added in pairs; no result is further from the exact one than in the large tiles' single chain.
#pragma once
#include "gemm_bf16_v2.h"

namespace mlm {

constexpr int kSplitWaves = 8;

// The fragments of one operand's ROWS rows (64 or 32) in one 32-deep slice.
template <bool KC, int ROWS> struct SplitOperand;

template <int ROWS> struct SplitOperand<true, ROWS> {
  static constexpr int NF = ROWS / 16;
  struct Raw { bf16x8 v[NF]; };
  const char* base;                    // the tile's first row (uniform)
  uint32_t off[NF];                    // bytes from there to this lane's unit of slice 0; below 4 GiB: 63 rows of at most 2^24 k
  uint32_t unit;                       // 16 (lane / 16)
  __device__ __forceinline__ void init(const void* P, int ld, int row0, int nrows, int lane) {
    base = (const char*)P + (size_t)row0 * ld * 2;
    unit = (lane >> 4) * 16;
#pragma unroll
    for (int f = 0; f < NF; ++f) off[f] = (uint32_t)(min(row0 + 16 * f + (lane & 15), nrows - 1) - row0) * (uint32_t)ld * 2 + unit;
  }
  __device__ __forceinline__ void load(Raw& r, int s) const {
    const char* p = base + (size_t)s * 64;
#pragma unroll
    for (int f = 0; f < NF; ++f) r.v[f] = *reinterpret_cast<const bf16x8*>(p + off[f]);
  }
  // slice s holds kleft < 32 of k, a multiple of 8: units past it are zeros
  __device__ __forceinline__ void load_end(Raw& r, int s, int kleft) const {
    const char* p = base + (size_t)s * 64;
    const bool in = (int)unit < kleft * 2;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(p + (in ? off[f] : off[f] - unit));
      const bf16x8 zero = {};
      r.v[f] = in ? v : zero;
    }
  }
  __device__ __forceinline__ void frags(const Raw& r, bf16x8 (&f)[NF]) const {
#pragma unroll
    for (int i = 0; i < NF; ++i) f[i] = r.v[i];
  }
};

template <int ROWS> struct SplitOperand<false, ROWS> {
  static constexpr int NF = ROWS / 16, NW = NF / 2;      // words (of two columns) a lane loads of a k-row
  struct Raw { uint32_t w[8][NW]; };
  const char* base;                    // the tile's first column (uniform)
  uint32_t col, off;                   // bytes to this lane's columns; and to its first k-row of slice 0
  int ld;
  __device__ __forceinline__ void init(const void* P, int ld_, int row0, int nrows, int lane) {
    ld = ld_;
    base = (const char*)P + (size_t)row0 * 2;
    col = (uint32_t)(min(row0 + NF * (lane & 15), nrows - NF) - row0) * 2;      // (nrows, a multiple of 8, is past row0)
    off = (uint32_t)(lane >> 4) * 8u * (uint32_t)ld * 2 + col;
  }
  static __device__ __forceinline__ void get(uint32_t (&w)[NW], const char* p) {
    if constexpr (NW == 2) {
      const uint2 v = *reinterpret_cast<const uint2*>(p);
      w[0] = v.x; w[1] = v.y;
    } else {
      w[0] = *reinterpret_cast<const uint32_t*>(p);
    }
  }
  __device__ __forceinline__ void load(Raw& r, int s) const {
    const char* p = base + (size_t)s * 64 * ld;
#pragma unroll
    for (int j = 0; j < 8; ++j) get(r.w[j], p + (size_t)j * 2 * ld + off);
  }
  __device__ __forceinline__ void load_end(Raw& r, int s, int kleft) const {
    const char* p = base + (size_t)s * 64 * ld;
    const int k0 = (threadIdx.x >> 4 & 3) * 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      get(r.w[j], p + (size_t)((uint32_t)min(k0 + j, kleft - 1) * (uint32_t)ld * 2 + col));
#pragma unroll
      for (int q = 0; q < NW; ++q) r.w[j][q] = k0 + j < kleft ? r.w[j][q] : 0u;
    }
  }
  __device__ __forceinline__ void frags(const Raw& r, bf16x8 (&f)[NF]) const {
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      uint4 v;
      const uint32_t sel = i & 1 ? 0x07060302u : 0x05040100u;         // the high or the low halves of two k-rows
      v.x = __builtin_amdgcn_perm(r.w[1][i >> 1], r.w[0][i >> 1], sel);
      v.y = __builtin_amdgcn_perm(r.w[3][i >> 1], r.w[2][i >> 1], sel);
      v.z = __builtin_amdgcn_perm(r.w[5][i >> 1], r.w[4][i >> 1], sel);
      v.w = __builtin_amdgcn_perm(r.w[7][i >> 1], r.w[6][i >> 1], sel);
      f[i] = __builtin_bit_cast(bf16x8, v);
    }
  }
};

// Max and sum over groups of N = 8 or 16 neighbouring lanes, handed to each of them.
template <int N> __device__ __forceinline__ float split_max(float v) {
  v = fmaxf(v, dpp_move<0xB1, 0xf, 0xf>(v, v));                    // quad_perm 1 0 3 2
  v = fmaxf(v, dpp_move<0x4E, 0xf, 0xf>(v, v));                    // quad_perm 2 3 0 1
  v = fmaxf(v, dpp_move<0x141, 0xf, 0xf>(v, v));                   // row_half_mirror
  if (N == 16) v = fmaxf(v, dpp_move<0x140, 0xf, 0xf>(v, v));      // row_mirror
  return v;
}
template <int N> __device__ __forceinline__ float split_sum(float v) {
  v += dpp_move<0xB1, 0xf, 0xf>(v, v);
  v += dpp_move<0x4E, 0xf, 0xf>(v, v);
  v += dpp_move<0x141, 0xf, 0xf>(v, v);
  if (N == 16) v += dpp_move<0x140, 0xf, 0xf>(v, v);
  return v;
}

template <int TM, int TN> constexpr size_t split_lds_bytes() { return (size_t)kSplitWaves * TM * TN * 4; }

// One tile.  Enters and leaves without a barrier of its own outside; uses split_lds_bytes<TM, TN>() of LDS.
template <bool A_KC, bool B_KC, int EPI, int TM, int TN>
__device__ __forceinline__ void gemm_split_tile(const GemmArgs& a, int tile_m, int tile_n, unsigned char* lds_raw) {
  constexpr int KW = kSplitWaves, NA = TM / 16, NB = TN / 16;
  constexpr int VEC = TM * TN / (64 * KW), TPR = TN / VEC;      // a thread finishes VEC columns of one row
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int m0 = tile_m * TM, n0 = tile_n * TN;
  SplitOperand<A_KC, TM> A;
  SplitOperand<B_KC, TN> B;
  A.init(a.A, a.lda, m0, a.M, lane);
  B.init(a.B, a.ldb, n0, a.N, lane);
  typename SplitOperand<A_KC, TM>::Raw ra[2];
  typename SplitOperand<B_KC, TN>::Raw rb[2];
  floatx4 acc[NB][NA];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // what the epilogue reads for its outputs, ahead of everything
  struct alignas(2 * VEC) OutVec { bf16 v[VEC]; };
  OutVec bias, pre;
  int target = -1;
  const int orow = tid / TPR, ocol = tid % TPR * VEC, gm = m0 + orow, gn = n0 + ocol;
  const int gmc = min(gm, a.M - 1), gnc = min(gn, a.N - VEC);
  if ((EPI == EPI_STORE || EPI == EPI_BIAS_GELU) && a.bias != nullptr) bias = *reinterpret_cast<const OutVec*>((const bf16*)a.bias + gnc);
  if (EPI == EPI_DGELU) pre = *reinterpret_cast<const OutVec*>((const bf16*)a.aux + (size_t)gmc * a.ldaux + gnc);
  if (EPI == EPI_CE) target = a.targets[gmc] - a.v0 - gn;

  // slices wave, wave + 8, ...; the last one of k may hold less than 32.  Both forms of a load are as many requests, so that what
  // is outstanding at a product is known whichever ran.
  const int kleft = a.K & 31, slices = (a.K + 31) >> 5, last = kleft ? slices - 1 : -1;
  const int n = slices > wave ? (slices - wave + KW - 1) / KW : 0;
  auto load = [&](int set, int i) {
    const int s = wave + i * KW;
    if (s == last) {
      A.load_end(ra[set], s, kleft);
      B.load_end(rb[set], s, kleft);
    } else {
      A.load(ra[set], s);
      B.load(rb[set], s);
    }
  };
  auto mul = [&](int set) {
    bf16x8 fa[NA], fb[NB];
    A.frags(ra[set], fa);
    B.frags(rb[set], fb);
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int i = 0; i < NB; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[i], fa[j], acc[i][j], 0, 0, 0);
  };
  if (n == 1) {
    load(0, 0);
    mul(0);
  } else if (n > 1) {
    load(0, 0);
    load(1, 1);
    int i = 0;
    for (; i + 3 < n; i += 2) {
      mul(0);
      load(0, i + 2);
      mul(1);
      load(1, i + 3);
    }
    mul(0);
    const bool three = i + 2 < n;
    if (three) load(0, i + 2);
    mul(1);
    if (three) mul(0);
  }

  // partial tiles: [wave][row][chunks of four columns], a row's chunks XORed with the row so that the eight lanes of a pass of
  // writes meet different banks (their rows are neighbours, or four / two apart where A is transposed in registers)
  float* lds = reinterpret_cast<float*>(lds_raw);
  constexpr int CH = TN / 4, RS = A_KC ? 0 : (NA == 4 ? 2 : 1);
  auto chunk_at = [&](int w, int row, int c) { return lds + ((size_t)w * TM + row) * TN + ((c ^ ((row >> RS) & (CH - 1) & 7)) * 4); };
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int row = A_KC ? 16 * j + l16 : NA * l16 + j;
    if constexpr (B_KC) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        *reinterpret_cast<float4*>(chunk_at(wave, row, 4 * i + lg)) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    } else if constexpr (NB == 4) {
      // tile i holds columns 4 c + i, c = 4 lg + e: one e of the four tiles is a chunk
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<float4*>(chunk_at(wave, row, 4 * lg + e)) = make_float4(acc[0][j][e], acc[1][j][e], acc[2][j][e], acc[3][j][e]);
    } else {
      // columns 2 c + i: two e of the two tiles
#pragma unroll
      for (int e = 0; e < 4; e += 2)
        *reinterpret_cast<float4*>(chunk_at(wave, row, 2 * lg + e / 2)) =
            make_float4(acc[0][j][e], acc[1][j][e], acc[0][j][e + 1], acc[1][j][e + 1]);
    }
  }
  __syncthreads();
  float v[VEC], p[KW][VEC];
#pragma unroll
  for (int w = 0; w < KW; ++w) {
    if constexpr (VEC == 2) {
      const float2 t = *reinterpret_cast<const float2*>(chunk_at(w, orow, ocol >> 2) + (ocol & 2));
      p[w][0] = t.x; p[w][1] = t.y;
    } else {
#pragma unroll
      for (int q = 0; q < VEC / 4; ++q) {
        const float4 t = *reinterpret_cast<const float4*>(chunk_at(w, orow, (ocol >> 2) + q));
        p[w][4 * q] = t.x; p[w][4 * q + 1] = t.y; p[w][4 * q + 2] = t.z; p[w][4 * q + 3] = t.w;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
#pragma unroll
    for (int w = 1; w < KW; w *= 2)
#pragma unroll
      for (int q = 0; q + w < KW; q += 2 * w) p[q][e] += p[q + w][e];
    v[e] = p[0][e];
  }

  const bool ok = gm < a.M && gn < a.N;              // N is a multiple of 8: a thread's columns are all in or all out
  OutVec o;
  if (EPI == EPI_STORE) {
    if (a.bias != nullptr) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[e] += (float)bias.v[e];
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) o.v[e] = (bf16)v[e];
  } else if (EPI == EPI_BIAS_GELU) {
    OutVec g;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float x = a.bias != nullptr ? v[e] + (float)bias.v[e] : v[e];
      g.v[e] = (bf16)x;
      o.v[e] = (bf16)gelu_fwd(x, a.gelu_tanh != 0);
    }
    if (ok) *reinterpret_cast<OutVec*>((bf16*)a.aux + (size_t)gm * a.ldaux + gn) = g;
  } else if (EPI == EPI_DGELU) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) o.v[e] = (bf16)(v[e] * gelu_bwd((float)pre.v[e], a.gelu_tanh != 0));
  } else if (EPI == EPI_CE) {
    float mx = -INFINITY, se = 0.f;
    if (gn < a.N) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) mx = fmaxf(mx, v[e]);
    }
    mx = split_max<TPR>(mx);
    const float mxl = mx * 1.4426950408889634f;
    if (gn < a.N) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) se += __builtin_amdgcn_exp2f(fmaf(v[e], 1.4426950408889634f, -mxl));
    }
    se = split_sum<TPR>(se);
    if (ok && target >= 0 && target < VEC) {
      float t = v[0];
#pragma unroll
      for (int e = 1; e < VEC; ++e) t = target == e ? v[e] : t;
      a.t_out[gm] = t;
    }
    if (gm < a.M && tid % TPR == 0) {
      a.part_m[(size_t)tile_n * a.M + gm] = mx;
      a.part_s[(size_t)tile_n * a.M + gm] = se;
    }
    if (a.C == nullptr) return;
#pragma unroll
    for (int e = 0; e < VEC; ++e) o.v[e] = (bf16)v[e];
  }
  if (ok) *reinterpret_cast<OutVec*>((bf16*)a.C + (size_t)gm * a.ldc + gn) = o;
}

// Work item id of `total` to a tile: an XCD (ids congruent mod 8) takes consecutive tiles of a walk along the shorter side of the
// output first, so that its L2 sees all panels of that side and an eighth of the other's.
template <int TM, int TN>
__device__ __forceinline__ void split_tile_of(const GemmArgs& a, int id, int* tile_m, int* tile_n) {
  const int tm = (a.M + TM - 1) / TM, tn = (a.N + TN - 1) / TN;
  const int total = tm * tn, x = id & 7, per = total >> 3, more = total & 7;
  const int q = x * per + (x < more ? x : more) + (id >> 3);
  if (tm <= tn) {
    *tile_n = (int)((unsigned)q / (unsigned)tm);
    *tile_m = q - *tile_n * tm;
  } else {
    *tile_m = (int)((unsigned)q / (unsigned)tn);
    *tile_n = q - *tile_m * tn;
  }
}

template <int TM, int TN> constexpr int split_waves_per_simd() { return TM * TN <= 2048 ? 4 : 2; }

template <bool A_KC, bool B_KC, int EPI, int TM, int TN>
__global__ __launch_bounds__(64 * kSplitWaves, (split_waves_per_simd<TM, TN>())) void gemm_bf16_split_kernel(GemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  int tile_m, tile_n;
  split_tile_of<TM, TN>(a, blockIdx.x, &tile_m, &tile_n);
  gemm_split_tile<A_KC, B_KC, EPI, TM, TN>(a, tile_m, tile_n, lds_raw);
}

// An input gradient and column sums beside it: the workgroups behind the tiles.
template <int TM, int TN>
__global__ __launch_bounds__(64 * kSplitWaves, (split_waves_per_simd<TM, TN>())) void gemm_bf16_split_colsum_kernel(GemmArgs a, ColsumJob job,
                                                                                                                     int tiles) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int id = blockIdx.x;
  if (id >= tiles) {
    colsum_block<bf16, 64 * kSplitWaves>(job, id - tiles, reinterpret_cast<float*>(lds_raw));
    return;
  }
  int tile_m, tile_n;
  split_tile_of<TM, TN>(a, id, &tile_m, &tile_n);
  gemm_split_tile<true, true, EPI_STORE, TM, TN>(a, tile_m, tile_n, lds_raw);
}

// Weight gradients of one K that do not depend on each other, in one launch.
struct SplitGroup {
  int tile_begin[kMaxGroup];           // first work item of each problem; past the grid for problems that do not exist
  GemmArgs args[kMaxGroup];
};
template <int TM, int TN>
__global__ __launch_bounds__(64 * kSplitWaves, (split_waves_per_simd<TM, TN>())) void gemm_bf16_split_group_kernel(SplitGroup g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int id = blockIdx.x;
  GemmArgs a = g.args[0];
  int first = 0;
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i)
    if (id >= g.tile_begin[i]) { a = g.args[i]; first = g.tile_begin[i]; }
  int tile_m, tile_n;
  split_tile_of<TM, TN>(a, id - first, &tile_m, &tile_n);
  gemm_split_tile<false, false, EPI_STORE, TM, TN>(a, tile_m, tile_n, lds_raw);
}

// A weight gradient w and an input gradient x that do not depend on each other; the one of longer k leads.
template <int TM, int TN>
__global__ __launch_bounds__(64 * kSplitWaves, (split_waves_per_simd<TM, TN>())) void gemm_bf16_split_dual_kernel(GemmArgs w, GemmArgs x,
                                                                                                                   int first) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int id = blockIdx.x, at = id < first ? id : id - first;
  int tile_m, tile_n;
  if ((id < first) == (x.K > w.K)) {
    split_tile_of<TM, TN>(x, at, &tile_m, &tile_n);
    gemm_split_tile<true, true, EPI_STORE, TM, TN>(x, tile_m, tile_n, lds_raw);
  } else {
    split_tile_of<TM, TN>(w, at, &tile_m, &tile_n);
    gemm_split_tile<false, false, EPI_STORE, TM, TN>(w, tile_m, tile_n, lds_raw);
  }
}

// ---- which products take these tiles (host arithmetic) -----------------------------------------------------------------------------
enum { SPLIT_NONE = 0, SPLIT_64, SPLIT_32X64, SPLIT_32 };
constexpr int kSplitTm[4] = {0, 64, 32, 32}, kSplitTn[4] = {0, 64, 64, 32};
inline int split_tiles(int form, int M, int N) {
  return ((M + kSplitTm[form] - 1) / kSplitTm[form]) * ((N + kSplitTn[form] - 1) / kSplitTn[form]);
}
// Microseconds of a launch of `tiles` tiles, the longest of `nk` slices and all together of `work` = sum of tiles x slices: a start, the
// longest wave's slices, further rounds of the chip (a workgroup of the larger two forms a compute unit, two of the smallest), and the
// operands' way through the caches.  Fitted to 1000 products of the three layouts (64 .. 8192 x 16 .. 6600 x 24 .. 8352), 300 groups of the
// weight gradients of a layer shard and 290 pairs of the logits' gradients; standard deviation 7-11 %.
enum { SPLIT_ALONE = 0, SPLIT_GROUP, SPLIT_DUAL };
inline double split_us(int kind, int form, int tiles, int nk, double work) {
  static const double c[3][3][5] = {            // start, per serial slice, per serial slice of a further round, per further round, work
      {{2.42, 0.99, 0.70, 1.48, 0.069}, {1.95, 0.79, 0.30, 0.39, 0.054}, {1.95, 0.46, 0.06, 0.50, 0.063}},
      {{2.80, 1.05, 0.50, 2.67, 0.060}, {2.04, 0.88, 0.03, 0.68, 0.089}, {2.32, 0.49, 0.00, 1.12, 0.071}},
      {{2.37, 1.09, 0.25, 0.00, 0.087}, {2.09, 0.82, 0.04, 0.20, 0.080}, {2.17, 0.45, 0.00, 0.32, 0.062}}};
  const double* q = c[kind][form - SPLIT_64];
  const int cus = gemm_cu_count(), per = form == SPLIT_32 ? 2 * cus : cus, serial = (nk + kSplitWaves - 1) / kSplitWaves;
  const int more = (tiles + per - 1) / per - 1;
  return q[0] + q[1] * serial + (q[2] * serial + q[3]) * more + q[4] * work / cus;
}
// Slices as dear as these many where every row of a k-contiguous operand (there are kc) starts at the same place of a 128-byte line: the
// sixteen rows of a request then seem to meet in one bank of the vector cache (1068 x 848 x 832 in 64 x 64 9.2 us, x 848 7.8; neither
// another deal of the slices, other first slices for every tile nor requests of whole lines changed that).
inline double split_slow(int kc, int K) { return K % 64 ? 1.0 : kc == 2 ? 1.4 : kc == 1 ? 1.1 : 1.0; }
inline double split_us(int form, int M, int N, int K, int kc) {
  const int t = split_tiles(form, M, N), nk = (K + 31) / 32;
  const double start = 2.0;
  return start + split_slow(kc, K) * (split_us(SPLIT_ALONE, form, t, nk, (double)t * nk) - start);
}
// Microseconds of t 128-wide tiles of all problems of a launch, at most one a compute unit, the longest of nk slices
inline double v2_few_us(int t, int nk) { return 3.0 + 0.245 * nk + 3.2 * t / gemm_cu_count(); }
// Microseconds of a product in the large tiles, nearer than the plan's price where tiles are few: one 128-wide tile a compute unit, whole or
// all in k-pieces (two launches: 15 us and more, where the plan expects 10).
inline double v2_few_us(const V2Plan& p, int K) {
  const int cus = gemm_cu_count(), nk = v2_slices(K);
  if (p.bn == V2_SMALL && p.split == 1 && p.full_tiles <= cus) return v2_few_us(p.full_tiles, nk);
  if (p.bn == V2_SMALL && p.full_tiles == 0) return 10.5 + 0.05 * nk / p.split + 11.0 * p.tail_tiles * p.split / cus;
  return p.cost;
}
// The form that is fastest by these prices, and its price (form SPLIT_NONE, price `than`: none beats that by an eighth).  wide: only forms of
// 64 columns (the cross-entropy partials' column tiles).  Large tiles / these, us: fwd 400 x 288 x 192 4.5 / 2.7, 123 x 1888 x 1888 15.9 / 7.2, 1024 x
// 1920 x 960 stays (10.3 / 16.3), dgrad 400 x 192 x 512 6.0 / 3.9, 915 x 928 x 464 8.3 / 6.1, 1068 x 848 x 848 12.1 / 7.8, wgrad 192 x 512 x 400 6.2 /
// 3.1, 688 x 168 x 2166 15.6 / 8.6.  Of 1000 drawn products 716 take one of these and the mean time falls to 0.665 (0.656 with the best choice
// every time); four are more than 3 % slower, 976 x 1304 x 86 most, 4.3 / 5.5.
constexpr double kSplitMargin = 0.88;
constexpr int kSplitMaxTiles = 4096;
struct SplitPick { int form; double us; };
inline SplitPick split_pick(int M, int N, int K, int kc, double than, bool wide = false) {
  SplitPick best = {SPLIT_NONE, kSplitMargin * than};
  if (gemm_v2_forced_bn()) return {SPLIT_NONE, than};
  for (int form = SPLIT_64; form <= (wide ? SPLIT_32X64 : SPLIT_32); ++form) {
    if (split_tiles(form, M, N) > kSplitMaxTiles) continue;
    const double us = split_us(form, M, N, K, kc);
    if (us < best.us) best = {form, us};
  }
  if (best.form == SPLIT_NONE) best.us = than;
  return best;
}
// ... of a single product
template <bool A_KC, bool B_KC, int EPI>
SplitPick split_pick_alone(int M, int N, int K, bool allow_split) {
  const V2Plan p = v2_plan(M, N, K, allow_split, v2_pick_bn<A_KC, B_KC, EPI>(M, N, K, allow_split));
  return split_pick(M, N, K, (A_KC ? 1 : 0) + (B_KC ? 1 : 0), v2_few_us(p, K), EPI == EPI_CE);
}

// Weight gradients of one K in one launch of these tiles, against the launch or launches of the plan p.  (Only where 128-wide tiles would
// find a compute unit each: beyond, these lose.)  T x H split p ways, large tiles / 64 x 64 / 32 x 64 / 32 x 32, us: 380 x 352, 4 6.7 / 5.7 / 5.5 / 5.0, 92 x
// 640, 8 4.4 / 3.9 / 3.6 / 4.3, 2092 x 320, 4 19 / 13 / 11.5 / 14; 48 x 672, 4 4.1 / 5.9 / 4.8 / 6.1 stays.
inline int split_group_pick(const GemmArgs* probs, int n, const V2GroupPlan& p) {
  if (gemm_v2_group_off() || gemm_v2_forced_bn() || n < 2 || n > kMaxGroup) return SPLIT_NONE;
  const int nk = (probs[0].K + 31) / 32;
  int small = 0;
  for (int q = 0; q < n; ++q) {
    if (probs[q].epi != EPI_STORE || probs[q].bias != nullptr || probs[q].K != probs[0].K) return SPLIT_NONE;
    small += v2_tiles(probs[q], V2_SMALL, V2_SMALL);
  }
  if (small > gemm_cu_count()) return SPLIT_NONE;
  double us = v2_few_us(small, v2_slices(probs[0].K));
  if (p.bn == 0) {
    us = 0.0;
    for (int q = 0; q < n; ++q) us += split_pick_alone<false, false, EPI_STORE>(probs[q].M, probs[q].N, probs[q].K, true).us;
  }
  us *= 0.95;
  int best = SPLIT_NONE;
  for (int form = SPLIT_64; form <= SPLIT_32; ++form) {
    int tiles = 0;
    for (int q = 0; q < n; ++q) tiles += split_tiles(form, probs[q].M, probs[q].N);
    const double t = split_us(SPLIT_GROUP, form, tiles, nk, (double)tiles * nk);
    if (t < us) { us = t; best = form; }
  }
  return best;
}

// A weight gradient a0 and an input gradient a1 in one launch of these tiles, against the launch or launches of d.  T x H x V, as they were / the
// three forms, us: 316 x 704 x 448 6.4 / 6.1 / 5.7 / 4.8, 2486 x 152 x 4200 42 / 29 / 37 / 41, 144 x 1280 x 2896 24 / 20 / 21 / 20; 442 x 768 x 6384 35 / 41 /
// 49 / 48 stays.
inline int split_dual_pick(const GemmArgs& a0, const GemmArgs& a1, const V2Dual& d) {
  if (gemm_v2_forced_bn() || d.bn == V2_B) return SPLIT_NONE;
  const int nk0 = (a0.K + 31) / 32, nk1 = (a1.K + 31) / 32, nk = nk0 > nk1 ? nk0 : nk1;
  const int small = v2_tiles(a0, V2_SMALL, V2_SMALL) + v2_tiles(a1, V2_SMALL, V2_SMALL);
  double us = d.bn == V2_SMALL ? v2_few_us(small, nk)
                               : split_pick_alone<false, false, EPI_STORE>(a0.M, a0.N, a0.K, true).us +
                                     split_pick_alone<true, true, EPI_STORE>(a1.M, a1.N, a1.K, true).us;
  us *= 0.95;
  int best = SPLIT_NONE;
  for (int form = SPLIT_64; form <= SPLIT_32; ++form) {
    const int t0 = split_tiles(form, a0.M, a0.N), t1 = split_tiles(form, a1.M, a1.N);
    if (t0 + t1 > kSplitMaxTiles) continue;
    const double t = split_us(SPLIT_DUAL, form, t0 + t1, nk, (double)t0 * nk0 + (double)t1 * nk1 * split_slow(2, a1.K));
    if (t < us) { us = t; best = form; }
  }
  return best;
}

template <typename Kernel, typename... Args>
hipError_t launch_split(LdsAttrOnce* attr, Kernel kern, size_t lds, int grid, hipStream_t st, Args... args) {
  if (hipError_t e = attr->ensure((const void*)kern, (int)lds); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kSplitWaves), lds, st, args...);
  return hipGetLastError();
}

template <bool A_KC, bool B_KC, int EPI, int TM, int TN>
hipError_t launch_gemm_bf16_split(const GemmArgs& a, int form, hipStream_t st) {
  static LdsAttrOnce attr;
  return launch_split(&attr, gemm_bf16_split_kernel<A_KC, B_KC, EPI, TM, TN>, split_lds_bytes<TM, TN>(), split_tiles(form, a.M, a.N), st, a);
}
template <bool A_KC, bool B_KC, int EPI>
hipError_t launch_gemm_bf16_split(const GemmArgs& a, int form, hipStream_t st) {
  if (form == SPLIT_64) return launch_gemm_bf16_split<A_KC, B_KC, EPI, 64, 64>(a, form, st);
  if constexpr (EPI != EPI_CE)
    if (form == SPLIT_32) return launch_gemm_bf16_split<A_KC, B_KC, EPI, 32, 32>(a, form, st);
  return launch_gemm_bf16_split<A_KC, B_KC, EPI, 32, 64>(a, form, st);
}

// A product by itself, in whichever tiles are priced lowest.
template <bool A_KC, bool B_KC, int EPI>
hipError_t launch_gemm_bf16_any(const GemmArgs& a, hipStream_t st) {
  const SplitPick p = split_pick_alone<A_KC, B_KC, EPI>(a.M, a.N, a.K, a.splitk_ws != nullptr);
  return p.form ? launch_gemm_bf16_split<A_KC, B_KC, EPI>(a, p.form, st) : launch_gemm_bf16_v2<A_KC, B_KC, EPI>(a, a.splitk_ws, st);
}

}  // namespace mlm
