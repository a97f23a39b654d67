// bf16 GEMM for outputs of few tiles (gfx950): C[m,n] = sum_k A(m,k) B(k,n) in tiles of 64 x 64, 32 x 64 or 32 x 32, whose
// k is dealt to the eight waves of a workgroup in 32-deep slices.
//   * Such a product is bound by latency, not by bytes or flops: the 128 x 128 tile leaves most compute units idle there, and
//     its ring of slices, its barriers and its epilogue are a chain of 5 us before anything is stored.  Here a wave copies its own slices
//     into LDS that nobody else reads (two ahead, no barrier in the loop), and the eight partial sums of an output meet once, in LDS.
//   * Larger ones are bound by what a compute unit takes in, 55-60 GB/s of slices (a 64 x 64 tile 8 KB a slice), whatever is under way:
//     three slices ahead in place of two changed nothing.  Fragments loaded straight into registers had reached 45, and 30 where both
//     operands are k-contiguous (3000 x 384 x 1536 26 us, 15 now; 400 x 288 x 192 2.7 both ways): sixteen neighbouring lanes ask for
//     sixteen rows there, the copies four lanes for 64 bytes of one.
//   * Sums: eight chains over k, added in pairs; no result is further from the exact one than in the large tiles' single chain.
#pragma once
#include "gemm_bf16_v2.h"

namespace mlm {

constexpr int kSplitWaves = 8;

// One operand's ROWS rows (64 or 32) of 32-deep slices: copies of a slice into the wave's own stretch of LDS (1 KB each, lane t's 16 bytes at
// 16 t), and its fragments from there.  LDS positions are permuted on the global side so that both kinds of fragment read are free of
// bank conflicts (a pass of a 16-byte read takes lanes 0-3, 12-15 and 20-27 or the others of its 32; one of a transposing read k-rows 0-3 and
// 8-11, 32 bytes each, or 4-7 and 12-15).
template <bool KC, int ROWS> struct SplitOperand;

// k-contiguous: 16 rows of 64 bytes a copy, so that four neighbouring lanes ask for one stretch of memory (loaded straight into registers a
// fragment asks for sixteen rows with sixteen neighbouring lanes: a quarter as many bytes a cycle).
template <int ROWS> struct SplitOperand<true, ROWS> {
  static constexpr int NC = ROWS / 16, NF = ROWS / 16;
  const char* base;                    // the tile's first row (uniform)
  uint32_t off[NC];                    // bytes from there to this lane's unit of slice 0; below 4 GiB: 63 rows of at most 2^24 k
  int unit;                            // its place in the slice, in elements of k
  static __device__ __forceinline__ int sw(int row) { return -(row >> 2) & 3; }
  __device__ __forceinline__ void init(const void* P, int ld, int row0, int nrows, int lane) {
    base = (const char*)P + (size_t)row0 * ld * 2;
    unit = ((lane & 3) ^ sw(lane >> 2)) * 8;
#pragma unroll
    for (int c = 0; c < NC; ++c) off[c] = (uint32_t)(min(row0 + 16 * c + (lane >> 2), nrows - 1) - row0) * (uint32_t)ld * 2 + unit * 2;
  }
  __device__ __forceinline__ const char* at(int s, int c) const { return base + (size_t)s * 64 + off[c]; }
  __device__ __forceinline__ int k_of(int) const { return unit; }
  static __device__ __forceinline__ bf16x8 frag(const unsigned char* ring, int f, int lane) {
    const int row = lane & 15;
    return *reinterpret_cast<const bf16x8*>(ring + f * 1024 + row * 64 + (((lane >> 4) ^ sw(row)) << 4));
  }
};

// Contiguous along m / n: 8 (16) k-rows of 128 (64) bytes a copy; transposed by the fragment read.
template <int ROWS> struct SplitOperand<false, ROWS> {
  static constexpr int U = ROWS / 8, KR = 64 / U, NC = 32 / KR, NF = ROWS / 16;      // units of a k-row, k-rows of a copy
  const char* base;                    // the tile's first column (uniform)
  uint32_t off[2];                     // bytes to this lane's unit of an even / odd copy
  int ld, row;                         // its k-row in the copy
  static __device__ __forceinline__ int sw(int k) { return (U == 8 ? (((k >> 1) & 1) | (((k >> 3) & 1) << 1)) : ((k >> 3) & 1)) << 1; }
  __device__ __forceinline__ void init(const void* P, int ld_, int row0, int nrows, int lane) {
    ld = ld_;
    base = (const char*)P + (size_t)row0 * 2;
    row = lane / U;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int u = (lane & (U - 1)) ^ sw(KR * c + row);
      off[c] = (uint32_t)row * (uint32_t)ld * 2 + (uint32_t)(min(row0 + u * 8, nrows - 8) - row0) * 2;
    }
  }
  __device__ __forceinline__ const char* at(int s, int c) const { return base + (size_t)(s * 32 + c * KR) * 2 * ld + off[c & 1]; }
  __device__ __forceinline__ int k_of(int c) const { return c * KR + row; }
  static __device__ __forceinline__ bf16x8 frag(const unsigned char* ring, int f, int lane) {
    const int l16 = lane & 15, lg = lane >> 4, u = 2 * f + ((l16 & 3) >> 1);
    v4s_t h[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = 8 * lg + 4 * r + (l16 >> 2);
      h[r] = lds_read_tr16(ring + k * (ROWS * 2) + ((u ^ sw(k)) << 4) + (l16 & 1) * 8);
    }
    const v8s_t v = __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
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

// two stages of a slice for every wave, or the partial tiles
template <int TM, int TN> constexpr size_t split_lds_bytes() {
  return (size_t)kSplitWaves * (TM * TN * 4 > 2 * (TM + TN) * 64 ? TM * TN * 4 : 2 * (TM + TN) * 64);
}

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

  // slices wave, wave + 8, ... through two stages of the wave's own LDS; nobody else reads them, so there is no barrier.  The last slice of k
  // may hold less than 32: units past it are copied from sixteen zero bytes.
  constexpr int BYTES_A = TM * 64, STAGE = (TM + TN) * 64, CPS = SplitOperand<A_KC, TM>::NC + SplitOperand<B_KC, TN>::NC;
  const int kleft = a.K & 31, slices = (a.K + 31) >> 5, last = kleft ? slices - 1 : -1;
  const int n = slices > wave ? (slices - wave + KW - 1) / KW : 0;
  unsigned char* ring = lds_raw + wave * (2 * STAGE);
  const uint32_t ring0 = lds_offset_of(ring);
  auto issue = [&](int i) {
    const int s = wave + i * KW;
    const uint32_t dst = ring0 + (i & 1) * STAGE;
    const bool end = s == last;
    auto copies = [&](const auto& op, uint32_t to) {
#pragma unroll
      for (int c = 0; c < std::decay_t<decltype(op)>::NC; ++c) {
        const bf16* src = reinterpret_cast<const bf16*>(op.at(s, c));
        if (end) src = op.k_of(c) < kleft ? src : reinterpret_cast<const bf16*>(&v2_zero16);
        dma16(src, to + c * 1024);
      }
    };
    copies(A, dst);
    copies(B, dst + BYTES_A);
  };
  if (n > 0) issue(0);
  if (n > 1) issue(1);
  for (int i = 0; i < n; ++i) {
    if (i + 1 < n) wait_vmcnt<CPS>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");                     // (no fragment is read ahead of the wait)
    const unsigned char* st = ring + (i & 1) * STAGE;
    bf16x8 fa[NA], fb[NB];
#pragma unroll
    for (int j = 0; j < NA; ++j) fa[j] = SplitOperand<A_KC, TM>::frag(st, j, lane);
#pragma unroll
    for (int j = 0; j < NB; ++j) fb[j] = SplitOperand<B_KC, TN>::frag(st + BYTES_A, j, lane);
    if (i + 2 < n) {
      __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): the stage's fragments are in registers
      __builtin_amdgcn_sched_barrier(0);
      issue(i + 2);
    }
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int q = 0; q < NB; ++q) acc[q][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[q], fa[j], acc[q][j], 0, 0, 0);
  }
  asm volatile("" ::: "memory");

  // partial tiles: [wave][row][chunks of four columns], a row's chunks XORed with the row so that the eight lanes of a pass of
  // writes meet different banks.  A wave's lies over its own stages (64 x 64) or other waves' (then all wait for each other first).
  float* lds = reinterpret_cast<float*>(lds_raw);
  constexpr int CH = TN / 4;
  if constexpr (TM * TN * 4 != 2 * STAGE) __syncthreads();
  auto chunk_at = [&](int w, int row, int c) { return lds + ((size_t)w * TM + row) * TN + ((c ^ (row & (CH - 1) & 7)) * 4); };
#pragma unroll
  for (int j = 0; j < NA; ++j)
#pragma unroll
    for (int i = 0; i < NB; ++i)
      *reinterpret_cast<float4*>(chunk_at(wave, 16 * j + l16, 4 * i + lg)) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
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
    const float mxl = ce_base(mx) * 1.4426950408889634f;
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
// longest wave's slices, further rounds of the chip (a workgroup of the larger two forms a compute unit, two of the smallest), the operands' way through
// the caches, and the wait of two workgroups of the smallest form for each other.  Fitted to 1500 products of the three layouts (16 .. 8192 x 16 .. 6600 x 24
// .. 20000), 300 groups of the weight gradients of a layer shard and 290 pairs of the logits' gradients; standard deviation 7-11 %.
enum { SPLIT_ALONE = 0, SPLIT_WGRAD, SPLIT_GROUP, SPLIT_DUAL };      // (a product by itself: forward or input gradient, weight gradient)
inline double split_us(int kind, int form, int tiles, int nk, double work) {
  // start, per serial slice, per serial slice of a further round, per further round, work, per serial slice of a second workgroup a unit
  static const double c[4][3][6] = {
      {{2.59, 0.80, 0.42, 1.94, 0.065, 0.0}, {2.20, 0.59, 0.24, 1.41, 0.051, 0.0}, {2.10, 0.38, 0.00, 1.06, 0.052, 0.2}},
      {{2.55, 0.706, 0.484, 1.80, 0.079, 0.0}, {2.27, 0.517, 0.495, 0.89, 0.063, 0.0}, {2.06, 0.360, 0.148, 0.50, 0.069, 0.152}},
      {{2.79, 0.88, 0.33, 2.57, 0.063, 0.0}, {2.45, 0.75, 0.22, 1.66, 0.054, 0.0}, {2.50, 0.41, 0.00, 1.10, 0.073, 0.0}},
      {{2.73, 0.67, 0.13, 0.63, 0.093, 0.0}, {2.49, 0.40, 0.00, 0.85, 0.091, 0.0}, {2.30, 0.31, 0.00, 0.57, 0.058, 0.0}}};
  const double* q = c[kind][form - SPLIT_64];
  const int cus = gemm_cu_count(), per = form == SPLIT_32 ? 2 * cus : cus, serial = (nk + kSplitWaves - 1) / kSplitWaves;
  const int more = (tiles + per - 1) / per - 1;
  const double over = tiles <= cus ? 0.0 : tiles >= 2 * cus ? 1.0 : (double)tiles / cus - 1.0;
  return q[0] + q[1] * serial + (q[2] * serial + q[3]) * more + q[4] * work / cus + q[5] * serial * over;
}
inline double split_us(int kind, int form, int M, int N, int K) {
  const int t = split_tiles(form, M, N), nk = (K + 31) / 32;
  return split_us(kind, form, t, nk, (double)t * nk);
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
// The form that is fastest by these prices, and its price (form SPLIT_NONE, price `than`: none beats that by a twelfth).  wide: only forms of
// 64 columns (the cross-entropy partials' column tiles).  Large tiles / 64 x 64 / 32 x 64 / 32 x 32, us: fwd 400 x 288 x 192 4.5 / 3.6 / 3.1 / 2.8, 123 x 1888 x
// 1920 15.4 / 10.2 / 8.2 / 6.8, 273 x 2776 x 2776 22.0 / 16.4 / 22.5 / 28; dgrad 400 x 192 x 512 6.0 / 4.3 / 3.4 / 2.9, 915 x 928 x 448 6.4 / 5.4 / 6.7 / 6.9,
// 2048 x 512 x 512 6.7 / 5.4 / 6.8 / 7.0; wgrad 192 x 512 x 400 6.1 / 4.3 / 3.6 / 3.1, 688 x 168 x 2166 15.5 / 12 / 10 / 8.5; fwd 1024 x 1920 x 960 stays, 10.3 / 12.2.
// wgrad 624 x 416 x 4059 19.0 / 18.9 / 15.5 / 22.5.  Of 818 drawn products of 7.5 us and more the mean time falls to 0.575 (0.559 with the best choice every
// time); six are more than 3 % slower, dgrad 40 x 4112 x 4904 most, 21.0 / 26.4.
constexpr double kSplitMargin = 0.92;
constexpr int kSplitMaxTiles = 4096;
struct SplitPick { int form; double us; };
inline SplitPick split_pick(int kind, int M, int N, int K, double than, bool wide = false) {
  SplitPick best = {SPLIT_NONE, kSplitMargin * than};
  if (gemm_v2_forced_bn()) return {SPLIT_NONE, than};
  for (int form = SPLIT_64; form <= (wide ? SPLIT_32X64 : SPLIT_32); ++form) {
    if (split_tiles(form, M, N) > kSplitMaxTiles) continue;
    const double us = split_us(kind, form, M, N, K);
    if (us < best.us) best = {form, us};
  }
  if (best.form == SPLIT_NONE) best.us = than;
  return best;
}
// ... of a single product
template <bool A_KC, bool B_KC, int EPI>
SplitPick split_pick_alone(int M, int N, int K, bool allow_split) {
  const V2Choice c = v2_choose<A_KC, B_KC, EPI>(M, N, K, allow_split);
  const double us = c.middle ? c.us : v2_few_us(c.plan, K);
  return split_pick(A_KC ? SPLIT_ALONE : SPLIT_WGRAD, M, N, K, us, EPI == EPI_CE);
}

// Weight gradients of one K in one launch of these tiles, against the launch or launches of the plan p.  (Only where 128-wide tiles would
// find a compute unit each: beyond, these lose.)  T x H split p ways, large tiles / 64 x 64 / 32 x 64 / 32 x 32, us: 95 x 384, 4 4.4 / 3.7 / 3.4 / 3.6, 1954
// x 288, 4 18.5 / 12.1 / 10.5 / 9.3; 247 x 896, 8 6.1 / 7.8 / 8.8 / 8.1 stays.
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
// three forms, us: 176 x 896 x 656 8.6 / 5.0 / 5.7 / 5.8, 3218 x 768 x 392 24 / 16 / 22 / 24, 338 x 560 x 3728 25 / 21 / 19 / 19; 442 x 768 x 6384 35 / 37 / 46 /
// 47 stays.  Of 622 drawn pairs 0.904 of the time in the mean (0.882 with the best choice every time), 34 more than 3 % slower (225 x 2592 x 640 8.1 / 10.0); at
// a margin of a tenth 15, but 1300 x 512 x 4000, which gains 4 us, too, stays in large tiles.
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
    const double t = split_us(SPLIT_DUAL, form, t0 + t1, nk, (double)t0 * nk0 + (double)t1 * nk1);
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
