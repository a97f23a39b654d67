// fp32 GEMM for dtype MLM_F32.  Here on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: 157 TFLOP/s on the whole chip, fp32
// products and fp32 accumulation, so the precision is that of a chain of fused multiply-adds); outputs that fill the chip and sums
// that are long go to gemm_f32_pieces.hip.
// Computes C[m,n] = sum_k A(m,k) B(k,n) with either operand stored k-contiguous or not, and the same fused epilogues as
// the bf16 kernel (bias, bias+GeLU with saved pre-activation, GeLU', dlogits).
//
// The order of k inside a sum is free.  The tile kernels use 16 x 16 x 4 MFMAs: the 16-deep chunk c of k is fed to four of
// them with k = 16c + 4g + j in lane group g = lane / 16 (j = 0..3), so a lane's four values of a k-contiguous operand are ONE
// 16-byte access; the B tile is the first operand, so a lane holds four consecutive columns of one row of the result.  The
// split kernel uses 32 x 32 x 2 ones with k = 8c + j in the lower half-wave and 8c + 4 + j in the upper one; its accumulator
// holds, in lane l, column l % 32 and rows 8 (e / 4) + 4 (l / 32) + e % 4.
//
// Three kernels by the number of output tiles (gemm_f32_pick.h holds the rule and the figures):
//   * 128 x 128 tile, 4 waves of 64 x 64: operand tiles of 32 k staged through LDS (registers -> LDS, double buffered).  For few k, 64 at
//     most: with more, products of so many tiles are faster in pieces (at 4096^3 it kept the matrix cores busy 86 % of their cycles).
//   * 64 x 64 tile, 8 waves: 2 x 2 waves of 32 x 32 in two groups that take the two halves of every 64-deep operand tile,
//     so a CU that holds one tile still has two waves per SIMD to cover LDS and global latency.
//   * 32 x 32 or 16 x 16 tile, 8 waves that split k, each copying its share of the operands into LDS that only it reads (no barrier in
//     the loop): for outputs of so few tiles that the serial k loop of one wave, not the matrix rate, is the time.
#include <string.h>
#include <type_traits>
#include <utility>
#include "gemm_f32_common.h"
#include "lds_dma.h"
#include "gemm_f32_pick.h"

namespace mlm {

// One 16 x 16 accumulator tile whose first row / column is (m0, n0): a lane holds four consecutive columns of one row.
template <int EPI>
__device__ __forceinline__ void f32_store_tile(const GemmArgs& a, const floatx4& acc, int m0, int n0, int lane) {
  f32_put4<EPI>(a, acc, m0 + (lane & 15), n0 + 4 * (lane >> 4));
}

// ---- operand tile of ROWS x KT staged through LDS by NT threads ----------------------------------------------------
// KC (k-contiguous in memory): LDS [row][KT + 4]; a fragment is one 16-byte read, rows 4 KT + 16 bytes apart fall on
// different bank groups.  Otherwise: LDS [k][ROWS + 4]; a fragment is four 4-byte reads, the four groups of 16 lanes read
// k-rows four apart, which the 4-float pad puts 16 banks apart.
template <bool KC, int ROWS, int KT, int NT>
struct F32Tile {
  static constexpr int LD = KC ? KT + 4 : ROWS + 4;
  static constexpr int FLOATS = KC ? ROWS * LD : KT * LD;
  static constexpr int PER = ROWS * KT / 4 / NT;             // float4 per thread
  static_assert(ROWS * KT % (4 * NT) == 0, "tile does not divide over the threads");
  float4 reg[PER];
  uint32_t ofs[PER];           // bytes from the tile's first element to this thread's i-th vector (kF32MaxK128 bounds them)
  // where thread tid's i-th vector lies in the tile
  __device__ static __forceinline__ int row_of(int i, int tid) {
    const int v = tid + i * NT;
    return KC ? v / (KT / 4) : (v % (ROWS / 4)) * 4;
  }
  __device__ static __forceinline__ int k_of(int i, int tid) {
    const int v = tid + i * NT;
    return KC ? (v % (KT / 4)) * 4 : v / (ROWS / 4);
  }
  __device__ __forceinline__ void init(int ld, int row0, int nrows, int tid) {
    // rows past the end repeat the last ones (their results are not stored); row counts, and K of a k-contiguous operand,
    // are multiples of 8: a group of four is inside or outside as a whole
#pragma unroll
    for (int i = 0; i < PER; ++i)
      ofs[i] = 4u * (KC ? (uint32_t)min(row_of(i, tid), nrows - 1 - row0) * ld + k_of(i, tid)
                        : (uint32_t)k_of(i, tid) * ld + min(row_of(i, tid), nrows - 4 - row0));
  }
  // tile: its first element (wave-uniform, so a whole tile inside [0, K) costs no address arithmetic per load); kleft = K
  // minus its first k: k past the end counts as zero
  template <bool WHOLE>
  __device__ __forceinline__ void load_one(const float* __restrict__ tile, int ld, int kleft, int tid, int i) {
    if (WHOLE) {
      reg[i] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(tile) + ofs[i]);
    } else {
      const int k = k_of(i, tid);
      const bool in = k < kleft;
      const float* base = in ? tile : tile - (KC ? (size_t)k : (size_t)k * ld);      // not inside: the vector's k = 0
      const float4 x = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(base) + ofs[i]);
      reg[i] = in ? x : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  __device__ __forceinline__ void store_one(float* s, int tid, int i) const {
    *reinterpret_cast<float4*>(s + (KC ? row_of(i, tid) * LD + k_of(i, tid) : k_of(i, tid) * LD + row_of(i, tid))) = reg[i];
  }
  // the four MFMA operands of chunk c (16 k) for the 16 rows from r0
  __device__ static __forceinline__ void frag(const float* s, int r0, int c, int lane, float (&f)[4]) {
    const int row = r0 + (lane & 15), k = 16 * c + 4 * (lane >> 4);
    if (KC) {
      const float4 v = *reinterpret_cast<const float4*>(s + row * LD + k);
      f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = s[(k + j) * LD + row];
    }
  }
};

template <typename F, int... N>
__device__ __forceinline__ void f32_static_for(F&& f, std::integer_sequence<int, N...>) {
  (f(std::integral_constant<int, N>{}), ...);
}

// BM x BN tile; WM x WN waves of (BM / WM) x (BN / WN), KS groups of them that share every KT-deep operand tile along k.  CH: a wave
// keeps that many sums of an element, of every CH-th four k each, and adds them at the end: KS CH chains of K / (KS CH) products.
template <bool A_KC, bool B_KC, int EPI, int BM, int BN, int WM, int WN, int KS, int KT, int CH = 1>
__device__ __forceinline__ void f32_tile(const GemmArgs& a, int tile) {
  constexpr int NT = 64 * WM * WN * KS, TM = BM / WM / 16, TN = BN / WN / 16, NC = KT / 16 / KS;
  typedef F32Tile<A_KC, BM, KT, NT> TA;
  typedef F32Tile<B_KC, BN, KT, NT> TB;
  constexpr int STAGE = TA::FLOATS + TB::FLOATS;
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = wave / (WM * WN), w = wave % (WM * WN);
  const int wm0 = (w / WN) * (BM / WM), wn0 = (w % WN) * (BN / WN);
  const int tiles_m = (a.M + BM - 1) / BM;
  const int m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
  const float* A = (const float*)a.A;
  const float* B = (const float*)a.B;
  static_assert(CH == 1 || CH == 4, "the four MFMAs of a chunk");
  floatx4 sum[CH][TM][TN];
#pragma unroll
  for (int h = 0; h < CH; ++h)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[h][i][j][e] = 0.f;
  floatx4 (&acc)[TM][TN] = sum[0];

  // Tile kt + 1 waits in registers while the first half of tile kt is multiplied, is written to the other LDS buffer in
  // the middle of it (free since the last barrier) and tile kt + 2 is requested vector by vector behind the writes: a
  // request has a whole tile's time to arrive.  Fragments are read one chunk ahead; for the first chunk of tile kt + 1 the
  // barrier sits behind the first MFMA of the last chunk of tile kt, whose fragments are in registers by then.  All of this is
  // issued one operation at a time between the MFMAs: issued in bursts, with the address arithmetic of the loads, it left the
  // pipe idle for 1500 of 5600 cycles per tile.  At sizes that are formed in pieces now: 1024 x 4096 x 1024 91 -> 84 us, with 16 x 16 x 4 instead of
  // 32 x 32 x 2 MFMAs (which also make the stores 16 bytes) 79; 4096^3 1074 -> 1011 -> 997; 1024^3 (64 x 64 tile) 28.8 -> 26.1 -> 23.5.
  TA ta;
  TB tb;
  ta.init(a.lda, m0, a.M, tid);
  tb.init(a.ldb, n0, a.N, tid);
  const float* tileA = A + (A_KC ? (size_t)m0 * a.lda : (size_t)m0);
  const float* tileB = B + (B_KC ? (size_t)n0 * a.ldb : (size_t)n0);
  const int nk = (a.K + KT - 1) / KT;
  constexpr int NV = TA::PER + TB::PER;             // vectors per thread and tile
  auto request_one = [&](auto whole, int kt, int v) {
    constexpr bool W = decltype(whole)::value;
    if (v < TA::PER) ta.template load_one<W>(tileA + (size_t)kt * KT * (A_KC ? 1 : a.lda), a.lda, a.K - kt * KT, tid, v);
    else tb.template load_one<W>(tileB + (size_t)kt * KT * (B_KC ? 1 : a.ldb), a.ldb, a.K - kt * KT, tid, v - TA::PER);
  };
  auto write_one = [&](int kt, int v) {
    float* d = lds_f32 + (kt & 1) * STAGE;
    if (v < TA::PER) ta.store_one(d, tid, v);
    else tb.store_one(d + TA::FLOATS, tid, v - TA::PER);
  };
  float fa[2][TM][4], fb[2][TN][4];
  auto fragment = [&](int buf, int kt, int c, int f) {
    const float* sA = lds_f32 + (kt & 1) * STAGE;
    if (f < TM) TA::frag(sA, wm0 + f * 16, grp * NC + c, lane, fa[buf][f < TM ? f : 0]);
    else TB::frag(sA + TA::FLOATS, wn0 + (f - TM) * 16, grp * NC + c, lane, fb[buf][f < TM ? 0 : f - TM]);
  };
  constexpr int NF = TM + TN, NMF = 4 * TM * TN;
  static_assert(NC % 2 == 0 && NC >= 2 && NF <= NMF, "chunk c of every tile is in buffer c & 1");
  typedef std::integral_constant<bool, true> yes_t;
  typedef std::integral_constant<bool, false> no_t;
#pragma unroll
  for (int v = 0; v < NV; ++v) request_one(no_t{}, 0, v);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    write_one(0, v);
    if (nk > 1) request_one(no_t{}, 1, v);
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < NF; ++f) fragment(0, 0, 0, f);
  // NEXT: there is a tile kt + 1; WHOLE: and a tile kt + 2 that lies inside [0, K)
  auto multiply = [&](auto has_next, auto whole, int kt) {
    constexpr bool NEXT = decltype(has_next)::value, WHOLE = decltype(whole)::value;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      f32_static_for([&](auto n_c) {                  // (a loop of this length is past the compiler's unrolling limit)
        constexpr int n = decltype(n_c)::value, q = n / (TM * TN), i = n / TN % TM, j = n % TN;
        sum[q % CH][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[c & 1][j][q], fa[c & 1][i][q], sum[q % CH][i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (NEXT && c == NC - 1 && n == 0) __syncthreads();
        if (n < NF) {
          if (c + 1 < NC) fragment((c + 1) & 1, kt, c + 1, n);
          else if (NEXT) fragment(0, kt + 1, 0, n);
        }
        if (NEXT && c == NC / 2 - 1) {
#pragma unroll
          for (int v = 0; v < NV; ++v)
            if (v * NMF / NV == n) {
              write_one(kt + 1, v);
              if (WHOLE) request_one(yes_t{}, kt + 2, v);
              else if (kt + 2 < nk) request_one(no_t{}, kt + 2, v);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
      }, std::make_integer_sequence<int, NMF>{});
    }
  };
  const int nwhole = a.K / KT;
  int kt = 0;
  for (; kt + 2 < nwhole; ++kt) multiply(yes_t{}, yes_t{}, kt);
  for (; kt + 1 < nk; ++kt) multiply(yes_t{}, no_t{}, kt);
  multiply(no_t{}, no_t{}, kt);
  if constexpr (CH == 4) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = (sum[0][i][j][e] + sum[1][i][j][e]) + (sum[2][i][j][e] + sum[3][i][j][e]);
  }
  if (KS > 1) __syncthreads();
  if (KS > 1) {
    // the groups' sums meet in LDS ([group - 1][wave][value][lane]) and are added in group order
    float* park = lds_f32 + w * (TM * TN * 4 * 64) + lane;
    constexpr int GS = WM * WN * TM * TN * 4 * 64;
    if (grp > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) park[(grp - 1) * GS + ((i * TN + j) * 4 + e) * 64] = acc[i][j][e];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 0; g < KS - 1; ++g)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i][j][e] += park[g * GS + ((i * TN + j) * 4 + e) * 64];
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) f32_store_tile<EPI>(a, acc[i][j], m0 + wm0 + i * 16, n0 + wn0 + j * 16, lane);
}

template <bool A_KC, bool B_KC, int EPI, int BM, int BN, int WM, int WN, int KS, int KT>
__global__ __launch_bounds__(64 * WM * WN * KS, 2) void gemm_f32_tile_kernel(GemmArgs a) {
  f32_tile<A_KC, B_KC, EPI, BM, BN, WM, WN, KS, KT>(a, blockIdx.x);
}

// 32 x 32 or 16 x 16 tile, 8 waves: wave w sums the w-th eighth of k (in chunks of 8 or 16) and the eight partial tiles are added in LDS,
// in wave order.  A wave copies its eighth, 16 k at a time, into LDS that only it reads, ahead of the products and without a barrier.
// What bounds it is the intake of operands (a 32 x 32 tile asks for 16 flops a byte), and at few tiles the serial eighth of k.  A copy takes
// 16 rows of 64 bytes, or whole k-rows: fragments loaded straight to registers have neighbouring lanes in different rows of a k-contiguous
// operand, one cache line each (us, registers / LDS: 408 x 56 x 7744 with both k-contiguous 29.4 / 21.4, 256 x 512 x 2048 16.6 / 12.0; with one 15.2 /
// 14.4; k-major 752 x 168 x 4504 34.5 / 26.6, but 256 x 512 x 256 4.05 / 4.1 and, in 16 x 16 tiles, 256 x 256 x 2048 8.6 / 9.2; of 278 products
// with both k-contiguous 0.85 of the time in the mean, with one 0.94, k-major 0.965, no sum changed).
// Stages: two of a 32 x 32 tile leave room for two workgroups a unit; three or four, one workgroup, 2-6 % slower in the mean (504 x 1072 x 48
// 4.8 / 6.3 / 6.2, 792 x 72 x 552 6.6 / 7.4 / 7.5, at best 5 % faster at 744 x 1040 x 696).  Four of a 16 x 16 tile: two cost 13 % at 160 x 104 x 7176.
constexpr int kF32SplitWaves = 8;

// One operand's 16 k of a 32 (16) row tile: copies of 1 KB (lane t's 16 bytes at 16 t) and the fragments from there, four k of a row per lane and
// chunk.  LDS positions are permuted on the global side, so that no read meets bank conflicts.
template <bool KC, int TS> struct F32SplitOperand;
template <int TS> struct F32SplitOperand<true, TS> {
  static constexpr int NC = TS / 16;             // a copy: 16 rows of 64 bytes
  const char* base;                              // the tile's first row (uniform)
  uint32_t off[NC];                              // bytes from there (at most 31 rows of 2^24 floats)
  int unit;                                      // this lane's first k of the 16
  static __device__ __forceinline__ int sw(int row) { return -(row >> 2) & 3; }
  __device__ __forceinline__ void init(const void* P, int ld, int row0, int nrows, int lane) {
    base = (const char*)P + (size_t)row0 * ld * 4;
    unit = ((lane & 3) ^ sw(lane >> 2)) * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) off[c] = 4u * ((uint32_t)(min(row0 + 16 * c + (lane >> 2), nrows - 1) - row0) * (uint32_t)ld + unit);
  }
  __device__ __forceinline__ const char* at(int k, int c) const { return base + (size_t)k * 4 + off[c]; }
  __device__ __forceinline__ int k_of(int) const { return unit; }
  // k = CK q + 4 lh .. + 3 of row l (CK = 8, 16)
  static __device__ __forceinline__ void frag(const unsigned char* lds, int q, int l, int lh, float (&f)[4]) {
    const float4 v = *reinterpret_cast<const float4*>(lds + l * 64 + ((((256 / TS / 4) * q + lh) ^ sw(l & 15)) << 4));
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  }
};
template <int TS> struct F32SplitOperand<false, TS> {
  static constexpr int U = TS / 4, KR = 64 / U, NC = 16 / KR;      // 16-byte units of a k-row, k-rows of a copy
  const char* base;
  uint32_t off[NC];
  int kk[NC];                                    // this lane's k of the 16
  // LDS row of k: the four (two) lane groups of a read, four k apart, meet different banks
  static __device__ __forceinline__ int row_of(int k) { return k ^ ((k >> 2) & (TS == 32 ? 1 : 3)); }
  int ld;
  __device__ __forceinline__ void init(const void* P, int ld_, int row0, int nrows, int lane) {
    ld = ld_;
    base = (const char*)P + (size_t)row0 * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      kk[c] = row_of(c * KR + lane / U);
      off[c] = 4u * ((uint32_t)kk[c] * (uint32_t)ld + (min(row0 + lane % U * 4, nrows - 4) - row0));
    }
  }
  __device__ __forceinline__ const char* at(int k, int c) const { return base + (size_t)k * ld * 4 + off[c]; }
  __device__ __forceinline__ int k_of(int c) const { return kk[c]; }
  static __device__ __forceinline__ void frag(const unsigned char* lds, int q, int l, int lh, float (&f)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = *reinterpret_cast<const float*>(lds + row_of((256 / TS) * q + 4 * lh + j) * (TS * 4) + l * 4);
  }
};
// What a copy reads for k past the wave's last.
static __device__ const uint4 f32_zero16 = {0u, 0u, 0u, 0u};

template <int TS> constexpr int f32_split_stages() { return TS == 16 ? 4 : 2; }
template <int TS> constexpr size_t f32_split_lds() { return (size_t)kF32SplitWaves * f32_split_stages<TS>() * TS * 128; }
template <bool A_KC, bool B_KC, int EPI, int TS = 32>
__device__ __forceinline__ void f32_split_tile(const GemmArgs& a, int tile) {
  // TS = 16: 16 x 16 tile, chunks of 16 k of which K is a multiple (f32_split_tile_of)
  constexpr int NWV = kF32SplitWaves, CK = 256 / TS, NE = TS * TS / 64, ST = f32_split_stages<TS>();
  using acc_t = std::conditional_t<TS == 32, floatx16, floatx4>;
  typedef F32SplitOperand<A_KC, TS> OA;
  typedef F32SplitOperand<B_KC, TS> OB;
  constexpr int STAGE = TS * 128, CPS = OA::NC + OB::NC;           // 16 k of both operands; copies
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  const int lane = threadIdx.x & 63, l32 = lane % TS, lh = lane / TS;      // (a lane's row; its four k of a chunk)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles_m = (a.M + TS - 1) / TS;
  const int m0 = (tile % tiles_m) * TS, n0 = (tile / tiles_m) * TS;
  const int nchunk = (a.K + CK - 1) / CK;
  const int k0 = CK * (int)((long)nchunk * wave / NWV), k1 = min(CK * (int)((long)nchunk * (wave + 1) / NWV), a.K);
  const int nk = (k1 - k0 + 15) >> 4;                              // (0: a wave without a chunk)
  OA oa;
  OB ob;
  oa.init(a.A, a.lda, m0, a.M, lane);
  ob.init(a.B, a.ldb, n0, a.N, lane);
  unsigned char* ring = reinterpret_cast<unsigned char*>(lds_f32) + wave * (ST * STAGE);
  const uint32_t ring0 = lds_offset_of(ring);
  auto issue = [&](int i, int stage) {
    const int k = k0 + 16 * i, left = k1 - k;
    auto copies = [&](const auto& op, uint32_t to) {
#pragma unroll
      for (int c = 0; c < std::decay_t<decltype(op)>::NC; ++c) {
        const bf16* src = reinterpret_cast<const bf16*>(op.at(k, c));
        if (left < 16) src = op.k_of(c) < left ? src : reinterpret_cast<const bf16*>(&f32_zero16);
        dma16(src, to + c * 1024);
      }
    };
    copies(oa, ring0 + stage * STAGE);
    copies(ob, ring0 + stage * STAGE + OA::NC * 1024);
  };
  acc_t acc;
#pragma unroll
  for (int e = 0; e < NE; ++e) acc[e] = 0.f;
#pragma unroll
  for (int i = 0; i < ST; ++i)
    if (i < nk) issue(i, i);
  int stage = 0;
  for (int i = 0; i < nk; ++i) {
    // (copies return in order: those of the stages behind this one may be under way)
    const int behind = nk - 1 - i;
    if (behind >= ST - 1) wait_vmcnt<(ST - 1) * CPS>();
    else if (ST > 3 && behind == 2) wait_vmcnt<2 * CPS>();
    else if (ST > 2 && behind == 1) wait_vmcnt<CPS>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");                                 // (no fragment is read ahead of the wait)
    const unsigned char* st = ring + stage * STAGE;
    float fa[16 / CK][4], fb[16 / CK][4];
#pragma unroll
    for (int q = 0; q < 16 / CK; ++q) {
      OA::frag(st, q, l32, lh, fa[q]);
      OB::frag(st + OA::NC * 1024, q, l32, lh, fb[q]);
    }
    if (behind >= ST) {
      __builtin_amdgcn_s_waitcnt(0xC07F);                          // lgkmcnt(0): the stage's fragments are in registers
      __builtin_amdgcn_sched_barrier(0);
      issue(i + ST, stage);
    }
    stage = stage == ST - 1 ? 0 : stage + 1;
#pragma unroll
    for (int q = 0; q < 16 / CK; ++q)
      if (q == 0 || k1 - k0 - 16 * i > 8) {                        // wave-uniform
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if constexpr (TS == 32) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[q][j], fb[q][j], acc, 0, 0, 0);
          else acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[q][j], fb[q][j], acc, 0, 0, 0);
      }
  }
  asm volatile("" ::: "memory");
  // parked over the wave's own stages, nobody else's: [value][lane]
  constexpr int RING = ST * STAGE / 4;
  static_assert(NE * 64 <= RING, "a partial tile fits the stages");
  {
    float* park = lds_f32 + wave * RING + lane;
#pragma unroll
    for (int e = 0; e < NE; ++e) park[e * 64] = acc[e];
  }
  __syncthreads();
  // wave w finishes the tile's values e = 2 w, 2 w + 1 (e = w of the four of a 16 x 16 tile)
  constexpr int PER = NE >= NWV ? NE / NWV : 1;
  const int n = n0 + l32;
  if (n >= a.N || wave * PER >= NE) return;
  const float bias = ((EPI == EPI_STORE || EPI == EPI_BIAS_GELU) && a.bias) ? ((const float*)a.bias)[n] : 0.f;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int e = wave * PER + q;
    float v = 0.f;
#pragma unroll
    for (int p = 0; p < NWV; ++p) v += lds_f32[p * RING + e * 64 + lane];
    const int m = m0 + 8 * (e >> 2) + 4 * lh + (e & 3);
    if (m < a.M) f32_put<EPI>(a, f32_row<EPI>(a, m), m, n, bias, v);
  }
}

template <bool A_KC, bool B_KC, int EPI, int TS>
__global__ __launch_bounds__(64 * kF32SplitWaves) void gemm_f32_split_kernel(GemmArgs a) {
  f32_split_tile<A_KC, B_KC, EPI, TS>(a, blockIdx.x);
}

// The tiles of several weight gradients in one launch: such a GEMM takes 3-6 us whatever its size, and nothing waits for the
// four of a layer shard one by one (four launches of 256 x {256, 512} x 256: 24 -> 11 us in one, 6.9 now).
__global__ __launch_bounds__(64 * kF32SplitWaves) void gemm_f32_split_group_kernel(F32Group g) {
  GemmArgs a;
  const int tile = f32_group_at(g, blockIdx.x, &a);
  f32_split_tile<false, false, EPI_STORE>(a, tile);
}
template <int BM, int BN, int WM, int WN, int KS, int KT, int CH>
__global__ __launch_bounds__(64 * WM * WN * KS, 2) void gemm_f32_tile_group_kernel(F32Group g) {
  GemmArgs a;
  const int tile = f32_group_at(g, blockIdx.x, &a);
  f32_tile<false, false, EPI_STORE, BM, BN, WM, WN, KS, KT, CH>(a, tile);
}

// A weight gradient (its tiles first) and an input gradient that do not depend on each other: 256 x 512 x 256 and 256 x 256 x 512
// take 5.9 us together.  (From registers 8.2, and 14 in two launches.)
template <int TS>
__global__ __launch_bounds__(64 * kF32SplitWaves) void gemm_f32_split_dual_kernel(GemmArgs w, GemmArgs x) {
  const int tiles_w = ((w.M + 31) / 32) * ((w.N + 31) / 32), id = blockIdx.x;
  if (id < tiles_w) f32_split_tile<false, false, EPI_STORE>(w, id);
  else f32_split_tile<true, true, EPI_STORE, TS>(x, id - tiles_w);
}

// The same in 64 x 64 tiles; the longer ones lead.
template <int CH>
__global__ __launch_bounds__(512, 2) void gemm_f32_tile_dual_kernel(GemmArgs w, GemmArgs x) {
  const int tiles_w = ((w.M + 63) / 64) * ((w.N + 63) / 64), tiles_x = ((x.M + 63) / 64) * ((x.N + 63) / 64);
  const bool x_first = x.K > w.K;
  const int id = blockIdx.x, first = x_first ? tiles_x : tiles_w, at = id < first ? id : id - first;
  if ((id < first) == x_first) f32_tile<true, true, EPI_STORE, 64, 64, 2, 2, 2, 64, CH>(x, at);
  else f32_tile<false, false, EPI_STORE, 64, 64, 2, 2, 2, 64, CH>(w, at);
}

// An input gradient and column sums beside it (the workgroups behind the tiles): a launch of 5 us saved, 1024 tokens x 1024 1270 ->
// 1264 us a step.
template <int TS>
__global__ __launch_bounds__(64 * kF32SplitWaves) void gemm_f32_split_colsum_kernel(GemmArgs a, ColsumJob job) {
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  static_assert(colsum_lds_floats<float, 64 * kF32SplitWaves>() * sizeof(float) <= f32_split_lds<TS>(), "column sums' LDS");
  const int tiles = ((a.M + TS - 1) / TS) * ((a.N + TS - 1) / TS), id = blockIdx.x;
  if (id < tiles) f32_split_tile<true, true, EPI_STORE, TS>(a, id);
  else colsum_block<float, 64 * kF32SplitWaves>(job, id - tiles, lds_f32);
}
template <int BM, int BN, int WM, int WN, int KS, int KT>
__global__ __launch_bounds__(64 * WM * WN * KS, 2) void gemm_f32_tile_colsum_kernel(GemmArgs a, ColsumJob job, int tiles) {
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  const int id = blockIdx.x;
  if (id < tiles) f32_tile<true, true, EPI_STORE, BM, BN, WM, WN, KS, KT>(a, id);
  else colsum_block<float, 64 * WM * WN * KS>(job, id - tiles, lds_f32);
}

// Launch of a kernel of f32_split_tile.  (64 KB of LDS in either form: what a launch may ask for as it is.)
static_assert(f32_split_lds<32>() <= 64 * 1024 && f32_split_lds<16>() <= 64 * 1024, "more LDS is an attribute of the kernel");
template <int TS, typename Kernel, typename... Args>
static hipError_t launch_f32_split(Kernel kern, dim3 grid, hipStream_t st, const Args&... args) {
  hipLaunchKernelGGL(kern, grid, dim3(64 * kF32SplitWaves), (f32_split_lds<TS>()), st, args...);
  return hipGetLastError();
}
template <bool A_KC, bool B_KC, int EPI, int TS>
static hipError_t launch_f32_split_alone(const GemmArgs& a, hipStream_t st) {
  return launch_f32_split<TS>(gemm_f32_split_kernel<A_KC, B_KC, EPI, TS>, dim3(((a.M + TS - 1) / TS) * ((a.N + TS - 1) / TS)), st, a);
}
template <int TS>
static hipError_t launch_f32_split_colsum(const GemmArgs& a, const ColsumJob& j, hipStream_t st) {
  return launch_f32_split<TS>(gemm_f32_split_colsum_kernel<TS>, dim3(((a.M + TS - 1) / TS) * ((a.N + TS - 1) / TS) + j.blocks), st, a, j);
}
template <int TS>
static hipError_t launch_f32_split_dual(const GemmArgs& w, const GemmArgs& x, int tiles_w, hipStream_t st) {
  return launch_f32_split<32>(gemm_f32_split_dual_kernel<TS>, dim3(tiles_w + ((x.M + TS - 1) / TS) * ((x.N + TS - 1) / TS)), st, w, x);
}

// LDS of a workgroup of f32_tile
template <bool A_KC, bool B_KC, int BM, int BN, int WM, int WN, int KS, int KT> constexpr size_t f32_tile_lds() {
  constexpr int NT = 64 * WM * WN * KS;
  constexpr size_t kStages = 2 * (size_t)(F32Tile<A_KC, BM, KT, NT>::FLOATS + F32Tile<B_KC, BN, KT, NT>::FLOATS) * 4;
  constexpr size_t kPark = (size_t)(KS - 1) * BM * BN * 4;
  constexpr size_t kLds = kStages > kPark ? kStages : kPark;
  static_assert(kLds <= 160 * 1024, "LDS budget");
  return kLds;
}

template <bool A_KC, bool B_KC, int EPI, int BM, int BN, int WM, int WN, int KS, int KT>
static hipError_t launch_f32_tile(const GemmArgs& a, hipStream_t st) {
  constexpr size_t kLds = f32_tile_lds<A_KC, B_KC, BM, BN, WM, WN, KS, KT>();
  auto kern = gemm_f32_tile_kernel<A_KC, B_KC, EPI, BM, BN, WM, WN, KS, KT>;
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(64 * WM * WN * KS), kLds, st, a);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int KS, int KT>
static hipError_t launch_f32_tile_colsum(const GemmArgs& a, const ColsumJob& j, hipStream_t st) {
  constexpr size_t kTile = f32_tile_lds<true, true, BM, BN, WM, WN, KS, KT>();
  constexpr size_t kSums = colsum_lds_floats<float, 64 * WM * WN * KS>() * sizeof(float), kLds = kTile > kSums ? kTile : kSums;
  auto kern = gemm_f32_tile_colsum_kernel<BM, BN, WM, WN, KS, KT>;
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  hipLaunchKernelGGL(kern, dim3(tiles + j.blocks), dim3(64 * WM * WN * KS), kLds, st, a, j, tiles);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int KS, int KT, int CH>
static hipError_t launch_f32_tile_group(const F32Group& g, int total, hipStream_t st) {
  constexpr size_t kLds = f32_tile_lds<false, false, BM, BN, WM, WN, KS, KT>();
  auto kern = gemm_f32_tile_group_kernel<BM, BN, WM, WN, KS, KT, CH>;
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(total), dim3(64 * WM * WN * KS), kLds, st, g);
  return hipGetLastError();
}

template <bool A_KC, bool B_KC, int EPI>
static hipError_t launch_f32_layout(const GemmArgs& a, hipStream_t st) {
  if (const int bt = f32_pieces_pick(a.M, a.N, a.K)) return launch_f32_pieces(a, bt, st);
  switch (f32_pick(a.M, a.N, a.K)) {
    case 32:
      return f32_split_tile_of(a.M, a.N, a.K) == 16 ? launch_f32_split_alone<A_KC, B_KC, EPI, 16>(a, st)
                                                    : launch_f32_split_alone<A_KC, B_KC, EPI, 32>(a, st);
    case 64: return launch_f32_tile<A_KC, B_KC, EPI, 64, 64, 2, 2, 2, 64>(a, st);
    default: return launch_f32_tile<A_KC, B_KC, EPI, 128, 128, 2, 2, 1, 32>(a, st);
  }
}

// Weight gradients (both operands k-major, plain store) of one K: those in pieces share a launch per tile size (f32_group_tiles), the others
// as f32_group_plan says.
hipError_t launch_gemm_f32_wgrads(const GemmArgs* all, int n_all, hipStream_t st) {
  bool together = n_all >= 2 && n_all <= kF32Group;
  for (int q = 0; q < n_all && together; ++q)
    together = !all[q].a_kc && !all[q].b_kc && all[q].epi == EPI_STORE && all[q].K == all[0].K;
  GemmArgs probs[kF32Group];
  int M[kF32Group], N[kF32Group], n = 0;
  for (int q = 0; q < n_all && !together; ++q)
    if (hipError_t e = launch_gemm_f32(all[q], st); e != hipSuccess) return e;
  if (!together) return hipSuccess;
  for (int q = 0; q < n_all; ++q) {
    M[q] = all[q].M;
    N[q] = all[q].N;
  }
  const F32GroupTiles tiles = f32_group_tiles(M, N, n_all, all[0].K);
  for (int bt : {128, 64}) {
    F32Group g;
    memset(&g, 0, sizeof(g));
    int m = 0, total = 0;
    for (int q = 0; q < n_all; ++q) {
      if (tiles.tile[q] != bt) continue;
      g.a[m] = all[q];
      g.tile_begin[m++] = total;
      total += ((all[q].M + bt - 1) / bt) * ((all[q].N + bt - 1) / bt);
    }
    if (m == 0) continue;
    for (int q = m; q < kF32Group; ++q) g.tile_begin[q] = total;
    if (hipError_t e = launch_f32_pieces_group(g, total, bt, st); e != hipSuccess) return e;
  }
  for (int q = 0; q < n_all; ++q) {
    if (tiles.tile[q]) continue;
    M[n] = all[q].M;
    N[n] = all[q].N;
    probs[n++] = all[q];
  }
  if (n == 0) return hipSuccess;
  const F32GroupPlan p = f32_group_plan(M, N, n, probs[0].K);
  auto launch = [&](int b, int chains, bool wide, bool narrow) {      // those that take the 128-wide tile alone, and / or the others
    F32Group g;
    memset(&g, 0, sizeof(g));
    int total = 0, m = 0;
    for (int q = 0; q < n; ++q) {
      if (!(f32_pick(M[q], N[q], probs[q].K) == 128 ? wide : narrow)) continue;
      g.a[m] = probs[q];
      g.tile_begin[m++] = total;
      total += ((M[q] + b - 1) / b) * ((N[q] + b - 1) / b);
    }
    for (; m < kF32Group; ++m) g.tile_begin[m] = total;
    if (b == 128) return launch_f32_tile_group<128, 128, 2, 2, 1, 32, 1>(g, total, st);
    if (b == 64) return chains == 8 ? launch_f32_tile_group<64, 64, 2, 2, 2, 64, 4>(g, total, st)
                                    : launch_f32_tile_group<64, 64, 2, 2, 2, 64, 1>(g, total, st);
    return launch_f32_split<32>(gemm_f32_split_group_kernel, dim3(total), st, g);
  };
  if (p.wide_apart)
    if (hipError_t e = launch(128, 1, true, false); e != hipSuccess) return e;
  if (p.tile) return launch(p.tile, p.chains, !p.wide_apart, true);
  for (int q = 0; q < n; ++q)
    if (!p.wide_apart || f32_pick(M[q], N[q], probs[q].K) != 128)
      if (hipError_t e = launch_gemm_f32(probs[q], st); e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_gemm_f32_dgrad_colsum(const GemmArgs& a, const ColsumJob& j, hipStream_t st) {
  if (const int bt = f32_pieces_pick(a.M, a.N, a.K)) return launch_f32_pieces_colsum(a, j, bt, st);
  switch (f32_pick(a.M, a.N, a.K)) {
    case 32: return f32_split_tile_of(a.M, a.N, a.K) == 16 ? launch_f32_split_colsum<16>(a, j, st) : launch_f32_split_colsum<32>(a, j, st);
    case 64: return launch_f32_tile_colsum<64, 64, 2, 2, 2, 64>(a, j, st);
    default: return launch_f32_tile_colsum<128, 128, 2, 2, 1, 32>(a, j, st);
  }
}

template <int CH>
static hipError_t launch_f32_tile_dual(const GemmArgs& w, const GemmArgs& x, dim3 grid, hipStream_t st) {
  constexpr size_t k0 = f32_tile_lds<false, false, 64, 64, 2, 2, 2, 64>(), k1 = f32_tile_lds<true, true, 64, 64, 2, 2, 2, 64>();
  constexpr size_t kLds = k0 > k1 ? k0 : k1;
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)gemm_f32_tile_dual_kernel<CH>, (int)kLds); e != hipSuccess) return e;
  hipLaunchKernelGGL(gemm_f32_tile_dual_kernel<CH>, grid, dim3(512), kLds, st, w, x);
  return hipGetLastError();
}

hipError_t launch_gemm_f32_dual(const GemmArgs& w, const GemmArgs& x, hipStream_t st) {
  const F32DualPick p = f32_dual_pick(w.M, w.N, w.K, x.M, x.N, x.K);
  const int b = p.tile;
  if (p.pieces) return launch_f32_pieces_dual(w, x, st);
  if (b == 0) {
    if (hipError_t e = launch_gemm_f32(w, st); e != hipSuccess) return e;
    return launch_gemm_f32(x, st);
  }
  auto tiles = [b](const GemmArgs& a) { return ((a.M + b - 1) / b) * ((a.N + b - 1) / b); };
  const dim3 grid(tiles(w) + tiles(x));
  if (b == 32) {
    return f32_split_tile_of(x.M, x.N, x.K) == 16 ? launch_f32_split_dual<16>(w, x, tiles(w), st) : launch_f32_split_dual<32>(w, x, tiles(w), st);
  }
  return p.chains == 8 ? launch_f32_tile_dual<4>(w, x, grid, st) : launch_f32_tile_dual<1>(w, x, grid, st);
}

hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t st) {
  if (a.a_kc && !a.b_kc) {
    switch (a.epi) {
      case EPI_STORE: return launch_f32_layout<true, false, EPI_STORE>(a, st);
      case EPI_BIAS_GELU: return launch_f32_layout<true, false, EPI_BIAS_GELU>(a, st);
      case EPI_DLOGITS: return launch_f32_layout<true, false, EPI_DLOGITS>(a, st);
      default: return hipErrorInvalidValue;
    }
  }
  if (a.a_kc && a.b_kc) {
    switch (a.epi) {
      case EPI_STORE: return launch_f32_layout<true, true, EPI_STORE>(a, st);
      case EPI_DGELU: return launch_f32_layout<true, true, EPI_DGELU>(a, st);
      default: return hipErrorInvalidValue;
    }
  }
  if (!a.a_kc && !a.b_kc && a.epi == EPI_STORE) return launch_f32_layout<false, false, EPI_STORE>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace mlm
