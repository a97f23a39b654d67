// fp32 products on the bf16 matrix cores, which are sixteen times as fast as the fp32 ones.  An fp32 value is the exact sum of three
// bf16 values, x = h + m + l, each what rounding to nearest leaves of the last (8 + 8 + 8 significant bits).  Of the nine products of
// two such sums the six largest are formed, exactly, in the matrix cores' fp32 sums; the three dropped ones are below 2^-26 |a b|.  The
// products of the largest pieces have sums of their own (cor[] holds the others), because the matrix core cuts off what lies below the
// last bit of a sum: all in one sum, results were 2e-7 of their size too low on average, and 2.5 times as far off.
// Against 64 bits (1024 x 1024 outputs, N(0, 1) x N(0, 0.02), 2-norms; fp32 matrix cores one chain / two chains / here): K = 1024 5.7e-7 /
// 4.1e-7 / 1.9e-7, 4096 1.2e-6 / 8.1e-7 / 4.0e-7; in the 64-wide tile, whose k is four chains, 9.8e-8 and 1.9e-7.  All-positive operands
// 4.6e-7 / 2.3e-7 / 1.7e-7 and 9.3e-7 / 4.7e-7 / 3.3e-7.  (Pieces below 2^-126 are the matrix core's denormals, exact to 2^-133: a value keeps all
// of its bits down to 2^-110.)
//
// Bound by the chip's power: at 4096^3 the clock falls to 1.65 GHz, where the matrix pipe is busy 70 % of the cycles, 207 TFLOP/s = 1.24
// PFLOP/s of bf16 products, what the bf16 kernels reach (fp32 matrix cores: 139).  A value is split once per workgroup, on its way from
// registers to LDS (22 vector operations per four values, spread between the MFMAs).  Two waves per SIMD: one alone issues these
// operations at half rate (four waves of 64 x 64 over 32 k a step, one workgroup per compute unit: no faster at 4096^3, and 130 us
// instead of 92 at 1024 x 8192 x 1024).  v_mfma_f32_32x32x16 rather
// than 16x16x32: half as many MFMAs to issue, and half of the operand registers, without which two waves do not fit beside 128 sums.
//   * 128 x 128 tile, 4 waves of 64 x 64, 16 k a step, two workgroups per compute unit.
//   * 64 x 64 tile for outputs of few tiles: 8 waves, 64 k a step, of which a group of two waves takes 16.  Twice the splitting per flop.
// gemm_f32_pick.h holds the rule and the figures.
#include <string.h>
#include <type_traits>
#include <utility>
#include "gemm_f32_common.h"
#include "lds_dma.h"

namespace mlm {

// Operand tile of ROWS x KT, KT = 16 KS, loaded by NT = ROWS KT / 8 threads into registers (two vectors of four) and stored as bf16
// pieces in LDS: [part of 16 k][piece] of [ROWS][16 k] (KC) or [16 k][ROWS].
template <bool KC, int ROWS, int KS>
struct F32PieceTile {
  static constexpr int KT = 16 * KS, NT = ROWS * KT / 8;
  // (parts 32 bytes apart in a bank row: a pass of an 8-byte write takes 16 lanes, which hold the row of four parts, and 128 bytes)
  static constexpr int PLANE = ROWS * 32, PART = 3 * PLANE + (KS > 1 ? 32 : 0), BYTES = KS * PART;
  float4 reg[2][2];            // of two tiles
  uint32_t ofs[KC ? 2 : 1];
  __device__ static __forceinline__ int row_of(int i, int tid) { return KC ? (tid + i * NT) / (KT / 4) : tid % (ROWS / 8) * 8; }
  __device__ static __forceinline__ int k_of(int tid) { return KC ? tid % (KT / 4) * 4 : tid / (ROWS / 8); }
  __device__ __forceinline__ void init(int ld, int row0, int nrows, int tid) {
    // rows past the end repeat the last ones (their results are not stored)
#pragma unroll
    for (int i = 0; i < (KC ? 2 : 1); ++i)
      ofs[i] = 4u * (KC ? (uint32_t)min(row_of(i, tid), nrows - 1 - row0) * ld + k_of(tid)
                        : (uint32_t)k_of(tid) * ld + min(row_of(i, tid), nrows - 8 - row0));
  }
  // tile: its first element (wave-uniform)
  __device__ __forceinline__ void load_one(const float* __restrict__ tile, int set, int i) {
    reg[set][i] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(tile) + ofs[KC ? i : 0] + (KC ? 0 : 16 * i));
  }
  // a tile of which only the first kin k count; the others are zeros
  __device__ __forceinline__ void load_some(const float* __restrict__ tile, int ld, int kin, int tid, int set, int i) {
    const int k = k_of(tid);
    const bool in = k < kin;
    const uint32_t at = ofs[KC ? i : 0] + (KC ? 0 : 16 * i), o = in ? at : at - 4u * (KC ? (uint32_t)k : (uint32_t)k * ld);
    const float4 x = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(tile) + o);
    reg[set][i] = in ? x : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // Bank swizzles: a pass of a 16-byte read meets every (row mod 8) twice, in groups of eight rows of either parity; a pass of a
  // transposing read takes 64 bytes of each of four consecutive k.
  __device__ static __forceinline__ int kc_at(int row, int k) { return row * 32 + ((((k >> 3) ^ (row >> 3)) & 1) << 4) + (k & 4) * 2; }
  __device__ static __forceinline__ int mn_at(int k, int row) {
    const int s = ROWS == 128 ? (k & 3) << 2 : (k & 2) << 1;      // (rows of 256 / 128 bytes)
    return k * (ROWS * 2) + (((row >> 3) ^ s) << 4) + (row & 7) * 2;
  }
  __device__ static __forceinline__ int lds_of(int i, int tid) {
    const int k = k_of(tid);
    return (k >> 4) * PART + (KC ? kc_at(row_of(i, tid), k & 15) : mn_at(k & 15, row_of(i, tid)));
  }
  // operand registers of the 32 x 32 x 16 MFMA for the 32 rows from r0
  __device__ static __forceinline__ bf16x8 frag(const unsigned char* plane, int r0, int lane) {
    if (KC) {
      const int row = r0 + (lane & 31);
      return *reinterpret_cast<const bf16x8*>(plane + kc_at(row, (lane >> 5) * 8));
    }
    const int l16 = lane & 15;
    v4s_t h[2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
      h[r] = lds_read_tr16(plane + mn_at(8 * (lane >> 5) + 4 * r + (l16 >> 2), r0 + (lane & 16) + 4 * (l16 & 3)));
    const v8s_t v = __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
};

__device__ __forceinline__ uint32_t f32p_pair(float x, float y) {
  uint32_t v;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(v) : "v"(x), "v"(y));
  return v;
}
__device__ __forceinline__ float f32p_lo(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float f32p_hi(uint32_t v) { return __builtin_bit_cast(float, v & 0xffff0000u); }

template <typename F, int... N>
__device__ __forceinline__ void f32p_static_for(F&& f, std::integer_sequence<int, N...>) {
  (f(std::integral_constant<int, N>{}), ...);
}

// Walk over the tiles: strips of eight tile rows, column by column.  Workgroup ids go to the eight XCDs in turn; of every `window` ids
// that are resident at a time, those of one XCD take consecutive positions, so that their L2 holds the panels that they share.
__device__ __forceinline__ int f32p_xcd_order(int id, int total, int window) {
  const int base = total <= window ? 0 : (int)((unsigned)id / (unsigned)window) * window;
  const int cnt = total - base < window ? total - base : window;
  const int p = id - base, x = p & 7, per = cnt >> 3, more = cnt & 7;
  return base + x * per + (x < more ? x : more) + (p >> 3);
}
__device__ __forceinline__ void f32p_tile_of(int tiles_m, int tiles_n, int q, int* tile_m, int* tile_n) {
  const int strip = (int)((unsigned)q / (unsigned)(8 * tiles_n)), r = q - strip * (8 * tiles_n);
  const int w = min(8, tiles_m - 8 * strip);
  *tile_n = (int)((unsigned)r / (unsigned)w);
  *tile_m = 8 * strip + r - *tile_n * w;
}

// The wave's tile of TM x TN tiles of 32 x 32 on the fp32 matrix cores, operands read from the caches.
template <bool A_KC, bool B_KC, int TM, int TN>
__device__ __forceinline__ void f32p_plain(const GemmArgs& a, int m0, int n0, int lane, floatx16 (&acc)[TN][TM]) {
  const int l32 = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  for (int k = 0; k < a.K; k += 8) {
    float fa[TM][4], fb[TN][4];
#pragma unroll
    for (int j = 0; j < TM; ++j) f32_frag_global<A_KC>((const float*)a.A, a.lda, min(m0 + 32 * j + l32, a.M - 1), k + 4 * lh, a.K, fa[j]);
#pragma unroll
    for (int i = 0; i < TN; ++i) f32_frag_global<B_KC>((const float*)a.B, a.ldb, min(n0 + 32 * i + l32, a.N - 1), k + 4 * lh, a.K, fb[i]);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[i][q], fa[j][q], acc[i][j], 0, 0, 0);
  }
}

// BT x BT tile; KS groups of waves of 64 x 64 (BT = 128, 2 x 2) or 64 x 32 (BT = 64, 1 x 2), each of which takes 16 of every 16 KS k.
template <bool A_KC, bool B_KC, int BT, int KS, typename Put>
__device__ __forceinline__ void f32p_tile(const GemmArgs& a, int tile, unsigned char* lds, Put&& put) {
  constexpr int BM = BT, BN = BT, TM = 2, TN = BT / 64, KT = 16 * KS, WG = BT / 32;      // waves of a group
  static_assert(BT == 128 || BT == 64, "wave layouts");
  typedef F32PieceTile<A_KC, BM, KS> TA;
  typedef F32PieceTile<B_KC, BN, KS> TB;
  constexpr int STAGE = TA::BYTES + TB::BYTES;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, grp = wave / WG;
  const int wm0 = BT == 128 ? ((wave >> 1) & 1) * 64 : 0, wn0 = (wave & 1) * (32 * TN);
  int tile_m, tile_n;
  f32p_tile_of((a.M + BM - 1) / BM, (a.N + BN - 1) / BN, tile, &tile_m, &tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  TA ta;
  TB tb;
  ta.init(a.lda, m0, a.M, tid);
  tb.init(a.ldb, n0, a.N, tid);
  const float* tileA = (const float*)a.A + (A_KC ? (size_t)m0 * a.lda : (size_t)m0);
  const float* tileB = (const float*)a.B + (B_KC ? (size_t)n0 * a.ldb : (size_t)n0);
  // an even number of steps, counted from the end of K: the first two may begin before 0 and hold zeros there
  const int nk = 2 * ((a.K + 2 * KT - 1) / (2 * KT));
  auto request_one = [&](int set, int kt, int v) {
    const int k = a.K - max(nk - kt, 1) * KT;
    if (v < 2) ta.load_one(tileA + (size_t)k * (A_KC ? 1 : a.lda), set, v & 1);
    else tb.load_one(tileB + (size_t)k * (B_KC ? 1 : a.ldb), set, v & 1);
  };
  uint32_t dst[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) dst[v] = v < 2 ? TA::lds_of(v, tid) : TA::BYTES + TB::lds_of(v - 2, tid);
  uint32_t pc[3][4];                     // pieces of the vectors at work
  float r0 = 0.f, r1 = 0.f, r2 = 0.f, r3 = 0.f, t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
  // step 0 .. 5 of vector v
  auto split_step = [&](int set, int v, int step) {
    const float4& x = v < 2 ? ta.reg[set][v & 1] : tb.reg[set][v & 1];
    const int q = 2 * (v & 1);
    if (step == 0) {
      pc[0][q] = f32p_pair(x.x, x.y);
      pc[0][q + 1] = f32p_pair(x.z, x.w);
      t0 = f32p_lo(pc[0][q]);
      t1 = f32p_hi(pc[0][q]);
    } else if (step == 1) {
      r0 = x.x - t0;
      r1 = x.y - t1;
      t2 = f32p_lo(pc[0][q + 1]);
      t3 = f32p_hi(pc[0][q + 1]);
    } else if (step == 2) {
      r2 = x.z - t2;
      r3 = x.w - t3;
      pc[1][q] = f32p_pair(r0, r1);
      t0 = f32p_lo(pc[1][q]);
    } else if (step == 3) {
      t1 = f32p_hi(pc[1][q]);
      pc[1][q + 1] = f32p_pair(r2, r3);
      r0 -= t0;
      t2 = f32p_lo(pc[1][q + 1]);
    } else if (step == 4) {
      r1 -= t1;
      t3 = f32p_hi(pc[1][q + 1]);
      r2 -= t2;
      r3 -= t3;
    } else {
      pc[2][q] = f32p_pair(r0, r1);
      pc[2][q + 1] = f32p_pair(r2, r3);
    }
  };
  // vector v's pieces; both vectors of a thread lie side by side where memory runs along the rows
  auto write = [&](int kt, int v) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      unsigned char* d = lds + (kt & 1) * STAGE + dst[v] + p * (v < 2 ? TA::PLANE : TB::PLANE);
      if (v < 2 ? A_KC : B_KC) {
        *reinterpret_cast<uint2*>(d) = make_uint2(pc[p][2 * (v & 1)], pc[p][2 * (v & 1) + 1]);
      } else if (v & 1) {
        *reinterpret_cast<uint4*>(d) = make_uint4(pc[p][0], pc[p][1], pc[p][2], pc[p][3]);
      }
    }
  };
  // the largest pieces of two steps, the others of one
  bf16x8 fa[2][TM], fb[2][TN], ga[2][TM], gb[2][TN];
  auto frag_a = [&](int kt, int j, int p) {
    const bf16x8 f = TA::frag(lds + (kt & 1) * STAGE + grp * TA::PART + p * TA::PLANE, wm0 + j * 32, lane);
    if (p == 0) fa[kt & 1][j] = f;
    else ga[p - 1][j] = f;
  };
  auto frag_b = [&](int kt, int i, int p) {
    const bf16x8 f = TB::frag(lds + (kt & 1) * STAGE + TA::BYTES + grp * TB::PART + p * TB::PLANE, wn0 + i * 32, lane);
    if (p == 0) fb[kt & 1][i] = f;
    else gb[p - 1][i] = f;
  };
  floatx16 acc[TN][TM], cor[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = cor[i][j][e] = 0.f;
  auto request_first = [&](int kt) {
    const int k = a.K - (nk - kt) * KT, kin = min(k + KT, KT), k0 = max(k, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      ta.load_some(tileA + (size_t)k0 * (A_KC ? 1 : a.lda), a.lda, kin, tid, kt, i);
      tb.load_some(tileB + (size_t)k0 * (B_KC ? 1 : a.ldb), a.ldb, kin, tid, kt, i);
    }
  };
  auto request_all = [&](int set, int kt) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      request_one(set, kt, v);
      __builtin_amdgcn_sched_barrier(0);       // (in the order in which the loop waits for them)
    }
  };
  auto store_all = [&](int kt) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
#pragma unroll
      for (int s = 0; s < 6; ++s) split_step(kt, v, s);
      write(kt, v);
    }
  };
  request_first(0);
  request_first(1);
  store_all(0);
  request_all(0, 2);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 3; ++p) {
#pragma unroll
    for (int j = 0; j < TM; ++j) frag_a(0, j, p);
#pragma unroll
    for (int i = 0; i < TN; ++i) frag_b(0, i, p);
  }
  store_all(1);
  request_all(1, 3);
#pragma unroll
  for (int s = 0; s < 6; ++s) split_step(0, 0, s);
  request_one(0, 4, 0);
  // Stage kt & 1 is written, for step kt + 2, while step kt is multiplied, whose operands are in registers by then.  What is read,
  // stored and requested past the last step is not multiplied.
  constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
  constexpr int TT = TM * TN, NMF = 6 * TT;
  constexpr int BAR = TT == 4 ? 2 : 1;
  auto multiply = [&](auto par_c, int kt) {
    constexpr int PAR = decltype(par_c)::value;
    f32p_static_for([&](auto n_c) {
      constexpr int n = decltype(n_c)::value, q = n / TT, j = n % TT / TN, i = n % TN;
      floatx16& s = q == 5 ? acc[i][j] : cor[i][j];
      const bf16x8& x = PB[q] == 0 ? fb[PAR][i] : gb[PB[q] == 0 ? 0 : PB[q] - 1][i];
      const bf16x8& y = PA[q] == 0 ? fa[PAR][j] : ga[PA[q] == 0 ? 0 : PA[q] - 1][j];
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, s, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (n == BAR) __syncthreads();
      // operands of step kt + 1: the smaller pieces behind their last MFMA
      if (n >= TT && n < TT + TM) frag_a(kt + 1, n - TT, 2);
      if (n >= TT + TM && n < TT + TM + TN) frag_b(kt + 1, n - TT - TM, 0);
      if (n >= 2 * TT && n < 2 * TT + TN) frag_b(kt + 1, n - 2 * TT, 2);
      if (n >= 2 * TT + TN && n < 2 * TT + TN + TM) frag_a(kt + 1, n - 2 * TT - TN, 0);
      if (n >= 4 * TT && n < 4 * TT + TM) frag_a(kt + 1, n - 4 * TT, 1);
      if (n >= 5 * TT && n < 5 * TT + TN) frag_b(kt + 1, n - 5 * TT, 1);
      // vectors 1 .. 3 of step kt + 2, then the first of step kt + 3, which waits for the barrier: no store is young at a barrier
      if (n == BAR) write(kt, 0);
#pragma unroll
      for (int t = n * 24 / NMF; t < (n + 1) * 24 / NMF; ++t) {
        const int v = (t / 6 + 1) & 3, st = t % 6, set = v == 0 ? 1 - PAR : PAR;
        split_step(set, v, st);
        if (st == 5) {
          if (v != 0) write(kt, v);
          request_one(set, v == 0 ? kt + 5 : kt + 4, v);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }, std::make_integer_sequence<int, NMF>{});
  };
  typedef std::integral_constant<int, 0> p0_t;
  typedef std::integral_constant<int, 1> p1_t;
  for (int kt = 0; kt < nk; kt += 2) {
    multiply(p0_t{}, kt);
    multiply(p1_t{}, kt + 1);
  }
#pragma unroll
  for (int j = 0; j < TM; ++j)
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] += cor[i][j][e];
  if constexpr (KS > 1) {
    // the groups' sums meet in LDS and are added in group order
    __syncthreads();
    float* park = reinterpret_cast<float*>(lds) + (wave % WG) * (TT * 16 * 64) + lane;
    constexpr int GS = WG * TT * 16 * 64;
    if (grp > 0) {
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) park[(grp - 1) * GS + ((i * TM + j) * 16 + e) * 64] = acc[i][j][e];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 0; g < KS - 1; ++g)
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[i][j][e] += park[g * GS + ((i * TM + j) * 16 + e) * 64];
  }
  // A value that is not finite, or rounds to one, makes every sum that it is a term of not finite, but not always the same as its
  // products' own sum (Inf times a piece that is zero is NaN): such a tile is formed again from the values themselves.
  float t = 0.f;
#pragma unroll
  for (int j = 0; j < TM; ++j)
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) t = fmaf(acc[i][j][e], 0.f, t);
  if (__any(!(t == 0.f))) f32p_plain<A_KC, B_KC, TM, TN>(a, m0 + wm0, n0 + wn0, lane, acc);
#pragma unroll
  for (int j = 0; j < TM; ++j)
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const floatx4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        put(v, m0 + wm0 + j * 32 + (lane & 31), n0 + wn0 + i * 32 + 8 * g + 4 * (lane >> 5));
      }
}
template <bool A_KC, bool B_KC, int BT, int KS> constexpr size_t f32p_lds() {
  constexpr size_t kStages = 2 * (size_t)(F32PieceTile<A_KC, BT, KS>::BYTES + F32PieceTile<B_KC, BT, KS>::BYTES);
  static_assert(kStages >= (size_t)(KS - 1) * BT * BT * 4 && kStages <= (KS == 1 ? 80 : 160) * 1024, "LDS budget");
  return kStages;
}

// KS by tile, threads of a workgroup, ids resident at a time
template <int BT> constexpr int f32p_ks() { return BT == 128 ? 1 : 4; }
template <int BT> constexpr int f32p_threads() { return 2 * BT * f32p_ks<BT>(); }
template <int BT> __device__ __forceinline__ int f32p_order(int id, int total) { return f32p_xcd_order(id, total, BT == 128 ? 512 : 256); }

extern __shared__ __attribute__((aligned(16))) unsigned char lds_f32p[];

template <bool A_KC, bool B_KC, int EPI, int BT>
__global__ __launch_bounds__(f32p_threads<BT>(), 2) void gemm_f32_pieces_kernel(GemmArgs a) {
  f32p_tile<A_KC, B_KC, BT, f32p_ks<BT>()>(a, f32p_order<BT>(blockIdx.x, gridDim.x), lds_f32p,
                                           [&](const floatx4& v, int m, int n) { f32_put4<EPI>(a, v, m, n); });
}
template <int BT>
__global__ __launch_bounds__(f32p_threads<BT>(), 2) void gemm_f32_pieces_group_kernel(F32Group g) {
  GemmArgs a;
  const int tile = f32_group_at(g, f32p_order<BT>(blockIdx.x, gridDim.x), &a);
  f32p_tile<false, false, BT, f32p_ks<BT>()>(a, tile, lds_f32p, [&](const floatx4& v, int m, int n) { f32_put4<EPI_STORE>(a, v, m, n); });
}
// an input gradient, and column sums beside it (the workgroups behind the tiles)
template <int BT>
__global__ __launch_bounds__(f32p_threads<BT>(), 2) void gemm_f32_pieces_colsum_kernel(GemmArgs a, ColsumJob job, int tiles) {
  const int id = blockIdx.x;
  if (id < tiles)
    f32p_tile<true, true, BT, f32p_ks<BT>()>(a, f32p_order<BT>(id, tiles), lds_f32p,
                                             [&](const floatx4& v, int m, int n) { f32_put4<EPI_STORE>(a, v, m, n); });
  else colsum_block<float, f32p_threads<BT>()>(job, id - tiles, reinterpret_cast<float*>(lds_f32p));
}

static int f32p_tiles(const GemmArgs& a, int bt) { return ((a.M + bt - 1) / bt) * ((a.N + bt - 1) / bt); }

template <bool A_KC, bool B_KC, int EPI, int BT>
static hipError_t launch_f32p_bt(const GemmArgs& a, hipStream_t st) {
  constexpr size_t kLds = f32p_lds<A_KC, B_KC, BT, f32p_ks<BT>()>();
  auto kern = gemm_f32_pieces_kernel<A_KC, B_KC, EPI, BT>;
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(f32p_tiles(a, BT)), dim3(f32p_threads<BT>()), kLds, st, a);
  return hipGetLastError();
}
template <bool A_KC, bool B_KC, int EPI>
static hipError_t launch_f32p(const GemmArgs& a, int bt, hipStream_t st) {
  return bt == 128 ? launch_f32p_bt<A_KC, B_KC, EPI, 128>(a, st) : launch_f32p_bt<A_KC, B_KC, EPI, 64>(a, st);
}

hipError_t launch_f32_pieces(const GemmArgs& a, int bt, hipStream_t st) {
  if (a.a_kc && !a.b_kc) {
    switch (a.epi) {
      case EPI_STORE: return launch_f32p<true, false, EPI_STORE>(a, bt, st);
      case EPI_BIAS_GELU: return launch_f32p<true, false, EPI_BIAS_GELU>(a, bt, st);
      case EPI_DLOGITS: return launch_f32p<true, false, EPI_DLOGITS>(a, bt, st);
      default: return hipErrorInvalidValue;
    }
  }
  if (a.a_kc && a.b_kc) {
    switch (a.epi) {
      case EPI_STORE: return launch_f32p<true, true, EPI_STORE>(a, bt, st);
      case EPI_DGELU: return launch_f32p<true, true, EPI_DGELU>(a, bt, st);
      default: return hipErrorInvalidValue;
    }
  }
  if (!a.a_kc && !a.b_kc && a.epi == EPI_STORE) return launch_f32p<false, false, EPI_STORE>(a, bt, st);
  return hipErrorInvalidValue;
}

template <int BT>
static hipError_t launch_f32p_group_bt(const F32Group& g, int total, hipStream_t st) {
  constexpr size_t kLds = f32p_lds<false, false, BT, f32p_ks<BT>()>();
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)gemm_f32_pieces_group_kernel<BT>, (int)kLds); e != hipSuccess) return e;
  hipLaunchKernelGGL(gemm_f32_pieces_group_kernel<BT>, dim3(total), dim3(f32p_threads<BT>()), kLds, st, g);
  return hipGetLastError();
}
hipError_t launch_f32_pieces_group(const F32Group& g, int total, int bt, hipStream_t st) {
  return bt == 128 ? launch_f32p_group_bt<128>(g, total, st) : launch_f32p_group_bt<64>(g, total, st);
}

template <int BT>
static hipError_t launch_f32p_colsum_bt(const GemmArgs& a, const ColsumJob& j, hipStream_t st) {
  constexpr size_t kTile = f32p_lds<true, true, BT, f32p_ks<BT>()>();
  static_assert(colsum_lds_floats<float, f32p_threads<BT>()>() * sizeof(float) <= kTile, "LDS of the column sums");
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)gemm_f32_pieces_colsum_kernel<BT>, (int)kTile); e != hipSuccess) return e;
  const int tiles = f32p_tiles(a, BT);
  hipLaunchKernelGGL(gemm_f32_pieces_colsum_kernel<BT>, dim3(tiles + j.blocks), dim3(f32p_threads<BT>()), kTile, st, a, j, tiles);
  return hipGetLastError();
}
hipError_t launch_f32_pieces_colsum(const GemmArgs& a, const ColsumJob& j, int bt, hipStream_t st) {
  return bt == 128 ? launch_f32p_colsum_bt<128>(a, j, st) : launch_f32p_colsum_bt<64>(a, j, st);
}

}  // namespace mlm
