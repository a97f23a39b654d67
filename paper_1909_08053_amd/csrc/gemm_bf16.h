// Epilogue of the bf16 MFMA GEMM for gfx950 (MI355X): C[m,n] = sum_k A(m,k) B(k,n), fp32 accumulation; the main loop is in
// gemm_bf16_v2.h.
//   * The B tile is the MFMA "A" operand (rows = n) and the A tile its "B" operand (columns = m).  Each lane therefore
//     holds, for ONE output row m of a 16 x 16 tile, four consecutive columns: row reductions (softmax statistics of
//     the fused cross entropy) stay inside a lane plus two cross-lane exchanges, and results are packed 4 at a time.
//   * Every wave stages 32 x 64 strips through its own LDS region and writes full 16-byte vectors, rows contiguous
//     (coalesced HBM stores); bias, GeLU (+ saved pre-activation), GeLU', the dlogits formula and the cross-entropy
//     partials are applied on the fp32 accumulators.
#pragma once
#include "common.h"

namespace mlm {

template <int BM, int BN, int WAVES_M, int WAVES_N>
struct GemmTile {
  static constexpr int NT = WAVES_M * WAVES_N * 64;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  static constexpr int TM = WM / 32, TN = WN / 32;
  static constexpr int STRIP = 32 * 68 * 2;                        // bf16-sized elements of one epilogue strip (32 x 68 floats)
  static constexpr int NSTRIP = TM * ((TN + 1) / 2) > 1 ? 2 : 1;   // strips per wave (one if the wave tile is one strip)
  static constexpr size_t LDS_EPI = (size_t)NSTRIP * WAVES_M * WAVES_N * STRIP * 2 + (size_t)2 * WAVES_N * BM * 4;
};

// ---------------------------------------------------------------------------------------------- epilogue
// acc[i][j][e] holds row m = m0 + wm0 + 16 j + (lane & 15) and column n = n0 + wn0 + 16 i + 4 (lane >> 4) + e of the output
// tile.  Must be entered after a workgroup barrier that follows the last LDS read of the main loop (the LDS
// is reused: two staging strips per wave, then the cross-wave reduction area of the cross-entropy partials).

// Per-row softmax statistics of the logits tile (fused cross entropy): row max and sum of exp over the tile's
// columns, plus the target logit if the target column lies in this tile.  RAGGED: the tile hangs over column N.
// acc[i][j][e] holds row m = m0w + 16 j + (lane & 15) and column
// n = n0w + 16 i + 4 (lane >> 4) + e.  The four lanes l16, l16 + 16, l16 + 32, l16 + 48 share a row.
template <int NB, int NA, int WN, bool RAGGED>
__device__ __forceinline__ void ce_tile_stats(const GemmArgs& a, const floatx4 (&acc)[NB][NA], int m0w, int n0w,
                                              int lane, float* red_m_w, float* red_s_w) {
  const int l16 = lane & 15, lg = lane >> 4;
  const int nvalid = a.N - (n0w + 4 * lg);     // RAGGED: register column c (relative) is real iff c < nvalid
  // All rows' maxima first, then all rows' sums: the cross-lane exchanges of the NA rows are independent and overlap
  // (8 % fewer cycles than row by row; the function is bound by its vector arithmetic -- 128 values per lane, each a
  // max, a fused multiply-add, an exp2, an add and the target select: 7400 cycles per 256 x 256 tile, measured).
  float mx[NA], se[NA], tv[NA];
  int loc[NA];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int row = m0w + j * 16 + l16;
    // column of the target relative to this lane's registers (integer test), one select per value
    loc[j] = (row < a.M) ? a.targets[row] - a.v0 - (n0w + 4 * lg) : -1;
    mx[j] = -INFINITY;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = i * 16 + e;
        const float v = (RAGGED && c >= nvalid) ? -INFINITY : acc[i][j][e];
        mx[j] = fmaxf(mx[j], v);
      }
  }
#pragma unroll
  for (int j = 0; j < NA; ++j) mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 16, 64));
#pragma unroll
  for (int j = 0; j < NA; ++j) mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 32, 64));
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const float mxl = ce_base(mx[j]) * 1.4426950408889634f;
    se[j] = 0.f;
    tv[j] = 0.f;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = i * 16 + e;
        const float v = acc[i][j][e];
        const float p = __builtin_amdgcn_exp2f(fmaf(v, 1.4426950408889634f, -mxl));
        se[j] += (RAGGED && c >= nvalid) ? 0.f : p;
      }
  }
  // the target logit: only if some row of this wave has its target inside the wave's WN columns (one wave tile in
  // seven at a vocabulary of 51200 split eight ways), else the pass -- two operations per value -- is skipped
  bool mine = false;
#pragma unroll
  for (int j = 0; j < NA; ++j) mine = mine || (loc[j] >= 0 && loc[j] < WN);
  if (__builtin_amdgcn_ballot_w64(mine) != 0) {
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) tv[j] = (loc[j] == i * 16 + e) ? acc[i][j][e] : tv[j];
  }
#pragma unroll
  for (int j = 0; j < NA; ++j) se[j] += __shfl_xor(se[j], 16, 64);
#pragma unroll
  for (int j = 0; j < NA; ++j) se[j] += __shfl_xor(se[j], 32, 64);
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int row = m0w + j * 16 + l16;
    // the lane group that owns the column has bits 2 and 3 of (target - 4 lg) clear
    if (loc[j] >= 0 && loc[j] < WN && (loc[j] & 12) == 0 && (!RAGGED || loc[j] < nvalid)) a.t_out[row] = tv[j];
    if (lg == 0) {
      red_m_w[j * 16 + l16] = mx[j];
      red_s_w[j * 16 + l16] = se[j];
    }
  }
}

// Fill of one staging strip: rows 32 j .. 32 j + 31, columns 64 h .. 64 h + 63 of the wave tile; S = strip row stride in
// elements of T.
template <typename T> __device__ __forceinline__ void strip_put4(T* p, float v0, float v1, float v2, float v3);
template <> __device__ __forceinline__ void strip_put4<bf16>(bf16* p, float v0, float v1, float v2, float v3) {
  bf16x4 v;
  v[0] = (bf16)v0; v[1] = (bf16)v1; v[2] = (bf16)v2; v[3] = (bf16)v3;
  *reinterpret_cast<bf16x4*>(p) = v;
}
template <> __device__ __forceinline__ void strip_put4<float>(float* p, float v0, float v1, float v2, float v3) {
  *reinterpret_cast<float4*>(p) = make_float4(v0, v1, v2, v3);
}
template <typename T, int S, int NB, int NA>
__device__ __forceinline__ void acc_fill_strip(T* strip, const floatx4 (&acc)[NB][NA], int j, int h, int lane) {
  const int l16 = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int jl = 0; jl < 2; ++jl)
#pragma unroll
    for (int il = 0; il < 4; ++il) {
      if (4 * h + il >= NB) continue;
      const floatx4& t = acc[4 * h + il][2 * j + jl];
      strip_put4<T>(strip + (jl * 16 + l16) * S + il * 16 + 4 * lg, t[0], t[1], t[2], t[3]);
    }
}

// The saved pre-activations that a lane meets at read-back (EPI_DGELU), all requested at once.  Requested strip by strip, behind the
// strip's writes, every strip waited for memory: the pre-activations were written a forward pass ago.  Launches with GeLU', with the
// derivative in ten vector operations instead of fourteen: 3000 x 1536 x 1536 30.4 -> 26.8 us, 8192 x 768 x 1536 39.4 -> 36.5,
// 4096 x 2560 x 2560 71.7 -> 68.4, 8192 x 1536 x 3072 87.3 -> 86.5.
template <int BM, int BN, int WAVES_M, int WAVES_N>
struct EpilogueAux {
  typedef GemmTile<BM, BN, WAVES_M, WAVES_N> Tcfg;
  static constexpr int NH = (Tcfg::TN + 1) / 2;
  bf16x8 v[Tcfg::TM * NH][4];
  __device__ __forceinline__ void request(const GemmArgs& a, int m0, int n0) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = m0 + (wave / WAVES_N) * Tcfg::WM + (lane >> 3), n = n0 + (wave % WAVES_N) * Tcfg::WN + (lane & 7) * 8;
#pragma unroll
    for (int s = 0; s < Tcfg::TM * NH; ++s)
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int gm = min(m + s / NH * 32 + it * 8, a.M - 1), gn = min(n + s % NH * 64, a.N - 8);
        v[s][it] = *reinterpret_cast<const bf16x8*>((const bf16*)a.aux + (size_t)gm * a.ldaux + gn);
      }
  }
};

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, bool GELU_TANH, typename Acc>
__device__ __forceinline__ void gemm_epilogue_impl(const GemmArgs& a, Acc& acc, unsigned char* lds_raw, int m0, int n0, int tile_n,
                                                   const EpilogueAux<BM, BN, WAVES_M, WAVES_N>* aux) {
  typedef GemmTile<BM, BN, WAVES_M, WAVES_N> Tcfg;
  constexpr int NT = Tcfg::NT, TM = Tcfg::TM, TN = Tcfg::TN, WM = Tcfg::WM, WN = Tcfg::WN;
  bf16* lds = reinterpret_cast<bf16*>(lds_raw);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  bf16* C = (bf16*)a.C;
  const bf16* bias = (const bf16*)a.bias;

  if (EPI == EPI_CE) {
    float* red_m = reinterpret_cast<float*>(lds_raw + (size_t)Tcfg::NSTRIP * WAVES_M * WAVES_N * Tcfg::STRIP * 2);
    float* red_s = red_m + WAVES_N * BM;
    float* rm = red_m + (wave % WAVES_N) * BM + wm0;
    float* rs = red_s + (wave % WAVES_N) * BM + wm0;
    if (n0 + BN > a.N) ce_tile_stats<WN / 16, WM / 16, WN, true>(a, acc, m0 + wm0, n0 + wn0, lane, rm, rs);
    else ce_tile_stats<WN / 16, WM / 16, WN, false>(a, acc, m0 + wm0, n0 + wn0, lane, rm, rs);
    __syncthreads();
    for (int rloc = tid; rloc < BM; rloc += NT) {
      const int row = m0 + rloc;
      if (row < a.M) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < WAVES_N; ++w) M = fmaxf(M, red_m[w * BM + rloc]);
        const float base = ce_base(M);
        float S = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES_N; ++w) S += red_s[w * BM + rloc] * __expf(red_m[w * BM + rloc] - base);
        a.part_m[(size_t)tile_n * a.M + row] = M;
        a.part_s[(size_t)tile_n * a.M + row] = S;
      }
    }
    if (C == nullptr) return;
  }

  // ---- store passes.  The fp32 accumulators go through per-wave LDS strips of 32 rows x 64 columns (two strips,
  // software-pipelined: strip s+1 is written while strip s is read back).  All element-wise work happens at
  // read-back time, where a lane owns 8 consecutive columns of one row: bias, the saved pre-activation and the
  // outputs are then 16-byte accesses with 128-byte contiguous row segments.
  // (an odd TN leaves a last strip of 32 columns: half of the strip is then neither written nor read back)
  constexpr int NH = (TN + 1) / 2, NSTEP = TM * NH;
  const int rb_r = lane >> 3, rb_c = (lane & 7) * 8;           // read-back: 8 rows x 8 column groups per iteration
  const bool full = (m0 + BM <= a.M) && (n0 + BN <= a.N);
  if ((EPI == EPI_STORE || EPI == EPI_CE) && bias == nullptr) {
    // Nothing but the rounding happens between accumulator and memory: round first and stage bf16 strips (half the
    // LDS traffic of the fp32 strips, no conversion at read-back).  Row stride 72 elements keeps rows 16-byte aligned.
    constexpr int SWB = 72;
    static_assert(2 * 32 * SWB <= Tcfg::NSTRIP * Tcfg::STRIP * 2, "bf16 strips fit in the wave's staging area");
    bf16* bstrip0 = lds + (size_t)wave * Tcfg::NSTRIP * Tcfg::STRIP;
#pragma unroll
    for (int step = 0; step <= NSTEP; ++step) {
      if (step < NSTEP) {
        const int j = step / NH, h = step % NH;
        bf16* strip = bstrip0 + (step & 1) * (32 * SWB);
        acc_fill_strip<bf16, SWB>(strip, acc, j, h, lane);
      }
      __builtin_amdgcn_wave_barrier();
      if (step > 0) {
        const int ps = step - 1;
        const int j = ps / NH, h = ps % NH;
        const bf16* strip = bstrip0 + (ps & 1) * (32 * SWB);
        const int gn = n0 + wn0 + h * 64 + rb_c;
        const bool colv = (TN % 2 == 0) || (h * 64 + rb_c < WN);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int r = rb_r + it * 8;
          const int gm = m0 + wm0 + j * 32 + r;
          const bf16x8 o = *reinterpret_cast<const bf16x8*>(strip + r * SWB + rb_c);
          if (colv && (full || (gm < a.M && gn < a.N))) *reinterpret_cast<bf16x8*>(C + (size_t)gm * a.ldc + gn) = o;
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
  constexpr int SW = 64 + 4;                                   // strip row stride in floats (272 B)
  static_assert(32 * SW * 4 <= Tcfg::STRIP * 2, "strip does not fit");
  float* strip0 = reinterpret_cast<float*>(lds + (size_t)wave * Tcfg::NSTRIP * Tcfg::STRIP);

#pragma unroll
  for (int step = 0; step <= NSTEP; ++step) {
    if (step < NSTEP) {
      const int j = step / NH, h = step % NH;
      float* strip = strip0 + (step & 1) * (Tcfg::STRIP / 2);
      acc_fill_strip<float, SW>(strip, acc, j, h, lane);
    }
    __builtin_amdgcn_wave_barrier();
    if (step > 0) {
      const int ps = step - 1;
      const int j = ps / NH, h = ps % NH;
      const float* strip = strip0 + (ps & 1) * (Tcfg::STRIP / 2);
      const int gn = n0 + wn0 + h * 64 + rb_c;                 // first of this lane's 8 columns
      const bool colv = (TN % 2 == 0) || (h * 64 + rb_c < WN);
      const int gnc = min(gn, a.N - 8);
      float bvals[8];
      if ((EPI == EPI_STORE || EPI == EPI_BIAS_GELU) && bias != nullptr) {
        const bf16x8 b8 = *reinterpret_cast<const bf16x8*>(bias + gnc);
#pragma unroll
        for (int e = 0; e < 8; ++e) bvals[e] = (float)b8[e];
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) bvals[e] = 0.f;
      }
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int r = rb_r + it * 8;
        const int gm = m0 + wm0 + j * 32 + r;
        const int gmc = min(gm, a.M - 1);
        const float4 lo = *reinterpret_cast<const float4*>(strip + r * SW + rb_c);
        const float4 hi = *reinterpret_cast<const float4*>(strip + r * SW + rb_c + 4);
        float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        const bool ok = colv && (full || (gm < a.M && gn < a.N));
        bf16x8 o;
        if (EPI == EPI_STORE || EPI == EPI_CE) {
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (bf16)(v[e] + bvals[e]);
        } else if (EPI == EPI_BIAS_GELU) {
          bf16x8 pre;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = v[e] + bvals[e];
            pre[e] = (bf16)x;
            o[e] = (bf16)gelu_fwd(x, GELU_TANH);
          }
          if (ok) *reinterpret_cast<bf16x8*>((bf16*)a.aux + (size_t)gm * a.ldaux + gn) = pre;
        } else if (EPI == EPI_DGELU) {
          const bf16x8 g8 = aux->v[ps][it];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (bf16)(v[e] * gelu_bwd((float)g8[e], GELU_TANH));
        } else if (EPI == EPI_DLOGITS) {
          const float coef = (a.loss_w ? a.loss_w[gmc] : 1.0f) / a.loss_stats[1];
          const float Mrl = a.Mrow[gmc] * 1.4426950408889634f;
          const float invS = coef / a.Srow[gmc];
          const int loc = a.targets[gmc] - a.v0 - gn;           // target column relative to this lane's first column
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float pz = __builtin_amdgcn_exp2f(fmaf(v[e], 1.4426950408889634f, -Mrl)) * invS;
            if (loc == e) pz -= coef;
            o[e] = (bf16)pz;
          }
        }
        if (ok) *reinterpret_cast<bf16x8*>(C + (size_t)gm * a.ldc + gn) = o;
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// acc: floatx4 [BN / WAVES_N / 16][BM / WAVES_M / 16]
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, typename Acc>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, Acc& acc, unsigned char* lds_raw, int m0, int n0, int tile_n,
                                              const EpilogueAux<BM, BN, WAVES_M, WAVES_N>* aux) {
  if (EPI == EPI_BIAS_GELU || EPI == EPI_DGELU) {
    // the GeLU form is a launch-wide constant: branch once, not per element
    if (a.gelu_tanh) gemm_epilogue_impl<BM, BN, WAVES_M, WAVES_N, EPI, true>(a, acc, lds_raw, m0, n0, tile_n, aux);
    else gemm_epilogue_impl<BM, BN, WAVES_M, WAVES_N, EPI, false>(a, acc, lds_raw, m0, n0, tile_n, aux);
  } else {
    gemm_epilogue_impl<BM, BN, WAVES_M, WAVES_N, EPI, true>(a, acc, lds_raw, m0, n0, tile_n, aux);
  }
}

}  // namespace mlm
