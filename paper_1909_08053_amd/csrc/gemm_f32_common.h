// What the fp32 GEMM kernels (gemm_f32.hip, gemm_f32_pieces.hip) share: fused epilogues, operands read from memory, problems of a launch.
#pragma once
#include "common.h"

namespace mlm {

// Epilogue of one accumulator element.
struct F32Row { float coef, Mr, invS; int loc; };
template <int EPI>
__device__ __forceinline__ F32Row f32_row(const GemmArgs& a, int m) {
  F32Row r = {0.f, 0.f, 0.f, -1};
  if (EPI == EPI_DLOGITS) {
    r.coef = (a.loss_w ? a.loss_w[m] : 1.0f) / a.loss_stats[1];
    r.Mr = a.Mrow[m];
    r.invS = r.coef / a.Srow[m];
    r.loc = a.targets[m] - a.v0;
  }
  return r;
}
template <int EPI>
__device__ __forceinline__ void f32_put(const GemmArgs& a, const F32Row& r, int m, int n, float bias, float v) {
  float* C = (float*)a.C + (size_t)m * a.ldc + n;
  if (EPI == EPI_STORE) {
    *C = v + bias;
  } else if (EPI == EPI_BIAS_GELU) {
    v += bias;
    ((float*)a.aux)[(size_t)m * a.ldaux + n] = v;
    *C = gelu_fwd(v, a.gelu_tanh != 0);
  } else if (EPI == EPI_DGELU) {
    *C = v * gelu_bwd(((const float*)a.aux)[(size_t)m * a.ldaux + n], a.gelu_tanh != 0);
  } else if (EPI == EPI_DLOGITS) {
    float g = expf(v - r.Mr) * r.invS;
    if (n == r.loc) g -= r.coef;
    *C = g;
  }
}
// Four consecutive columns of row m.
template <int EPI>
__device__ __forceinline__ void f32_put4(const GemmArgs& a, const floatx4& acc, int m, int n) {
  if (m >= a.M || n >= a.N) return;                   // N is a multiple of 8: four columns are all in or all out
  float* C = (float*)a.C + (size_t)m * a.ldc + n;
  float v[4] = {acc[0], acc[1], acc[2], acc[3]};
  if ((EPI == EPI_STORE || EPI == EPI_BIAS_GELU) && a.bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += ((const float*)a.bias)[n + e];
  }
  if (EPI == EPI_BIAS_GELU) {
    *reinterpret_cast<float4*>((float*)a.aux + (size_t)m * a.ldaux + n) = make_float4(v[0], v[1], v[2], v[3]);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_fwd(v[e], a.gelu_tanh != 0);
  } else if (EPI == EPI_DGELU) {
    const float4 g = *reinterpret_cast<const float4*>((const float*)a.aux + (size_t)m * a.ldaux + n);
    const float gv[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= gelu_bwd(gv[e], a.gelu_tanh != 0);
  } else if (EPI == EPI_DLOGITS) {
    const F32Row r = f32_row<EPI>(a, m);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = expf(v[e] - r.Mr) * r.invS;
      if (n + e == r.loc) v[e] -= r.coef;
    }
  }
  *reinterpret_cast<float4*>(C) = make_float4(v[0], v[1], v[2], v[3]);
}

// (a k-contiguous operand has K a multiple of 8; K of the weight gradient counts tokens and can be any number: its last
// chunk is filled up with zeros)
template <bool KC>
__device__ __forceinline__ void f32_frag_global(const float* __restrict__ P, int ld, int row, int k, int K, float (&f)[4]) {
  if (KC) {
    const float4 v = *reinterpret_cast<const float4*>(P + (size_t)row * ld + k);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f[j] = P[(size_t)min(k + j, K - 1) * ld + row];
      f[j] = k + j < K ? f[j] : 0.f;
    }
  }
}

// The problems of a launch that holds several.
constexpr int kF32Group = 4;
struct F32Group {
  GemmArgs a[kF32Group];
  int tile_begin[kF32Group];           // first tile of each problem (past the grid for problems that do not exist)
};
__device__ __forceinline__ int f32_group_at(const F32Group& g, int id, GemmArgs* a) {      // the problem of tile id, and its number there
  int first = 0;
  *a = g.a[0];
#pragma unroll
  for (int q = 1; q < kF32Group; ++q)
    if (id >= g.tile_begin[q]) { *a = g.a[q]; first = g.tile_begin[q]; }     // workgroup-uniform
  return id - first;
}

// Products on the bf16 matrix cores (gemm_f32_pieces.hip), in tiles of bt x bt.  group: plain products with both operands k-major.
hipError_t launch_f32_pieces(const GemmArgs& a, int bt, hipStream_t st);
hipError_t launch_f32_pieces_group(const F32Group& g, int total, int bt, hipStream_t st);
hipError_t launch_f32_pieces_dual(const GemmArgs& w, const GemmArgs& x, hipStream_t st);       // in 64 x 64 tiles
hipError_t launch_f32_pieces_colsum(const GemmArgs& a, const ColsumJob& j, int bt, hipStream_t st);

}  // namespace mlm
