// Vocabulary-parallel input embedding of one shard (Section 3 of the paper: the embedding table is the output
// embedding's matrix E [H, v], split along the vocabulary; each shard contributes the rows of the ids it owns and
// zeros elsewhere, and the reduction g sums the partials).  E_r is stored [H, V_l] -- the layout the logits GEMM
// wants -- so a token's embedding is a COLUMN of E_r: H elements at stride V_l.  Both directions therefore walk the
// tokens in the order of their local id: consecutive waves touch neighbouring columns, which share cache lines, and
// the backward pass gets the tokens of one id as one contiguous, token-ordered segment (a deterministic sum with no
// atomics).  The order is a stable rank-sort computed by brute force (integer work, exact).
#include "common.h"
#include "rng.h"

namespace mlm {

// key[t] = local id if the token's id is in [v0, v0 + Vl), else Vl (sorts last); perm[rank(t)] = t with
// rank(t) = #{t' : key[t'] < key[t]} + #{t' < t : key[t'] == key[t]}.
// The T x T comparisons are split over blockIdx.y: block (x, y) counts, for its 256 tokens, the tokens t' of slice y
// that precede them, and writes the partial count; embed_scatter_kernel adds the slices' counts (integers: exact in
// any order) and scatters.  Keys are staged through LDS in chunks of 256 and compared four per LDS read.  A chunk other
// than the block's own lies wholly before or after its tokens, so ties there need no look at the index: two vector
// operations per comparison (8192 tokens: 31 -> 11 us with the index compared everywhere and 1024-token slices before).
constexpr int kRankChunk = 256;

__device__ __forceinline__ int embed_key(const int32_t* ids, int i, int v0, int Vl) {
  const int loc = ids[i] - v0;
  return (loc >= 0 && loc < Vl) ? loc : Vl;
}

__global__ __launch_bounds__(kRankChunk) void embed_rank_kernel(int T, int nslice, const int32_t* __restrict__ ids, int v0,
                                                                int Vl, int32_t* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) int32_t sk[kRankChunk];
  const int t0 = blockIdx.x * kRankChunk, t = t0 + threadIdx.x;
  const int my = t < T ? embed_key(ids, t, v0, Vl) : 0;
  // slice y covers chunks y, y + nslice, ... of kRankChunk tokens
  int rank = 0;
  for (int c0 = blockIdx.y * kRankChunk; c0 < T; c0 += nslice * kRankChunk) {
    __syncthreads();
    const int i0 = c0 + threadIdx.x;
    sk[threadIdx.x] = i0 < T ? embed_key(ids, i0, v0, Vl) : 0x7FFFFFFF;      // padding sorts after everything
    __syncthreads();
    if (c0 != t0) {
      const int lim = c0 < t0 ? my + 1 : my;          // tokens before t in index order win ties
#pragma unroll 8
      for (int i = 0; i < kRankChunk; i += 4) {
        const int4 k = *reinterpret_cast<const int4*>(&sk[i]);
        rank += k.x < lim ? 1 : 0;
        rank += k.y < lim ? 1 : 0;
        rank += k.z < lim ? 1 : 0;
        rank += k.w < lim ? 1 : 0;
      }
    } else {
#pragma unroll 8
      for (int i = 0; i < kRankChunk; ++i) rank += sk[i] < my + (i < (int)threadIdx.x ? 1 : 0) ? 1 : 0;
    }
  }
  if (t < T) partial[(size_t)blockIdx.y * T + t] = rank;
}

__global__ __launch_bounds__(256) void embed_scatter_kernel(int T, int nslice, const int32_t* __restrict__ partial,
                                                            int32_t* __restrict__ perm) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= T) return;
  int rank = 0;
  for (int y = 0; y < nslice; ++y) rank += partial[(size_t)y * T + t];
  perm[rank] = t;
}

// Gather and its gradient work on tiles of 64 sorted positions x 64 rows of E_r, transposed through LDS: on the E_r side a
// lane is a position, so a wave reads (or updates) 64 nearby columns of one row, and on the token side 16-byte vectors (or
// lanes) run along the row of the partial (or dz0).  With a wave per position and row group, 98304 workgroups at 8192 tokens
// x 3072 were bound by their launches and by 2-byte stores: 53 us forward and 65 us backward on one shard of eight, 26 and 23 now.
constexpr int kEmbTile = 64;
// (row stride of the LDS tile: an odd number of 32-bit words)
template <typename T> constexpr int emb_stride() { return kEmbTile + 4 / (int)sizeof(T); }

// out[t, :] = E_r[:, loc(t)], or zeros for a token outside the shard.  The positions of a tile that lie outside come last,
// so a tile whose first one does is all zeros.
template <typename T>
__global__ __launch_bounds__(256) void embed_fwd_kernel(int Tn, int H, int Vl, int v0, const int32_t* __restrict__ ids,
                                                        const int32_t* __restrict__ perm, const T* __restrict__ E,
                                                        T* __restrict__ out) {
  constexpr int S = emb_stride<T>(), VN = Vec16<T>::N, SEG = kEmbTile / VN;
  __shared__ __attribute__((aligned(16))) T tile[kEmbTile * S];
  __shared__ int stok[kEmbTile], sloc[kEmbTile];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k0 = blockIdx.x * kEmbTile, h0 = blockIdx.y * kEmbTile;
  if (threadIdx.x < kEmbTile) {
    const int k = k0 + lane, t = perm[min(k, Tn - 1)], loc = ids[t] - v0;
    stok[lane] = k < Tn ? t : -1;
    sloc[lane] = k < Tn && loc >= 0 && loc < Vl ? loc : -1;
  }
  __syncthreads();
  const bool some = sloc[0] >= 0;                     // block-uniform
  if (some) {
    const int loc = sloc[lane];
    T v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int h = h0 + wave * 16 + i;
      v[i] = loc >= 0 && h < H ? E[(size_t)h * Vl + loc] : from_f32<T>(0.f);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) tile[lane * S + wave * 16 + i] = v[i];
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < kEmbTile / (256 / SEG); ++i) {
    const int p = i * (256 / SEG) + threadIdx.x / SEG, c = (threadIdx.x % SEG) * VN;
    const int t = stok[p];
    if (t < 0 || h0 + c >= H) continue;               // H is a multiple of 8: a vector is all in or all out
    uint4 w = make_uint4(0u, 0u, 0u, 0u);
    if (some) {
      const uint32_t* src = reinterpret_cast<const uint32_t*>(&tile[p * S + c]);
      w = make_uint4(src[0], src[1], src[2], src[3]);
    }
    *reinterpret_cast<uint4*>(out + (size_t)t * H + h0 + c) = w;
  }
}

// dE_r[:, loc] += the sum of the rows of dz0 whose token has local id loc, in token order (fp32).  The wave whose 16
// positions hold the head of a run of equal ids sums all of it, sixteen rows at a time: their loads are in flight together (one
// row after the other, three dependent trips to memory each, 8192 equal tokens took 4.4 ms).
// Element-sized accesses to dE_r: neighbouring columns belong to other lanes and workgroups.  A workgroup takes NWV waves = 16 NWV
// positions x HR rows: 64 x 64, or 16 x 16 where that leaves compute units idle -- every lane of an access to dE_r may touch
// another line, and the lines of a few workgroups queue on their compute units (200 tokens x 320, 1024 columns: 7.9 us,
// 16 x 64 6.1, 16 x 16 5.1).
template <typename T, int NWV, int HR>
__global__ __launch_bounds__(64 * NWV) void embed_bwd_kernel(int Tn, int H, int Vl, int v0, const int32_t* __restrict__ ids,
                                                        const int32_t* __restrict__ perm, const T* __restrict__ dz,
                                                        T* __restrict__ dE) {
  constexpr int NP = 16 * NWV, RPL = HR * NP / (64 * NWV);         // positions; rows of dE per lane
  __shared__ float tile[NP * (HR + 1)];
  __shared__ int stok[NP + 1], sloc[NP + 2];          // sloc[i + 1]: position k0 + i, from the one before the tile to the one behind
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k0 = blockIdx.x * NP, h0 = blockIdx.y * HR, col = lane % HR, hc = min(h0 + col, H - 1);
  if (threadIdx.x <= NP + 1) {
    const int k = k0 + (int)threadIdx.x - 1;
    const int t = k >= 0 && k < Tn ? perm[k] : -1, loc = t >= 0 ? ids[t] - v0 : -1;
    sloc[threadIdx.x] = loc >= 0 && loc < Vl ? loc : -1;
    if (threadIdx.x > 0) stok[threadIdx.x - 1] = t;
  }
  __syncthreads();
  if (sloc[1] < 0) return;                            // sorted: the whole tile is outside the shard (block-uniform)
  const int p0 = __builtin_amdgcn_readfirstlane(wave) * 16;
  // lane i: local id of position p0 + i - 1 and token of position p0 + i; read back as scalars
  const int lloc = sloc[min(p0 + lane, NP + 1)], ltok = max(stok[min(p0 + lane, NP)], 0);
  float v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = to_f32(dz[(size_t)__builtin_amdgcn_readlane(ltok, i) * H + hc]);
  float acc = 0.f;
  int head = -1;                                      // position (in the tile) of the run being summed
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int prev = __builtin_amdgcn_readlane(lloc, i), loc = __builtin_amdgcn_readlane(lloc, i + 1);
    if (loc < 0 || loc != prev) {                     // a new run, or the end of the shard's tokens
      if (head >= 0) tile[head * (HR + 1) + col] = acc;
      head = loc >= 0 ? p0 + i : -1;
      acc = v[i];
    } else {
      acc += v[i];                                    // (of a run that an earlier wave sums: head is -1)
    }
  }
  if (head >= 0) {
    const int loc = __builtin_amdgcn_readlane(lloc, 16);
    // (most runs end inside the wave's positions)
    for (int kk = __builtin_amdgcn_readlane(lloc, 17) == loc ? k0 + p0 + 16 : Tn; kk < Tn; kk += 16) {
      const int k = kk + (lane & 15), tk = k < Tn ? perm[k] : -1;
      const bool same = tk >= 0 && ids[tk] - v0 == loc;
      // positions of the run among these sixteen: sorted, so the first n (wave-uniform)
      const int n = __builtin_ctz(~((uint32_t)__builtin_amdgcn_ballot_w64(same) & 0xFFFFu));
      if (n == 0) break;
      const int first = __builtin_amdgcn_readfirstlane(tk);      // (before the selection: every lane takes part)
      const int tok = same ? tk : first;
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = to_f32(dz[(size_t)__builtin_amdgcn_readlane(tok, i) * H + hc]);
#pragma unroll
      for (int i = 0; i < 16; ++i) acc = i < n ? acc + v[i] : acc;
      if (n < 16) break;
    }
    tile[head * (HR + 1) + col] = acc;
  }
  __syncthreads();
  const int p = threadIdx.x % NP, r0 = threadIdx.x / NP * RPL;       // this lane's position, the first of its rows
  const int loc = sloc[p + 1];
  if (loc < 0 || loc == sloc[p]) return;              // outside, or not the head of its run
  T was[RPL];                                         // (all read before the first is written)
#pragma unroll
  for (int i = 0; i < RPL; ++i) was[i] = dE[(size_t)min(h0 + r0 + i, H - 1) * Vl + loc];
#pragma unroll
  for (int i = 0; i < RPL; ++i) {
    const int r = r0 + i;
    if (h0 + r < H) dE[(size_t)(h0 + r) * Vl + loc] = from_f32<T>(to_f32(was[i]) + tile[p * (HR + 1) + r]);
  }
}

// dz0 = dropout-mask(dx0) / (1 - p); dpos[i, :] = sum over the batch of dz0[batch s + i, :].  One thread per
// (position, 16-byte vector); the batch is walked in order (deterministic).
template <typename T>
__global__ __launch_bounds__(256) void embed_bwd_replicated_kernel(int b, int s, int H, const T* dx0, T* dz0,
                                                                   T* __restrict__ dpos, DropArgs drop) {
  constexpr int VN = Vec16<T>::N;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;      // vector index inside the [s, H] block
  const size_t per = (size_t)s * H / VN;
  if (idx >= per) return;
  float acc[VN];
#pragma unroll
  for (int e = 0; e < VN; ++e) acc[e] = 0.f;
  for (int bi = 0; bi < b; ++bi) {
    const size_t off = ((size_t)bi * per + idx) * VN;
    Vec16<T> x, o;
    x.load(dx0 + off);
    float v[VN];
#pragma unroll
    for (int e = 0; e < VN; ++e) v[e] = x.get(e);
    if (drop.enabled) drop_apply<VN>(drop, off, v);
#pragma unroll
    for (int e = 0; e < VN; ++e) {
      o.set(e, v[e]);
      acc[e] += o.get(e);
    }
    if (dz0 != nullptr && (drop.enabled || dz0 != dx0)) o.store(dz0 + off);
  }
  if (dpos != nullptr) {
    Vec16<T> o;
#pragma unroll
    for (int e = 0; e < VN; ++e) o.set(e, acc[e]);
    o.store(dpos + idx * VN);
  }
}

// The rank partials ([nslice][T] int32) live in the partial output buffer until the gather overwrites it: a row of
// the partial has H elements, so up to H * sizeof(element) / 4 slices fit.
hipError_t launch_embed_fwd(int dtype, int T, int H, int Vl, int v0, const int32_t* ids, const void* E, int32_t* perm,
                            void* partial, hipStream_t st) {
  const int esz = dtype == MLM_BF16 ? 2 : 4;
  int nslice = (T + kRankChunk - 1) / kRankChunk;
  nslice = nslice < 1 ? 1 : (nslice > 16 ? 16 : nslice);
  if (nslice > H * esz / 4) nslice = H * esz / 4;
  hipLaunchKernelGGL(embed_rank_kernel, dim3((T + kRankChunk - 1) / kRankChunk, nslice), dim3(kRankChunk), 0, st, T, nslice, ids, v0, Vl,
                     (int32_t*)partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(embed_scatter_kernel, dim3((T + 255) / 256), dim3(256), 0, st, T, nslice, (const int32_t*)partial,
                     perm);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 grid((T + kEmbTile - 1) / kEmbTile, (H + kEmbTile - 1) / kEmbTile);
  if (dtype == MLM_BF16)
    hipLaunchKernelGGL((embed_fwd_kernel<bf16>), grid, dim3(256), 0, st, T, H, Vl, v0, ids, perm, (const bf16*)E,
                       (bf16*)partial);
  else
    hipLaunchKernelGGL((embed_fwd_kernel<float>), grid, dim3(256), 0, st, T, H, Vl, v0, ids, perm, (const float*)E,
                       (float*)partial);
  return hipGetLastError();
}

template <typename T>
static hipError_t embed_bwd_dispatch(int Tn, int H, int Vl, int v0, const int32_t* ids, const int32_t* perm, const T* dz, T* dE,
                                     hipStream_t st) {
  const dim3 large((Tn + 63) / 64, (H + 63) / 64), small((Tn + 15) / 16, (H + 15) / 16);
  if ((int)(large.x * large.y) < gemm_cu_count())
    hipLaunchKernelGGL((embed_bwd_kernel<T, 1, 16>), small, dim3(64), 0, st, Tn, H, Vl, v0, ids, perm, dz, dE);
  else
    hipLaunchKernelGGL((embed_bwd_kernel<T, 4, 64>), large, dim3(256), 0, st, Tn, H, Vl, v0, ids, perm, dz, dE);
  return hipGetLastError();
}

hipError_t launch_embed_bwd(int dtype, int T, int H, int Vl, int v0, const int32_t* ids, const int32_t* perm,
                            const void* dz, void* dE, hipStream_t st) {
  return dtype == MLM_BF16 ? embed_bwd_dispatch<bf16>(T, H, Vl, v0, ids, perm, (const bf16*)dz, (bf16*)dE, st)
                           : embed_bwd_dispatch<float>(T, H, Vl, v0, ids, perm, (const float*)dz, (float*)dE, st);
}

hipError_t launch_embed_bwd_replicated(int dtype, int b, int s, int H, const void* dx0, void* dz0, void* dpos,
                                       const mlm_dropout* drop, hipStream_t st) {
  const DropArgs da = make_drop_args(drop);
  if (dtype == MLM_BF16) {
    const size_t per = (size_t)s * H / 8;
    hipLaunchKernelGGL((embed_bwd_replicated_kernel<bf16>), dim3((unsigned)((per + 255) / 256)), dim3(256), 0, st, b, s,
                       H, (const bf16*)dx0, (bf16*)dz0, (bf16*)dpos, da);
  } else {
    const size_t per = (size_t)s * H / 4;
    hipLaunchKernelGGL((embed_bwd_replicated_kernel<float>), dim3((unsigned)((per + 255) / 256)), dim3(256), 0, st, b,
                       s, H, (const float*)dx0, (float*)dz0, (float*)dpos, da);
  }
  return hipGetLastError();
}

}  // namespace mlm
