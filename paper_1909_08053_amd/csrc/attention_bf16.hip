// bf16 MFMA attention over a shard's local heads (gfx950): forward with a streaming softmax, and a
// backward (dQ per query block; dK/dV per key block; in one launch or two, attn_bwd_mode) that recomputes the probabilities from
// the saved log-sum-exp.  Nothing of size s x s touches HBM and no atomics are used, so results are
// deterministic.
//
// Layout trick shared by the three kernels: score tiles are computed TRANSPOSED relative to the row that a
// wave owns, so that v_mfma_f32_32x32x16_bf16 leaves, in every lane, 16 score values that all belong to ONE
// owned row (a query in forward / dQ, a key in dK/dV).  Row statistics (max, sum, lse, delta) are then
// per-lane scalars (plus one cross-half shuffle), and the probability registers are already in the operand
// layout of the second MFMA (k index = the other sequence axis) -- P never goes through LDS.  The streamed
// tiles (K, V, Q, dO) are copied HBM -> LDS asynchronously, several tiles ahead, and an operand that must be read
// with k along the sequence axis is fetched from the same LDS tile with the transposing read instruction.
//
// Mask: allowed(i, j) = (j < key_len[b]) && (!causal || j <= i); excluded entries get probability exactly 0.
//
// Dropout of the probabilities (DROP instantiations): the forward kernel draws the keep decision of element
// ((batch, head, i), j) from the counter-based generator -- a lane's 16 scores of a 32-key half tile are four runs of
// four consecutive keys, i.e. four generator blocks -- zeroes the dropped probabilities before the second MFMA, folds
// 1 / (1 - p) into the final normalisation and saves the decisions as one bit per key.  The row sum and the
// log-sum-exp stay those of the undropped scores.  The backward kernels read the saved bits instead of running the
// generator again: dQ loads its query row's two words per tile, dK/dV gets the tile's 64 x 128-bit block through the
// DMA ring.  delta = rowsum(dO o O) needs no change: O already contains the dropout.
#include "attention_modes.h"
#include "lds_dma.h"
#include "rng.h"

namespace mlm {

constexpr int ATILE = 64;           // rows of the streamed tile (keys in fwd/dQ, queries in dK/dV)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

constexpr int ANW = 4;              // waves per workgroup: 32 owned rows each
constexpr int ANT = ANW * 64;

// Workgroup id -> (block along the sequence, local head, batch).  Workgroups are handed to the eight XCDs round-robin
// by id and every XCD has its own L2, so the (batch, head) index takes the low three bits of the id: all sequence
// blocks of one (batch, head) pair -- they stream the same K / V (or Q / dO) rows -- run on ONE XCD and re-read those
// rows from its L2 (x-fastest ids put the eight blocks of a pair on eight XCDs and every XCD fetched every pair).
// Within an XCD the ids keep the sequence block as the faster index, so the longest causal blocks still start first.
// Grid: attn_grid(nx, hl, b) workgroups in x; ids whose pair does not exist (hl b not a multiple of 8) exit at once.
struct AttnBlock { int xb, hd, bi; bool valid; };
__device__ __forceinline__ AttnBlock attn_block(int nx, int hl, int b) {
  const int id = blockIdx.x, r = id >> 3;
  const int bh = (r / nx) * 8 + (id & 7);
  AttnBlock o;
  o.xb = r % nx;
  o.valid = bh < hl * b;
  o.hd = bh % hl;
  o.bi = bh / hl;
  return o;
}
static inline dim3 attn_grid(int nx, int hl, int b) { return dim3(8 * nx * ((hl * b + 7) / 8)); }

__device__ __forceinline__ bf16x8 pack8(const floatx16& v, int off) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16)v[off + e];
  return r;
}

// ---- streamed [64][D] bf16 tiles copied HBM -> LDS by the DMA path -------------------------------------------
// A tile is 64 rows of U = D/8 16-byte units, stored densely (the copy writes 1 KB per wave instruction in lane
// order) with the unit index XOR-swizzled per row, so that both kinds of operand read are bank-conflict free:
//   * "kc" fragments (contraction along D: 16 lanes read one 16-byte unit of 16 consecutive rows), and
//   * transposing reads (contraction along the tile's rows: 32 lanes read 64 bytes of 4 consecutive rows).
template <int D>
struct ATile {
  static constexpr int U = D / 8;
  static constexpr int BYTES = ATILE * D * 2;
  static constexpr int QPW = U / ANW;              // 1-KB copies per wave and tile
  static_assert(U % ANW == 0 && (U == 8 || U == 12 || U == 16 || U == 24), "head size");
  __device__ static __forceinline__ int sw(int row) {
    if (U == 16) return ((row & 3) << 2) | ((row >> 2) & 3);
    if (U == 12) return (row >> 2) & 3;
    return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);   // U = 8 and U = 24: the row stride is 8 units mod 16
  }
  // operand with k along D: 8 consecutive elements [16 ks + 8 lh, +8) of row r0 + l32
  __device__ static __forceinline__ bf16x8 frag_kc(const unsigned char* tile, int r0, int ks, int lane) {
    const int row = r0 + (lane & 31), c = 2 * ks + (lane >> 5);
    return *reinterpret_cast<const bf16x8*>(tile + row * (U * 16) + ((c ^ sw(row)) << 4));
  }
  // operand with k along the tile's rows, for column d0 + l32: k-slot (lh, e) <-> row 16 c4 + 8 (e/4) + 4 lh + e%4,
  // which is how a transposed score accumulator lays out its rows
  __device__ static __forceinline__ bf16x8 frag_tr(const unsigned char* tile, int c4, int d0, int lane) {
    const int g = lane >> 4, j = lane & 15;
    const int col = d0 + 16 * (g & 1) + 4 * (j & 3);
    const int cu = col >> 3, half = (col >> 2) & 1;
    v4s_t h[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int row = 16 * c4 + 4 * (g >> 1) + 8 * r + (j >> 2);
      h[r] = lds_read_tr16(tile + row * (U * 16) + ((cu ^ sw(row)) << 4) + half * 8);
    }
    const v8s_t v = __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
};

// Which 16 bytes of a tile each lane copies (fixed per lane), and the copy of one tile.  After REP copies of a wave the lane is
// STEP rows further down at the same unit but for the swizzle, which differs in one bit (FLIP elements): a row and a column per
// copy would be up to 12 registers of kernels that have none left.
template <int D>
struct ATileSrc {
  typedef ATile<D> TL;
  static constexpr int REP = TL::U % 12 == 0 ? 3 : 1, STEP = 64 * REP / TL::U, FLIP = TL::U == 16 ? 8 : 16;
  static_assert(TL::QPW <= (TL::U == 16 ? 4 : 2) * REP, "one bit of the swizzle (two at 16 units)");
  int row[REP], col[REP];
  __device__ __forceinline__ void init(int wave, int lane) {
#pragma unroll
    for (int i = 0; i < REP; ++i) {
      const int u = 64 * (wave * TL::QPW + i) + lane;
      row[i] = u / TL::U;
      col[i] = ((u % TL::U) ^ TL::sw(row[i])) * 8;
    }
  }
  // P: element (0, 0) of the streamed matrix (row stride ld); rows beyond nrows - 1 re-read the last row (callers mask)
  __device__ __forceinline__ void issue_one(const bf16* P, int ld, int row0, int nrows, uint32_t lds_tile, int wave_u, int i) const {
    dma16(P + (size_t)min(row0 + row[i % REP] + i / REP * STEP, nrows - 1) * ld + (col[i % REP] ^ (i / REP * FLIP)),
          lds_tile + (wave_u * TL::QPW + i) * 1024);
  }
  __device__ __forceinline__ void issue(const bf16* P, int ld, int row0, int nrows, uint32_t lds_tile, int wave_u) const {
#pragma unroll
    for (int i = 0; i < TL::QPW; ++i) issue_one(P, ld, row0, nrows, lds_tile, wave_u, i);
  }
};

// ------------------------------------------------------------------------------------------ forward
// Workgroup = 128 queries of one (batch, head), 4 waves of 32 queries.  K and V tiles of 64 keys stream through a
// three-stage LDS ring filled by DMA two tiles ahead; per tile: S^T = K Q^T (12 MFMAs at d = 96), online softmax in
// registers, O^T += V^T P^T with V read through the transposing LDS loads (12 MFMAs).  One barrier per tile.
// How the waves of a forward / dQ workgroup divide its rows and the streamed tiles: RW waves along the rows (32 each), KG
// waves along the 64 keys of a tile, NG groups of RW x KG = 4 waves that take every NG-th tile through a DMA ring of their
// own.  The partial results of the KG NG waves that own the same rows are merged through LDS at the end.
//   WIDE  (4 x 1 x 1): no merge, and two workgroups fit a compute unit (d <= 128), so that one's first copies and last
//         stores run under the other's steps.
//   PAIR  (4 x 1 x 2): halves the serial chain of the longest (causal) blocks and puts two waves on every SIMD where a
//         compute unit has one workgroup.  d = 192 has no LDS for the second ring.
//   SPLIT (2 x 2 x NG): 64 rows per workgroup, for launches that leave compute units without one; each wave multiplies
//         half of a tile.
// (attention_modes.h holds the rule and the figures)
template <int D, int MODE> struct AttnSplit {
  static constexpr int RW = MODE == ATTN_SPLIT ? 2 : 4, KG = ANW / RW;
  static constexpr int NG = MODE == ATTN_WIDE || D > 128 ? 1 : 2;
  static constexpr int NST = D == 128 ? 2 : 3;                       // ring stages per group (LDS budget)
  static constexpr int NT = NG * ANT, G = KG * NG;                   // threads; waves that share a row
  static constexpr int MINW = NG == 2 || (MODE == ATTN_WIDE && D <= 128) ? 2 : 1;   // waves per SIMD the registers must allow
  static constexpr size_t RING = (size_t)NG * NST * 2 * ATILE * D * 2;
  static constexpr size_t PARK = (size_t)(G - 1) * RW * (D / 2 + 2) * 64 * 4;
  static constexpr size_t LDS = RING > PARK ? RING : PARK;
  static_assert(LDS <= 160 * 1024, "LDS budget");
};
template <int D> constexpr int dkv_dsplit() { return D >= 128 ? 2 : 1; }
// dK/dV: two wave groups (alternate query tiles, merged through LDS at the end) for the head sizes whose registers
// allow two waves per SIMD once the wave's own K / V rows are kept in LDS instead of registers; ring stages per group
// by the LDS budget (rings + the 128 owned K and V rows).
template <int D> constexpr int dkv_groups() { return D <= 128 ? 2 : 1; }
template <int D> constexpr int dkv_stages() { return (D == 96 || D == 128) ? 2 : 3; }
template <int D> constexpr bool dkv_own_lds() { return D <= 96; }    // d = 128: half the D columns per workgroup, rows stay in registers

// (two waves per SIMD requested: with at most 256 registers per lane the MFMA accumulators live in ordinary VGPRs, so
// the softmax arithmetic needs no accumulator-register moves)
template <int D, bool DROP, int MODE, bool FOLD>
__global__ __launch_bounds__((AttnSplit<D, MODE>::NT), (AttnSplit<D, MODE>::MINW)) void attn_fwd_bf16_kernel(AttnArgs a) {
  typedef ATile<D> TL;
  typedef AttnSplit<D, MODE> SP;
  constexpr int RW = SP::RW, KG = SP::KG, NK = 2 / KG;               // NK: 32-key halves of a tile per wave
  constexpr int BQ = 32 * RW, STAGE = 2 * TL::BYTES, LPT = 2 * TL::QPW;   // LPT: copies per tile and wave (K + V)
  constexpr int NST = SP::NST, NG = SP::NG;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  // wave-uniform values must be known as such: the mask test below is a scalar branch
  const int grp = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8);    // wave group: takes the tiles NG j + grp
  const int wave_u = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);   // wave inside its group (copies a quarter of a tile)
  // FOLD (attn_fwd_fold): the workgroup's rows are the x-th half block from the end and the x-th from the start, so that every workgroup
  // has the same number of tiles to multiply; the waves that share a SIMD, one of each group, have late and early rows.
  constexpr int CH = BQ / 2, RC = RW / 2;
  static_assert(!FOLD || NG == 2, "both groups of waves");
  const int wave = (wave_u % RW) ^ (FOLD ? RC * grp : 0), kh = wave_u / RW;  // its 32 queries, and its 32 keys of a tile (KG = 2)
  const int nqb = (a.s + BQ - 1) / BQ;
  const AttnBlock blk = attn_block(nqb, a.hl, a.b);
  if (!blk.valid) return;
  const int qb = nqb - 1 - blk.xb;                // longest (causal) blocks first
  const int hd = blk.hd, bi = blk.bi;
  const int ld = 3 * a.hl * D;
  const bf16* base = (const bf16*)a.qkv + (size_t)bi * a.s * ld;
  const int klen = attn_key_len(a.key_len, bi, a.s);
  const int late = (a.s + CH - 1) / CH - 1 - blk.xb;        // the half blocks are `late` and xb, of which there is one if they are the same
  const bool twice = FOLD && wave < RC && late == blk.xb;
  const int q_end = FOLD ? CH * (late + 1) : qb * BQ + BQ;
  const int qw0 = FOLD ? CH * (wave < RC ? blk.xb : late) + 32 * (wave % RC) : qb * BQ + wave * 32;
  const int qi = twice ? a.s : qw0 + l32;                   // (rows from s on are not stored)

  bf16x8 qf[D / 16];
  {
    const bf16* qrow = base + (size_t)min(qi, a.s - 1) * ld + hd * D;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16 + lh * 8);
  }
  floatx16 o[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
  float m = -INFINITY, lsum = 0.f;
  const size_t prow = ((size_t)bi * a.hl + hd) * a.s + min(qi, a.s - 1);   // row of the [b, hl, s, s] probabilities
  int kv_end = klen;
  if (a.causal) kv_end = min(kv_end, q_end);
  const int nt = (kv_end + ATILE - 1) / ATILE;
  const float sc = kLog2e / sqrtf((float)D);
  const bf16* Kb = base + (a.hl + hd) * D;
  const bf16* Vb = base + (2 * a.hl + hd) * D;
  ATileSrc<D> src;
  src.init(wave_u, lane);
  unsigned char* ring = lds_raw + grp * (NST * STAGE);   // this group's ring
  const uint32_t lds0 = lds_offset_of(ring);
  const int njt = (nt + NG - 1) / NG;              // steps: group g handles tile NG j + g in step j (if it exists)
  // The ring is always kept full: past the last tile the copies re-read tile nt - 1 into a stage nobody reads, so
  // the outstanding-copy count is the same in every iteration.
#pragma unroll
  for (int t = 0; t < NST - 1; ++t) {
    const int tc = min(NG * t + grp, nt - 1) * ATILE;
    src.issue(Kb, ld, tc, a.s, lds0 + t * STAGE, wave_u);
    src.issue(Vb, ld, tc, a.s, lds0 + t * STAGE + TL::BYTES, wave_u);
  }
  int stage = 0;
  for (int j = 0; j < njt; ++j) {
    const int t = NG * j + grp;
    const int k0 = t * ATILE, kw0 = k0 + (KG == 2 ? 32 * kh : 0);    // the tile's first key, this wave's first key
    wait_vmcnt<LPT*(NST - 2)>();                   // this wave's copies of step j have landed; step j + 1 may be in flight
    __builtin_amdgcn_s_barrier();                 // everyone's have; and everyone is done with step j - 1
    // The copies that re-arm the stage of step j - 1 (= stage of step j + NST - 1) are NOT issued here in one burst:
    // all eight waves leave the barrier together, 48 one-KB copies queue in the CU's address unit and every wave sits
    // in front of its first fragment read for 0.6 us of a 2-us step (in-kernel timestamps).  They are issued one at
    // a time between the exponentials below, where the wave has no LDS read in flight that the copy's compiler-level
    // memory barrier would pin (placed behind the MFMAs of the two products instead, it measured no gain: 24.9 against
    // 23.5 us).  Head sizes above 96 keep the burst: the longer live ranges cost them registers they do not have.
    const int pst = stage == 0 ? NST - 1 : stage - 1;
    const int tc_next = min(t + NG * (NST - 1), nt - 1) * ATILE;
    const uint32_t dstK = lds0 + pst * STAGE, dstV = dstK + TL::BYTES;
    const unsigned char* sK = ring + stage * STAGE;
    const unsigned char* sV = sK + TL::BYTES;
    stage = stage == NST - 1 ? 0 : stage + 1;
    constexpr bool SPREAD = D <= 96;
    // else: no such tile / all padding / entirely above this wave's diagonal (wave-uniform); key kw0 of a live tile is
    // allowed for every query of the wave
    const bool live = t < nt && kw0 < klen && !(a.causal && kw0 > qw0 + 31) && !twice;
    if (!SPREAD || !live) {
      src.issue(Kb, ld, tc_next, a.s, dstK, wave_u);
      src.issue(Vb, ld, tc_next, a.s, dstV, wave_u);
    }
    if (!live) continue;
    floatx16 sacc[NK];
    float lsum_t = 0.f;
#pragma unroll
    for (int kt = 0; kt < NK; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[kt][e] = 0.f;
    // the two 32-key halves are independent accumulation chains: alternate them so that a dependent MFMA never
    // follows its predecessor directly
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
      for (int kt = 0; kt < NK; ++kt)
        sacc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_kc(sK, (KG == 2 ? kh : kt) * 32, ks, lane), qf[ks], sacc[kt], 0, 0, 0);
    // raw scores s; probabilities p = exp2(s * sc - max) with the scale folded into one fma per element
    const bool need_mask = (a.causal && kw0 + 32 * NK - 1 > qw0) || (kw0 + 32 * NK > klen);   // wave-uniform
    float mt = -INFINITY;
    if (need_mask) {
#pragma unroll
      for (int kt = 0; kt < NK; ++kt)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = kw0 + kt * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
          const bool off = key >= klen || (a.causal && key > qi);
          sacc[kt][e] = off ? -INFINITY : sacc[kt][e];
          mt = fmaxf(mt, sacc[kt][e]);
        }
    } else {
#pragma unroll
      for (int kt = 0; kt < NK; ++kt)
#pragma unroll
        for (int e = 0; e < 16; ++e) mt = fmaxf(mt, sacc[kt][e]);
    }
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64)) * sc;
    const float mn = fmaxf(m, mt);               // finite from the first tile on: key 0 is allowed for every query
#pragma unroll
    for (int kt = 0; kt < NK; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[kt][e], sc, -mn));
        sacc[kt][e] = p;
        lsum_t += p;
        if (SPREAD) {
#pragma unroll
          for (int c = 0; c < LPT; ++c)                    // copy c after element (16 NK c + 8 NK) / LPT of the 16 NK
            if (kt * 16 + e == (16 * NK * c + 8 * NK) / LPT) {
              if (c < TL::QPW) src.issue_one(Kb, ld, tc_next, a.s, dstK, wave_u, c);
              else src.issue_one(Vb, ld, tc_next, a.s, dstV, wave_u, c - TL::QPW);
            }
        }
      }
    // rescale the running sums only when some row's maximum moved (wave-uniform test)
    if (__builtin_amdgcn_ballot_w64(mn > m) != 0) {
      const float corr = __builtin_amdgcn_exp2f(m - mn);
      lsum *= corr;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] *= corr;
      m = mn;
    }
    lsum += lsum_t;
    if (DROP) {
#pragma unroll
      for (int kt = 0; kt < NK; ++kt) {
        uint32_t word = 0;                       // this lane's 16 of the 32 keep bits of keys kw0 + 32 kt ..
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const uint32_t k4 = drop_keep4(a.drop, (prow * a.s + kw0 + kt * 32 + 8 * g + 4 * lh) >> 2);
#pragma unroll
          for (int e = 0; e < 4; ++e) sacc[kt][4 * g + e] = ((k4 >> e) & 1u) ? sacc[kt][4 * g + e] : 0.f;
          word |= k4 << (8 * g + 4 * lh);
        }
        word |= __shfl_xor(word, 32, 64);        // the other half-wave holds the other 16 bits
        if (lh == kt && qi < a.s) a.keep_bits[prow * a.keep_pitch + (kw0 >> 5) + kt] = word;
      }
    }
#pragma unroll
    for (int c = 0; c < 2 * NK; ++c) {
      const bf16x8 pf = pack8(sacc[c >> 1], 8 * (c & 1));
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_tr(sV, (KG == 2 ? 2 * kh : 0) + c, dt * 32, lane), pf, o[dt], 0, 0, 0);
    }
  }
  wait_vmcnt<0>();                                // copies still in flight target this workgroup's LDS
  // merge the (m, l, O) of the waves that own the same rows: all but the first park theirs in LDS ([value][lane] per wave:
  // conflict-free)
  if (SP::G > 1) {
    __syncthreads();
    constexpr int NR = D / 2 + 2;
    const int part = kh + KG * grp;
    float* park = reinterpret_cast<float*>(lds_raw) + (size_t)wave * NR * 64 + lane;
    constexpr int PSTEP = RW * NR * 64;
    if (part > 0) {
      float* dst = park + (part - 1) * PSTEP;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) dst[(dt * 16 + e) * 64] = o[dt][e];
      dst[(D / 2) * 64] = m;
      dst[(D / 2 + 1) * 64] = lsum;
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int p = 0; p < SP::G - 1; ++p, park += PSTEP) {
      const float m1 = park[(D / 2) * 64], l1 = park[(D / 2 + 1) * 64];
      const float mn = fmaxf(m, m1);              // part 0 always has key 0: finite
      const float c0 = __builtin_amdgcn_exp2f(m - mn), c1 = __builtin_amdgcn_exp2f(m1 - mn);
      lsum = lsum * c0 + l1 * c1;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] = o[dt][e] * c0 + park[(dt * 16 + e) * 64] * c1;
      m = mn;
    }
  }
  lsum += __shfl_xor(lsum, 32, 64);
  if (qi < a.s) {
    const float inv = (DROP ? a.drop.scale : 1.0f) / lsum;
    bf16* crow = (bf16*)a.ctx + ((size_t)bi * a.s + qi) * (a.hl * D) + hd * D;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = (bf16)(o[dt][4 * g + e] * inv);
        *reinterpret_cast<bf16x4*>(crow + dt * 32 + 8 * g + 4 * lh) = ov;
      }
    if (lh == 0) a.lse[((size_t)bi * a.hl + hd) * a.s + qi] = (m + log2f(lsum)) * kLn2;
  }
}

// ------------------------------------------------------------------------------------------ backward: dQ
// Same streaming structure as the forward kernel.  Per tile: S^T = K Q^T and dP^T = V dO^T (contraction along D),
// P = exp2(S sc - lse), dS = P o (dP - delta), dQ^T += K^T dS^T with K read a second time through the transposing
// loads.  As a kernel of its own it forms delta_i = sum_d dO_id O_id from the rows that the lanes hold anyway and stores it, with the
// log-sum-exp in log2 units, for the dK/dV kernel, which runs after it.
// MERGED: part of the joint kernel below; attn_delta_bf16_kernel has stored both.
template <int D, bool DROP, int MODE, bool MERGED>
__device__ __forceinline__ void attn_bwd_dq_block(const AttnArgs a, const AttnBlock blk) {
  typedef ATile<D> TL;
  typedef AttnSplit<D, MODE> SP;
  constexpr int RW = SP::RW, KG = SP::KG, NK = 2 / KG;
  constexpr int BQ = 32 * RW, STAGE = 2 * TL::BYTES, LPT = 2 * TL::QPW, NST = SP::NST, NG = SP::NG;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int grp = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8);   // wave group: takes the tiles NG j + grp
  const int wave_u = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);   // wave inside its group (uniform: scalar mask branches)
  const int wave = wave_u % RW, kh = wave_u / RW;  // its 32 queries, and its 32 keys of a tile (KG = 2)
  const int part = kh + KG * grp;
  const int nqb = (a.s + BQ - 1) / BQ;
  const int qb = nqb - 1 - blk.xb;
  const int hd = blk.hd, bi = blk.bi;
  const int ld = 3 * a.hl * D;
  const bf16* base = (const bf16*)a.qkv + (size_t)bi * a.s * ld;
  const int klen = attn_key_len(a.key_len, bi, a.s);
  const int q0 = qb * BQ, qw0 = q0 + wave * 32, qi = qw0 + l32;
  const int qc = min(qi, a.s - 1);

  const size_t vrow = ((size_t)bi * a.hl + hd) * a.s;           // of the [b, hl, s] vectors
  bf16x8 qf[D / 16], dof[D / 16];
  float dl = MERGED ? a.delta[vrow + qc] : 0.f;
  {
    const bf16* qrow = base + (size_t)qc * ld + hd * D;
    const bf16* drow = (const bf16*)a.dctx + ((size_t)bi * a.s + qc) * (a.hl * D) + hd * D;
    const bf16* orow = (const bf16*)a.ctx + ((size_t)bi * a.s + qc) * (a.hl * D) + hd * D;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      qf[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16 + lh * 8);
      dof[ks] = *reinterpret_cast<const bf16x8*>(drow + ks * 16 + lh * 8);
      if (MERGED) continue;
      const bf16x8 of = *reinterpret_cast<const bf16x8*>(orow + ks * 16 + lh * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) dl = fmaf((float)dof[ks][e], (float)of[e], dl);
    }
    if (!MERGED) dl += __shfl_xor(dl, 32, 64);
  }
  const float lse2 = a.lse[vrow + qc] * kLog2e;
  const uint32_t* kbrow = DROP ? a.keep_bits + (((size_t)bi * a.hl + hd) * a.s + qc) * a.keep_pitch : nullptr;
  if (!MERGED && part == 0 && lh == 0 && qi < a.s) {   // for the dK/dV kernel: [0] delta, [1] log-sum-exp in log2 units
    a.delta[vrow + qi] = dl;
    a.delta[(size_t)a.b * a.hl * a.s + vrow + qi] = lse2;
  }
  floatx16 dq[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[dt][e] = 0.f;
  int kv_end = klen;
  if (a.causal) kv_end = min(kv_end, q0 + BQ);
  const int nt = (kv_end + ATILE - 1) / ATILE;
  const float scale = 1.0f / sqrtf((float)D);
  const float sc = kLog2e * scale;
  const bf16* Kb = base + (a.hl + hd) * D;
  const bf16* Vb = base + (2 * a.hl + hd) * D;
  ATileSrc<D> src;
  src.init(wave_u, lane);
  unsigned char* ring = lds_raw + grp * (NST * STAGE);
  const uint32_t lds0 = lds_offset_of(ring);
  const int njt = (nt + NG - 1) / NG;
#pragma unroll
  for (int t = 0; t < NST - 1; ++t) {
    const int tc = min(NG * t + grp, nt - 1) * ATILE;
    src.issue(Kb, ld, tc, a.s, lds0 + t * STAGE, wave_u);
    src.issue(Vb, ld, tc, a.s, lds0 + t * STAGE + TL::BYTES, wave_u);
  }
  int stage = 0;
  for (int j = 0; j < njt; ++j) {
    const int t = NG * j + grp;
    const int k0 = t * ATILE, kw0 = k0 + (KG == 2 ? 32 * kh : 0);
    wait_vmcnt<LPT*(NST - 2)>();
    __builtin_amdgcn_s_barrier();
    // the copies that re-arm the stage of step j - 1 are issued one at a time inside the element-wise pass below
    // (as in the forward kernel: a burst here holds every wave of the CU in front of its first fragment read)
    constexpr bool SPREAD = D <= 96;
    const int pst = stage == 0 ? NST - 1 : stage - 1;
    const int tc_next = min(t + NG * (NST - 1), nt - 1) * ATILE;
    const uint32_t dstK = lds0 + pst * STAGE, dstV = dstK + TL::BYTES;
    auto copy_after = [&](int el) {                  // el: element index 0 .. 16 NK - 1 of the pass (compile time after unrolling)
#pragma unroll
      for (int c = 0; c < LPT; ++c)
        if (el == (16 * NK * c + 8 * NK) / LPT) {
          if (c < TL::QPW) src.issue_one(Kb, ld, tc_next, a.s, dstK, wave_u, c);
          else src.issue_one(Vb, ld, tc_next, a.s, dstV, wave_u, c - TL::QPW);
        }
    };
    const unsigned char* sK = ring + stage * STAGE;
    const unsigned char* sV = sK + TL::BYTES;
    stage = stage == NST - 1 ? 0 : stage + 1;
    const bool live = t < nt && kw0 < klen && !(a.causal && kw0 > qw0 + 31);
    if (!SPREAD || !live) {
      src.issue(Kb, ld, tc_next, a.s, dstK, wave_u);
      src.issue(Vb, ld, tc_next, a.s, dstV, wave_u);
    }
    if (!live) continue;
    uint2 kw = make_uint2(0xFFFFFFFFu, 0xFFFFFFFFu);          // keep bits of this query row, this wave's keys
    if (DROP && KG == 1) kw = *reinterpret_cast<const uint2*>(kbrow + (k0 >> 5));
    if (DROP && KG == 2) kw.x = kbrow[kw0 >> 5];
    // Head size 128 takes the tile's two 32-key halves one after the other: both at a time are 32 registers more than there are
    // (8 .. 19 spilled ones).
    constexpr int NHB = D == 128 && NK == 2 ? 2 : 1, NKB = NK / NHB;
#pragma unroll
    for (int hb = 0; hb < NHB; ++hb) {
      const int kh0 = kw0 + 32 * NKB * hb;           // first key of this part
      if (NHB > 1 && (kh0 >= klen || (a.causal && kh0 > qw0 + 31))) continue;
      floatx16 sacc[NKB], pacc[NKB];
#pragma unroll
      for (int kt = 0; kt < NKB; ++kt)
#pragma unroll
        for (int e = 0; e < 16; ++e) { sacc[kt][e] = 0.f; pacc[kt][e] = 0.f; }
      // four (two) independent accumulation chains, interleaved
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
        for (int kt = 0; kt < NKB; ++kt) {
          const int r0 = (KG == 2 ? kh : hb * NKB + kt) * 32;
          sacc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_kc(sK, r0, ks, lane), qf[ks], sacc[kt], 0, 0, 0);   // S^T[key][query]
          pacc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_kc(sV, r0, ks, lane), dof[ks], pacc[kt], 0, 0, 0);  // dP^T[key][query]
        }
      __builtin_amdgcn_sched_barrier(0);
      const bool need_mask = (a.causal && kh0 + 32 * NKB - 1 > qw0) || (kh0 + 32 * NKB > klen);   // wave-uniform
      if (DROP) {
        // gradient w.r.t. the undropped probability: keep o dP / (1 - p)
#pragma unroll
        for (int kt = 0; kt < NKB; ++kt) {
          const uint32_t w = (hb * NKB + kt == 0 ? kw.x : kw.y) >> (4 * lh);
#pragma unroll
          for (int e = 0; e < 16; ++e)
            pacc[kt][e] = ((w >> (8 * (e >> 2) + (e & 3))) & 1u) ? pacc[kt][e] * a.drop.scale : 0.f;
        }
      }
      if (need_mask) {
#pragma unroll
        for (int kt = 0; kt < NKB; ++kt)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int key = kh0 + kt * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
            const bool off = key >= klen || (a.causal && key > qi);
            const float p = off ? 0.f : __builtin_amdgcn_exp2f(fmaf(sacc[kt][e], sc, -lse2));
            sacc[kt][e] = p * (pacc[kt][e] - dl);     // dS^T
            if (SPREAD) copy_after(kt * 16 + e);
          }
      } else {
#pragma unroll
        for (int kt = 0; kt < NKB; ++kt)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            sacc[kt][e] = __builtin_amdgcn_exp2f(fmaf(sacc[kt][e], sc, -lse2)) * (pacc[kt][e] - dl);
            if (SPREAD) copy_after(kt * 16 + e);
          }
      }
#pragma unroll
      for (int c = 0; c < 2 * NKB; ++c) {
        const bf16x8 dsf = pack8(sacc[c >> 1], 8 * (c & 1));
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
          dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_tr(sK, (KG == 2 ? 2 * kh : 2 * NKB * hb) + c, dt * 32, lane), dsf, dq[dt], 0, 0, 0);   // dQ^T[dcol][query]
      }
    }
  }
  wait_vmcnt<0>();
  // dQ = the sum over the waves that own the same rows, in a fixed order (all but the first park their accumulators in
  // LDS: [value][lane] per wave)
  if (SP::G > 1) {
    __syncthreads();
    float* park = reinterpret_cast<float*>(lds_raw) + (size_t)wave * (D / 2) * 64 + lane;
    constexpr int PSTEP = RW * (D / 2) * 64;
    if (part > 0) {
      float* dst = park + (part - 1) * PSTEP;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) dst[(dt * 16 + e) * 64] = dq[dt][e];
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int p = 0; p < SP::G - 1; ++p, park += PSTEP)
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) dq[dt][e] += park[(dt * 16 + e) * 64];
  }
  if (qi < a.s) {
    bf16* orow = (bf16*)a.dqkv + ((size_t)bi * a.s + qi) * ld + hd * D;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = (bf16)(dq[dt][4 * g + e] * scale);
        *reinterpret_cast<bf16x4*>(orow + dt * 32 + 8 * g + 4 * lh) = ov;
      }
  }
}

// ------------------------------------------------------------------------------------------ backward: dK, dV
// Workgroup = 128 keys of one (batch, head), a wave owns 32 keys.  Q and dO tiles of 64 queries stream through the DMA
// ring together with the tile's log-sum-exp (log2 units) and delta vectors, which the dQ kernel or, in the joint launch,
// attn_delta_bf16_kernel left in the workspace.
// Per 32-query half tile: S = Q K^T and dP = dO V^T (contraction along D), P = exp2(S sc - lse), dS = P o (dP - delta),
// then dV^T += dO^T P and dK^T += Q^T dS with Q and dO read a second time through the transposing loads.
// Head sizes up to 96 run TWO wave groups (8 waves, two per SIMD): group g takes the query tiles 2 j + g through its own
// ring and the groups' dK / dV sums are added through LDS at the end, which halves the serial chain of the key blocks
// with the most queries (for causal masks block 0 streams every query tile and sets the kernel's duration).  Two waves
// per SIMD leave 256 registers per lane, so the wave's own K and V rows are not held in registers there: the block's
// 128 K and V rows are copied to LDS once and their fragments are read per use.
// Larger heads keep one group (their accumulators alone need more registers) and split the D columns of dK / dV over
// two workgroups instead.
// SPLIT: 64 keys per workgroup, and two waves of each group share a tile's 64 queries (attn_bwd_mode, attn_dkv_split: when).
template <int D, bool DROP, bool SPLIT>
__device__ __forceinline__ void attn_bwd_dkv_block(const AttnArgs a, const AttnBlock blk) {
  typedef ATile<D> TL;
  constexpr int RW = SPLIT ? 2 : ANW, KG = ANW / RW, BKB = 32 * RW, VEC = 2 * ATILE * 4;          // VEC: bytes of the lse + delta vectors of a tile
  constexpr int KBB = DROP ? ATILE * 16 : 0;                  // keep bits of the tile: 64 queries x 128 keys
  constexpr int STAGE = 2 * TL::BYTES + VEC + KBB, LPT = 2 * TL::QPW + 1 + (DROP ? 1 : 0);
  constexpr int NG = dkv_groups<D>(), NST = dkv_stages<D>(), G = KG * NG;
  constexpr bool OWN_LDS = NG == 2 && dkv_own_lds<D>();        // own K / V rows in LDS (after the rings)
  // Large heads: the dK / dV accumulators of all D columns plus the owned K / V rows do not fit the register file
  // (they spilled: 2.3x / 5.6x the d = 96 time at d = 128 / 192).  Two workgroups then share a key block, each
  // accumulating one half of the D columns of dK and dV (the scores are computed by both); this also doubles the
  // number of workgroups where a shard has few heads.
  constexpr int DS = dkv_dsplit<D>(), DH = D / DS;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  // known wave-uniform: mask tests become scalar branches
  const int grp = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8);   // wave group: even / odd query tiles
  const int wave_u = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);       // wave inside its group (copies a quarter of a tile)
  const int wave = wave_u % RW, qh = wave_u / RW;  // its 32 keys, and its 32 queries of a tile (KG = 2)
  const int kb = blk.xb / DS;                      // key block; for causal, block 0 has the most queries: first
  const int dh0 = (blk.xb % DS) * DH;              // first of this workgroup's dK / dV columns
  const int hd = blk.hd, bi = blk.bi;
  const int ld = 3 * a.hl * D;
  const bf16* base = (const bf16*)a.qkv + (size_t)bi * a.s * ld;
  const int klen = attn_key_len(a.key_len, bi, a.s);
  const int kb0 = kb * BKB, kw0 = kb0 + wave * 32, kj = kw0 + l32;
  const int kc = min(kj, a.s - 1);
  ATileSrc<D> src;
  src.init(wave_u, lane);
  const uint32_t lds0 = lds_offset_of(lds_raw);

  // the block's own K and V rows: registers (one group) or BKB / 64 64-row tiles each in LDS (two groups; rows past the
  // end of the sequence repeat the last row, exactly as the register path clamps them)
  bf16x8 kf[OWN_LDS ? 1 : D / 16], vf[OWN_LDS ? 1 : D / 16];
  const unsigned char* ownK = lds_raw + NG * NST * STAGE;
  const unsigned char* ownV = ownK + (BKB / ATILE) * TL::BYTES;
  if (OWN_LDS) {
    // group 0 copies the K rows, group 1 the V rows
    const bf16* P = base + ((grp == 0 ? a.hl : 2 * a.hl) + hd) * D;
    const uint32_t dst = lds0 + NG * NST * STAGE + grp * (BKB / ATILE) * TL::BYTES;
    src.issue(P, ld, kb0, a.s, dst, wave_u);
    if (BKB > ATILE) src.issue(P, ld, kb0 + ATILE, a.s, dst + TL::BYTES, wave_u);
  } else {
    const bf16* krow = base + (size_t)kc * ld + (a.hl + hd) * D;
    const bf16* vrow = base + (size_t)kc * ld + (2 * a.hl + hd) * D;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      kf[ks] = *reinterpret_cast<const bf16x8*>(krow + ks * 16 + lh * 8);
      vf[ks] = *reinterpret_cast<const bf16x8*>(vrow + ks * 16 + lh * 8);
    }
  }
  const unsigned char* myK = ownK + (wave >> 1) * TL::BYTES;   // the tile that holds this wave's 32 rows, at (wave & 1) 32
  const unsigned char* myV = ownV + (wave >> 1) * TL::BYTES;
  const int own_r0 = (wave & 1) * 32;
  floatx16 dk[DH / 32], dv[DH / 32];
#pragma unroll
  for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) { dk[dt][e] = 0.f; dv[dt][e] = 0.f; }
  const float scale = 1.0f / sqrtf((float)D);
  const float sc = kLog2e * scale;
  const int nqt = (a.s + ATILE - 1) / ATILE;
  int qt0 = a.causal ? kb0 / ATILE : 0;
  if (kb0 >= klen) qt0 = nqt;                     // every key of the block is padding: gradients are zero
  const int nt = nqt - qt0;                       // tiles to stream (block-uniform)
  const int njt = (nt + NG - 1) / NG;             // steps: group g handles tile NG j + g in step j (if it exists)
  const bf16* Qb = base + hd * D;
  const int ldo = a.hl * D;
  const bf16* dOb = (const bf16*)a.dctx + (size_t)bi * a.s * ldo + hd * D;
  // per-query vectors in the workspace: [0] delta, [1] log-sum-exp in log2 units (by the dQ kernel or attn_delta_bf16_kernel)
  const size_t nrow_all = (size_t)a.b * a.hl * a.s;
  const float* vec_b = ((wave_u & 1) ? a.delta + nrow_all : a.delta) + ((size_t)bi * a.hl + hd) * a.s;
  unsigned char* ring = lds_raw + grp * (NST * STAGE);        // this group's ring
  const uint32_t ring0 = lds0 + grp * (NST * STAGE);
  auto issue_tile = [&](int t, int st) {          // tile index relative to qt0 (clamped), ring stage
    const int r0 = (qt0 + min(t, nt - 1)) * ATILE;
    const uint32_t sb = ring0 + st * STAGE;
    src.issue(Qb, ld, r0, a.s, sb, wave_u);
    src.issue(dOb, ldo, r0, a.s, sb + TL::BYTES, wave_u);
    // waves 0, 2 copy the delta vector, waves 1, 3 the log-sum-exp vector (same data twice: uniform copy counts)
    dma4(vec_b + min(r0 + lane, a.s - 1), sb + 2 * TL::BYTES + (wave_u & 1) * (ATILE * 4));
    if (DROP) {
      // lane t copies the four words of query r0 + t that cover this block's keys (and, of 64 keys, the other half of
      // their 128: a row holds whole groups of four words); every wave copies the same kilobyte: uniform copy counts
      const uint32_t* src_bits = a.keep_bits + (((size_t)bi * a.hl + hd) * a.s + min(r0 + lane, a.s - 1)) * a.keep_pitch +
                                 ((kb0 >> 5) & ~3);
      dma16(reinterpret_cast<const bf16*>(src_bits), sb + 2 * TL::BYTES + VEC);
    }
  };
  if (nt > 0) {
#pragma unroll
    for (int t = 0; t < NST - 1; ++t) issue_tile(NG * t + grp, t);
  }
  int stage = 0;
  for (int j = 0; j < njt; ++j) {
    const int t = NG * j + grp;
    const int q0 = (qt0 + t) * ATILE;
    wait_vmcnt<LPT*(NST - 2)>();                   // this wave's copies of step j (and of the own rows) have landed
    __builtin_amdgcn_s_barrier();                 // everyone's have; and everyone is done with step j - 1
    // (issued in one burst: spreading these copies over the element-wise passes, as the forward and dQ kernels do,
    // measured slower here -- the passes read the per-query vectors from LDS and the copies' compiler-level memory
    // barrier pins those reads)
    issue_tile(t + NG * (NST - 1), stage == 0 ? NST - 1 : stage - 1);
    const unsigned char* sQ = ring + stage * STAGE;
    const unsigned char* sdO = sQ + TL::BYTES;
    const float* sDl = reinterpret_cast<const float*>(sdO + TL::BYTES);
    const float* sLse = sDl + ATILE;
    const uint32_t* sBits = reinterpret_cast<const uint32_t*>(sLse + ATILE);   // [64 queries][4 words]
    stage = stage == NST - 1 ? 0 : stage + 1;
    const int ql = q0 + (KG == 2 ? 32 * qh + 31 : ATILE - 1);      // this wave's last query of the tile
    if (t >= nt || (a.causal && ql < kw0)) continue;               // no such tile / every query precedes this wave's keys
    const bool need_mask = (a.causal && q0 < kw0 + 31) || (kw0 + 32 > klen) || (q0 + ATILE > a.s);   // wave-uniform
#pragma unroll
    for (int qi = 0; qi < 2 / KG; ++qi) {
      const int qs = KG == 2 ? qh : qi;
      floatx16 sacc, pacc;
#pragma unroll
      for (int e = 0; e < 16; ++e) { sacc[e] = 0.f; pacc[e] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) {
        const bf16x8 kk = OWN_LDS ? TL::frag_kc(myK, own_r0, ks, lane) : kf[OWN_LDS ? 0 : ks];
        const bf16x8 vv = OWN_LDS ? TL::frag_kc(myV, own_r0, ks, lane) : vf[OWN_LDS ? 0 : ks];
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_kc(sQ, qs * 32, ks, lane), kk, sacc, 0, 0, 0);    // S[query][key]
        pacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_kc(sdO, qs * 32, ks, lane), vv, pacc, 0, 0, 0);   // dP[query][key]
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int qoff = qs * 32 + 8 * g + 4 * lh;
        const float4 l4 = *reinterpret_cast<const float4*>(sLse + qoff);
        const float4 d4 = *reinterpret_cast<const float4*>(sDl + qoff);
        const float lv4[4] = {l4.x, l4.y, l4.z, l4.w};
        const float dv4[4] = {d4.x, d4.y, d4.z, d4.w};
        float p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(sacc[4 * g + e], sc, -lv4[e]));
        if (need_mask) {
          asm volatile("");                            // (stays a scalar branch: without it every tile pays for the selects)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int q = q0 + qoff + e;
            p[e] = (kj >= klen || q >= a.s || (a.causal && kj > q)) ? 0.f : p[e];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (DROP) {
            const bool keep = (sBits[(qoff + e) * 4 + (SPLIT ? (kb0 >> 5) & 3 : 0) + wave] >> l32) & 1u;
            sacc[4 * g + e] = keep ? p[e] * a.drop.scale : 0.f;                                       // dropped P (for dV)
            pacc[4 * g + e] = p[e] * ((keep ? pacc[4 * g + e] * a.drop.scale : 0.f) - dv4[e]);        // dS
          } else {
            sacc[4 * g + e] = p[e];                                // P
            pacc[4 * g + e] = p[e] * (pacc[4 * g + e] - dv4[e]);   // dS
          }
        }
      }
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const int c = 2 * qs + cc;
        const bf16x8 pf = pack8(sacc, 8 * cc);
        const bf16x8 dsf = pack8(pacc, 8 * cc);
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt) {
          dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_tr(sdO, c, dh0 + dt * 32, lane), pf, dv[dt], 0, 0, 0);    // dV^T[dcol][key]
          dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TL::frag_tr(sQ, c, dh0 + dt * 32, lane), dsf, dk[dt], 0, 0, 0);    // dK^T[dcol][key]
        }
      }
    }
  }
  wait_vmcnt<0>();
  // dK, dV = the sums over the waves that own the same keys, in a fixed order (all but the first park their accumulators in
  // LDS: [value][lane] per wave)
  if (G > 1) {
    __syncthreads();
    constexpr int NV = 2 * (DH / 32) * 16, PSTEP = RW * NV * 64;
    const int part = qh + KG * grp;
    float* park = reinterpret_cast<float*>(lds_raw) + (size_t)wave * NV * 64 + lane;
    if (part > 0) {
      float* dst = park + (part - 1) * PSTEP;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          dst[(dt * 16 + e) * 64] = dk[dt][e];
          dst[((DH / 32 + dt) * 16 + e) * 64] = dv[dt][e];
        }
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int p = 0; p < G - 1; ++p, park += PSTEP)
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          dk[dt][e] += park[(dt * 16 + e) * 64];
          dv[dt][e] += park[((DH / 32 + dt) * 16 + e) * 64];
        }
  }
  if (kj < a.s) {
    bf16* krow = (bf16*)a.dqkv + ((size_t)bi * a.s + kj) * ld + (a.hl + hd) * D;
    bf16* vrow = (bf16*)a.dqkv + ((size_t)bi * a.s + kj) * ld + (2 * a.hl + hd) * D;
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 ok, ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ok[e] = (bf16)(dk[dt][4 * g + e] * scale);
          ov[e] = (bf16)dv[dt][4 * g + e];
        }
        *reinterpret_cast<bf16x4*>(krow + dh0 + dt * 32 + 8 * g + 4 * lh) = ok;
        *reinterpret_cast<bf16x4*>(vrow + dh0 + dt * 32 + 8 * g + 4 * lh) = ov;
      }
  }
}

// The two as kernels of their own (attn_bwd_mode: when).
template <int D, bool DROP, int MODE>
__global__ __launch_bounds__((AttnSplit<D, MODE>::NT), (AttnSplit<D, MODE>::MINW)) void attn_bwd_dq_bf16_kernel(AttnArgs a) {
  constexpr int BQ = 32 * AttnSplit<D, MODE>::RW;
  const AttnBlock blk = attn_block((a.s + BQ - 1) / BQ, a.hl, a.b);
  if (blk.valid) attn_bwd_dq_block<D, DROP, MODE, false>(a, blk);
}
template <int D, bool DROP, bool SPLIT>
__global__ __launch_bounds__(dkv_groups<D>() * ANT) void attn_bwd_dkv_bf16_kernel(AttnArgs a) {
  constexpr int BKB = SPLIT ? 64 : 128;
  const AttnBlock blk = attn_block((a.s + BKB - 1) / BKB * dkv_dsplit<D>(), a.hl, a.b);
  if (blk.valid) attn_bwd_dkv_block<D, DROP, SPLIT>(a, blk);
}

// ------------------------------------------------------------------------------------------ backward in one launch
// dQ and dK/dV blocks in one grid.  Under a causal mask the blocks of either kernel differ by up to 16 x at 2048 tokens, and with
// about one workgroup per compute unit the longest is the kernel's time while the others idle; together, the longest of both
// kinds first, the short blocks of one fill up behind the long ones of the other.  Without a mask, two kinds that leave compute
// units idle share them.  dK/dV then cannot wait for dQ's delta: it comes from a small kernel ahead of both.
// Order on an XCD: groups of `pg` pairs (whose K, V, Q and dO rows its L2 holds), in a group the blocks of rank 0 of all pairs,
// of rank 1, .., the two kinds spread evenly over the ranks.
struct AttnJoint { int nq, nk, pg; };      // dQ and dK/dV blocks of a pair, pairs of a group

template <int D, bool DROP, int MODE, bool SPLIT>
__global__ __launch_bounds__((AttnSplit<D, MODE>::NT), (AttnSplit<D, MODE>::MINW)) void attn_bwd_bf16_kernel(AttnArgs a, AttnJoint jt) {
  static_assert(AttnSplit<D, MODE>::NT == dkv_groups<D>() * ANT, "both kinds of block have the same number of waves");
  const int pairs = a.hl * a.b, npx = (pairs + 7) / 8, per = jt.nq + jt.nk;
  int r = blockIdx.x >> 3;
  const int g = r / (jt.pg * per);
  r -= g * jt.pg * per;
  const int size = min(jt.pg, npx - g * jt.pg);               // (the last group may be smaller)
  const int rank = r / size, pair = (g * jt.pg + r - rank * size) * 8 + (blockIdx.x & 7);
  if (pair >= pairs) return;
  const int before = rank * jt.nq / per;                       // dQ blocks among the ranks below
  const bool is_dq = (rank + 1) * jt.nq / per > before;
  AttnBlock blk;
  blk.xb = is_dq ? before : rank - before;
  blk.hd = pair % a.hl;
  blk.bi = pair / a.hl;
  blk.valid = true;
  if (is_dq) attn_bwd_dq_block<D, DROP, MODE, true>(a, blk);
  else attn_bwd_dkv_block<D, DROP, SPLIT>(a, blk);
}

// delta = rowsum(dO o O), and the log-sum-exp in log2 units: four lanes per (batch, head, query), 16-byte loads.  Bound by the
// launch (3 us up to 8192 x 384).
template <int D>
__global__ __launch_bounds__(256) void attn_delta_bf16_kernel(AttnArgs a) {
  const size_t rows = (size_t)a.b * a.hl * a.s, r = ((size_t)blockIdx.x * 256 + threadIdx.x) >> 2;
  if (r >= rows) return;                                       // whole groups of four lanes
  const int i = r % a.s, hd = r / a.s % a.hl, bi = r / a.s / a.hl, c = threadIdx.x & 3;
  const size_t at = ((size_t)bi * a.s + i) * (a.hl * D) + hd * D;
  float dl = 0.f;
#pragma unroll
  for (int u = 0; u < D / 32; ++u) {
    const bf16x8 d = *reinterpret_cast<const bf16x8*>((const bf16*)a.dctx + at + 32 * u + 8 * c);
    const bf16x8 o = *reinterpret_cast<const bf16x8*>((const bf16*)a.ctx + at + 32 * u + 8 * c);
#pragma unroll
    for (int e = 0; e < 8; ++e) dl = fmaf((float)d[e], (float)o[e], dl);
  }
  dl += __shfl_xor(dl, 1, 64);
  dl += __shfl_xor(dl, 2, 64);
  if (c == 0) {
    a.delta[r] = dl;
    a.delta[rows + r] = a.lse[r] * kLog2e;
  }
}

// ------------------------------------------------------------------------------------------ launchers
bool attn_bf16_supported(int d) { return d == 64 || d == 96 || d == 128 || d == 192; }

template <int D, bool DROP, int MODE, bool FOLD>
static hipError_t launch_fwd_m(const AttnArgs& a, hipStream_t st) {
  typedef AttnSplit<D, MODE> SP;
  auto kern = attn_fwd_bf16_kernel<D, DROP, MODE, FOLD>;
  static LdsAttrOnce attr;
  if (SP::LDS > 64 * 1024)
    if (hipError_t e = attr.ensure((const void*)kern, (int)SP::LDS); e != hipSuccess) return e;
  const dim3 grid = attn_grid((a.s + 32 * SP::RW - 1) / (32 * SP::RW), a.hl, a.b);
  hipLaunchKernelGGL(kern, grid, dim3(SP::NT), SP::LDS, st, a);
  return hipGetLastError();
}

// (kernels of their own: with the fold a run-time switch, blocks took 8.2 us for 7.5 at 4 heads of 96, 200 tokens)
template <int D, bool DROP>
static hipError_t launch_fwd_dd(const AttnArgs& a, hipStream_t st) {
  const AttnMode m = attn_mode(a.s, a.hl * a.b, a.causal != 0, D);
  const bool fold = a.causal && attn_fwd_fold(m, a.s, a.hl * a.b);
  if constexpr (D <= 128) {
    if (m == ATTN_PAIR) return fold ? launch_fwd_m<D, DROP, ATTN_PAIR, true>(a, st) : launch_fwd_m<D, DROP, ATTN_PAIR, false>(a, st);
    if (m == ATTN_SPLIT && fold) return launch_fwd_m<D, DROP, ATTN_SPLIT, true>(a, st);
  }
  return m == ATTN_SPLIT ? launch_fwd_m<D, DROP, ATTN_SPLIT, false>(a, st) : launch_fwd_m<D, DROP, ATTN_WIDE, false>(a, st);
}

template <int D>
static hipError_t launch_fwd_d(const AttnArgs& a, hipStream_t st) {
  return a.drop.enabled ? launch_fwd_dd<D, true>(a, st) : launch_fwd_dd<D, false>(a, st);
}

// LDS of a dK/dV block: rings and the owned K / V rows (two groups); at the end the parked accumulators.
template <int D, bool DROP, bool SPLIT> constexpr size_t dkv_lds_bytes() {
  constexpr int RW = SPLIT ? 2 : ANW, NG = dkv_groups<D>(), G = NG * ANW / RW;
  constexpr size_t kStage = 2 * ATile<D>::BYTES + 2 * ATILE * 4 + (DROP ? ATILE * 16 : 0);
  constexpr size_t kOwn = (NG == 2 && dkv_own_lds<D>()) ? RW * ATile<D>::BYTES : 0;
  constexpr size_t kRing = (size_t)NG * dkv_stages<D>() * kStage + kOwn;
  constexpr size_t kPark = (size_t)(G - 1) * RW * 2 * (D / dkv_dsplit<D>() / 32) * 16 * 64 * 4;
  return kRing > kPark ? kRing : kPark;
}

template <int D, bool DROP, int MODE, bool SPLIT>
static hipError_t launch_bwd_joint(const AttnArgs& a, hipStream_t st) {
  typedef AttnSplit<D, MODE> SP;
  auto kern = attn_bwd_bf16_kernel<D, DROP, MODE, SPLIT>;
  constexpr size_t kDkv = dkv_lds_bytes<D, DROP, SPLIT>(), kLds = SP::LDS > kDkv ? SP::LDS : kDkv;
  static_assert(kLds <= 160 * 1024, "LDS budget");
  static LdsAttrOnce attr;
  if (hipError_t e = attr.ensure((const void*)kern, (int)kLds); e != hipSuccess) return e;
  const size_t rows = (size_t)a.b * a.hl * a.s;
  hipLaunchKernelGGL((attn_delta_bf16_kernel<D>), dim3((unsigned)((rows + 63) / 64)), dim3(256), 0, st, a);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  constexpr int BKB = SPLIT ? 64 : 128;
  AttnJoint jt;
  jt.nq = (a.s + 32 * SP::RW - 1) / (32 * SP::RW);
  jt.nk = (a.s + BKB - 1) / BKB * dkv_dsplit<D>();
  const int npx = (a.hl * a.b + 7) / 8, per = jt.nq + jt.nk;
  jt.pg = (2 * (gemm_cu_count() / 8) + per - 1) / per;         // two workgroups per compute unit of the XCD to choose from
  if (jt.pg > npx) jt.pg = npx;
  hipLaunchKernelGGL(kern, dim3((unsigned)(8 * npx * per)), dim3(SP::NT), kLds, st, a, jt);
  return hipGetLastError();
}

template <int D, bool DROP, int MODE>
static hipError_t launch_dq_m(const AttnArgs& a, hipStream_t st) {
  typedef AttnSplit<D, MODE> SP;
  static LdsAttrOnce attr;
  if (SP::LDS > 64 * 1024)
    if (hipError_t e = attr.ensure((const void*)attn_bwd_dq_bf16_kernel<D, DROP, MODE>, (int)SP::LDS); e != hipSuccess) return e;
  const dim3 grid = attn_grid((a.s + 32 * SP::RW - 1) / (32 * SP::RW), a.hl, a.b);
  hipLaunchKernelGGL((attn_bwd_dq_bf16_kernel<D, DROP, MODE>), grid, dim3(SP::NT), SP::LDS, st, a);
  return hipGetLastError();
}

template <int D, bool DROP, bool SPLIT>
static hipError_t launch_dkv(const AttnArgs& a, hipStream_t st) {
  constexpr int BKB = SPLIT ? 64 : 128;
  constexpr size_t kLds = dkv_lds_bytes<D, DROP, SPLIT>();
  static_assert(kLds <= 160 * 1024, "LDS budget");
  static LdsAttrOnce attr;
  if (kLds > 64 * 1024)
    if (hipError_t e = attr.ensure((const void*)attn_bwd_dkv_bf16_kernel<D, DROP, SPLIT>, (int)kLds); e != hipSuccess) return e;
  const dim3 grid = attn_grid((a.s + BKB - 1) / BKB * dkv_dsplit<D>(), a.hl, a.b);
  hipLaunchKernelGGL((attn_bwd_dkv_bf16_kernel<D, DROP, SPLIT>), grid, dim3(dkv_groups<D>() * ANT), kLds, st, a);
  return hipGetLastError();
}

template <int D, bool DROP>
static hipError_t launch_bwd_dd(const AttnArgs& a, hipStream_t st) {
  const int pairs = a.hl * a.b;
  const bool causal = a.causal != 0;
  if constexpr (D > 128) {
    return launch_bwd_joint<D, DROP, ATTN_WIDE, false>(a, st);
  } else {
    const AttnBwdMode bm = attn_bwd_mode(a.s, pairs, causal, dkv_dsplit<D>());
    if (bm == ATTN_BWD_JOINT) return launch_bwd_joint<D, DROP, ATTN_PAIR, false>(a, st);
    if (bm == ATTN_BWD_JOINT_SPLIT) return launch_bwd_joint<D, DROP, ATTN_SPLIT, true>(a, st);
    const AttnMode m = attn_mode(a.s, pairs, causal, D);
    hipError_t e = m == ATTN_PAIR    ? launch_dq_m<D, DROP, ATTN_PAIR>(a, st)
                   : m == ATTN_SPLIT ? launch_dq_m<D, DROP, ATTN_SPLIT>(a, st)
                                     : launch_dq_m<D, DROP, ATTN_WIDE>(a, st);
    if (e != hipSuccess) return e;
    if constexpr (D <= 96)
      if (!causal && attn_dkv_split(a.s, pairs)) return launch_dkv<D, DROP, true>(a, st);
    return launch_dkv<D, DROP, false>(a, st);
  }
}

template <int D>
static hipError_t launch_bwd_d(const AttnArgs& a, hipStream_t st) {
  return a.drop.enabled ? launch_bwd_dd<D, true>(a, st) : launch_bwd_dd<D, false>(a, st);
}

hipError_t launch_attn_fwd_bf16(const AttnArgs& a, hipStream_t st) {
  switch (a.d) {
    case 64: return launch_fwd_d<64>(a, st);
    case 96: return launch_fwd_d<96>(a, st);
    case 128: return launch_fwd_d<128>(a, st);
    case 192: return launch_fwd_d<192>(a, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_attn_bwd_bf16(const AttnArgs& a, hipStream_t st) {
  switch (a.d) {
    case 64: return launch_bwd_d<64>(a, st);
    case 96: return launch_bwd_d<96>(a, st);
    case 128: return launch_bwd_d<128>(a, st);
    case 192: return launch_bwd_d<192>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mlm
