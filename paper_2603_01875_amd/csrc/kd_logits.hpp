// What the logit kernels are made of: the work maps, and the epilogues that turn a finished tile of both models' logits into
// statistics, row sums or dL/dz_s, on either tile loop.  The kernels are in kd_kernels.hip and kd_strip_hv.hip.
#pragma once
#include "kd_common.hpp"

// tile configurations (overridable for tuning experiments)
#ifndef KD_LOGIT_CFG
#define KD_LOGIT_CFG 2, 2, 4, 64, 3     // MI, NI, WN, BK, NST: 128 x 256 tile, 8 waves
#endif

namespace kd {

typedef TileCfg<KD_LOGIT_CFG> LCfg;   // logit tiles: two accumulators per tile
constexpr int BK = LCfg::BK;
constexpr int NI = LCfg::NI;
static_assert(LCfg::BM == kTileM && BN == kTileN, "planner and kernels disagree");
constexpr int BM = LCfg::BM;
constexpr int MI = LCfg::MI;
typedef LCfg::Acc AccTile;
__device__ __forceinline__ int acc_m(int wm, int mt, int r, int lane) { return LCfg::acc_m(wm, mt, r, lane); }
__device__ __forceinline__ int acc_n(int wn, int nt, int lane) { return LCfg::acc_n(wn, nt, lane); }

// ------------------------------------------------------------------------------------------
// work maps
// ------------------------------------------------------------------------------------------

// Index q over an (na x nb) grid walked in (ba x bb) blocks, a fastest inside a block.
__device__ __forceinline__ void block_decode(int q, int na, int ba, int bb, int& a, int& b) {
  const int per = ba * bb;
  const int blk = q / per, w = q - blk * per;
  const int nblk_a = na / ba;
  a = (blk % nblk_a) * ba + w % ba;
  b = (blk / nblk_a) * bb + w / ba;
}

struct LogitArgs {
  const bf16_t* W_s; const bf16_t* h_s; const bf16_t* W_t; const bf16_t* h_t;
  int T, V, H_s, H_t;  // H_*: contraction length and row stride of the (re-packed) hidden states
  int ld_s, ld_t;      // elements from row to row of the heads ([V][H]: H, or the contraction length where re-packed; [H][V]: V)
  const int* meta;     // device-side plan: valid tokens, token tiles, vocabulary splits
  int v0, v_end;       // vocabulary rows [v0, v_end) handled by this launch
  int n_vt;            // ... in this many tiles
  int bb;              // grad kernel, eight-wave loop: block width of the work map along the vocabulary (bb | n_vt).
                       // An XCD's 32 workgroups cover 2 token tiles x 16 vocabulary tiles where the
                       // counts allow: measured 2-3 % faster than 4 x 8 for this kernel (1 x 32 and
                       // 8 x 4 are slower), while the statistics kernels do not care
  float c;             // log2(e) / tau
  float beta;
  float t_scale;       // fp8 teacher: z_t = t_scale * (product of the e4m3 codes); 1 otherwise
  int T_pad;
  float* partials;     // stats: [ranges][5][T_pad];  jsd: [ranges][2][T_pad]
  const f32x4* rowinfo;// [T_pad]: {lse2_t, lse2_s, mask/(n tau), row term}
  const float* akl;    // AKL only: [AKL_ROWS][T_pad] per-token values (see the AKL_* indices)
  unsigned long long* akl_fine;  // ... [T_pad][AKL_BINS][2] sums of the row pass (strip loop)
  float akl_width;     // ... cells in a bin of this search pass (strip loop)
  bf16_t* dz;          // chunk of dL/dz_s, ldz columns, in the order of dz_chunk
  int ldz;
  int last_chunk;      // this launch handles the last chunk of the vocabulary
  int dz_accumulate;   // add to dz instead of overwriting it (further teachers of a multi-teacher call)
  long long* clock_out;// measurement aid (may be null): workgroup 0 of the statistics kernel stores the shader
                       // cycles and the 100 MHz ticks its tile loop took
};

// TF8: the teacher operands are e4m3 bytes (one byte per element, 128 elements per k-step).
// WHV: the heads are stored [H][V] (vocabulary contiguous), i.e. k-major for the logit products.
template <bool TF8, bool WHV>
__device__ __forceinline__ WorkItem logit_item(const LogitArgs& a, int vt, int tt) {
  WorkItem it;
  const int m0 = a.v0 + vt * BM;
  it.B0 = a.h_s + (int64_t)tt * BN * a.H_s;
  if (WHV) {
    it.A0 = a.W_s + m0;
    it.A1 = a.W_t + m0;
    it.B1 = a.h_t + (int64_t)tt * BN * a.H_t;
  } else if (TF8) {
    it.A0 = a.W_s + (int64_t)m0 * a.ld_s;
    it.A1 = (const bf16_t*)((const char*)a.W_t + (int64_t)m0 * a.H_t);
    it.B1 = (const bf16_t*)((const char*)a.h_t + (int64_t)tt * BN * a.H_t);
  } else {
    it.A0 = a.W_s + (int64_t)m0 * a.ld_s;
    it.A1 = a.W_t + (int64_t)m0 * a.ld_t;
    it.B1 = a.h_t + (int64_t)tt * BN * a.H_t;
  }
  it.a_rows = min(BM, a.v_end - m0);
  it.b_rows = min(BN, a.T - tt * BN);
  it.nk0 = a.H_s / BK;
  it.nk1 = a.H_t / (TF8 ? 2 * BK : BK);
  it.m0 = m0;
  it.n0 = tt * BN;
  it.aux = 0;
  return it;
}

// One workgroup = one (token tile, vocabulary split); it walks the split's tiles in order.
struct SplitMap {
  const LogitArgs& a;
  int tt, split, lo, cnt;
  __device__ SplitMap(const LogitArgs& a_) : a(a_) {
    const int n_tt = meta_get(a.meta, META_N_TT), n_split = meta_get(a.meta, META_N_SPLIT);
    const int active = n_tt * n_split;               // the grid is sized for the unmasked worst case
    tt = split = lo = cnt = 0;
    if ((int)blockIdx.x >= active) return;
    group_decode(xcd_logical_id(blockIdx.x, active), n_tt, n_split, tt, split);
    lo = (int)(((int64_t)split * a.n_vt) / n_split);
    const int hi = (int)(((int64_t)(split + 1) * a.n_vt) / n_split);
    cnt = hi - lo;
  }
  __device__ int n_items() const { return cnt; }
};
template <bool TF8, bool WHV>
struct SplitWork : SplitMap {
  using SplitMap::SplitMap;
  __device__ WorkItem item(int i) const { return logit_item<TF8, WHV>(a, lo + i, tt); }
};

// The strip loop's share of a workgroup.  With n_split > 0: one (token tile, vocabulary range), the ranges in units
// of 64 rows, walked in tiles of three units and a rest.  With n_split == 0: the (token tile x 192-row tile) grid,
// four token tiles at a time, strided over kNumCU persistent workgroups (which evens out better where few tiles per
// workgroup meet an awkward number of token tiles: 29 x 43 tiles in five rounds, not six).
// HV: the heads are stored [H][V] (their rows are k-rows).
template <bool HV>
struct StripWork {
  const LogitArgs& a;
  int n_tt, tt, split, row0, row1, cnt, L, G, n_vt;
  __device__ StripWork(const LogitArgs& a_, int n_split) : a(a_) {
    n_tt = meta_get(a.meta, META_N_TT);
    tt = split = row0 = row1 = cnt = L = n_vt = 0;
    G = 1;
    if (n_split == 0) {
      G = min((int)gridDim.x, kNumCU);
      n_vt = (a.v_end - a.v0 + StripCfg::BM - 1) / StripCfg::BM;
      if ((int)blockIdx.x >= G) return;
      L = xcd_logical_id(blockIdx.x, G);
      cnt = L < n_tt * n_vt ? (n_tt * n_vt - L + G - 1) / G : 0;
      return;
    }
    const int active = n_tt * n_split;               // the grid is sized for the unmasked worst case
    if ((int)blockIdx.x >= active) return;
    group_decode(xcd_logical_id(blockIdx.x, active), n_tt, n_split, tt, split);
    const int units = (a.v_end - a.v0 + 63) / 64;
    row0 = a.v0 + 64 * (int)(((int64_t)split * units) / n_split);
    row1 = min(a.v_end, a.v0 + 64 * (int)(((int64_t)(split + 1) * units) / n_split));
    cnt = (row1 - row0 + StripCfg::BM - 1) / StripCfg::BM;
  }
  __device__ int n_items() const { return cnt; }
  __device__ StripItem item(int i) const {
    const auto p = kernel_args<LogitArgs>();
    StripItem it;
    int m0 = row0 + i * StripCfg::BM, n0 = tt * BN, end = row1;
    if (n_vt > 0) {
      const int q = i * G + L, n_four = n_tt / 4, grp = q / (4 * n_vt), w = q - grp * 4 * n_vt;
      const int g = grp < n_four ? 4 : n_tt - 4 * n_four;
      const int vt = w / g;
      n0 = (4 * grp + w - vt * g) * BN;
      m0 = p->v0 + vt * StripCfg::BM;
      end = p->v_end;
    }
    it.a_rows = min(StripCfg::BM, end - m0);
    it.out_rows = (it.a_rows + 63) / 64 * 64;        // zeros behind the chunk's last row: the k-steps of grad_h_s are whole
    it.m0 = m0;
    it.n0 = n0;
    it.k0 = p->H_s; it.k1 = p->H_t;
    it.lda0 = 2 * p->ld_s; it.ldb0 = 128 * it.k0;
    it.lda1 = 2 * p->ld_t; it.ldb1 = 128 * it.k1;
    it.A0 = (const char*)p->W_s + (int64_t)m0 * (HV ? 2 : it.lda0);
    it.A1 = (const char*)p->W_t + (int64_t)m0 * (HV ? 2 : it.lda1);
    it.B0 = (const char*)p->h_s + (int64_t)n0 * (2 * it.k0);
    it.B1 = (const char*)p->h_t + (int64_t)n0 * (2 * it.k1);
    it.aux = it.b_blocks = 0;
    return it;
  }
};
// Teacher product only (one accumulator): the AKL threshold search.
template <bool WHV>
struct TeacherSplitWork : SplitMap {
  using SplitMap::SplitMap;
  __device__ WorkItem item(int i) const {
    WorkItem it = logit_item<false, WHV>(a, lo + i, tt);
    it.A0 = it.A1; it.B0 = it.B1;       // phase 0 is the teacher product
    it.nk0 = it.nk1;
    return it;
  }
};

// Persistent workgroups striding over the (token tile x vocabulary tile) grid of a chunk.
struct ChunkMap {
  const LogitArgs& a;
  int L, G, n_tiles, n_tt, ba;
  __device__ ChunkMap(const LogitArgs& a_) : a(a_) {
    G = gridDim.x;
    L = xcd_logical_id(blockIdx.x, G);
    n_tt = meta_get(a.meta, META_N_TT);
    ba = 1;                                          // ba | n_tt, ba * bb <= 32: one block per XCD
    for (int d = 2; d * a.bb <= 32; ++d) if (n_tt % d == 0) ba = d;
    n_tiles = n_tt * a.n_vt;
  }
  __device__ int n_items() const { return L < n_tiles ? (n_tiles - L + G - 1) / G : 0; }
  __device__ void tile(int i, int& tt, int& vt) const { block_decode(i * G + L, n_tt, ba, a.bb, tt, vt); }
};
template <bool TF8, bool WHV>
struct ChunkWork : ChunkMap {
  using ChunkMap::ChunkMap;
  __device__ WorkItem item(int i) const {
    int tt, vt;
    tile(i, tt, vt);
    return logit_item<TF8, WHV>(a, vt, tt);
  }
};
// ------------------------------------------------------------------------------------------
// epilogues of the logit tiles
// ------------------------------------------------------------------------------------------
constexpr float NEG_BIG = -1.0e30f;   // logit given to vocabulary rows beyond V: every exp of it is 0
// Running maxima start here, far below any real scaled logit and far above NEG_BIG * c (the host
// bounds tau so that c > 1e-9): a lane that has seen only masked rows keeps this maximum, so the
// exponent of a masked entry stays hugely negative instead of cancelling to a rounding residual.
constexpr float M_FLOOR = -1.0e20f;
constexpr float LN2 = 0.6931471805599453f;

// Adaptive KL: per-token values kept between its passes, [AKL_ROWS][T_pad] floats.
enum { AKL_FKL = 0, AKL_RKL = 1,   // the token's forward / reverse KL
       AKL_LO = 2, AKL_HI = 3,     // search interval of the head threshold (base-2 teacher log-probability):
                                   // mass{lt >= LO} > mu >= mass{lt >= HI}
                                   // (strip loop, during the search: LO as the number of its cell, HI the grid's lower end)
       AKL_LTMAX = 4,              // the largest teacher log-probability of the token
       AKL_WR = 5,                 // weight of the reverse KL (the forward KL has 1 - that)
                                   // (strip loop, between search passes: the mass above the interval)
       AKL_CROWD = 6,              // strip loop: many entries in the token's last interval
       AKL_ROWS = kAklRows };
constexpr int AKL_K = kAklThresholds;   // thresholds tried per search pass of the eight-wave loop: 17-fold narrowing
constexpr int AKL_BINS = kAklBins;      // bins of a search pass of the strip loop
// The strip loop's grid of a token, from `low` up: its cell, and edge j.  The search and its merge must both use these expressions:
// an entry lies in the cell between the two edges that it compares with, and in no other pass in another one.
__device__ __forceinline__ float akl_cell(float low, float ltmax) { return (ltmax + 1.0e-3f - low) * (1.f / kAklCells); }
__device__ __forceinline__ float akl_edge(float j, float low, float cell) { return fmaf(j, cell, low); }
constexpr float AKL_TOP_EPS = 1.0e-4f;   // entries this close (base-2 log) to the token's largest one count as "the top entry"

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float flog2(float x) { return __builtin_amdgcn_logf(x); }

// How a lane sees a finished tile: NC token columns of (up to) NE vocabulary entries each, entry e of the lane's
// share lying at vocabulary row m(e) of the tile (four consecutive e are four consecutive rows), column j at
// token n(j).  One partial result per token leaves a workgroup: gather() sums those of the lanes that share a token.
struct TileGeo {         // 128 x 256 tile of eight waves (kd_mfma.hpp)
  static constexpr int NC = NI, NE = MI * 16;
  static constexpr bool IN_LDS = false;              // where GradEpi keeps what it knows of the tokens
  int wm, wn, lane;
  __device__ TileGeo() {
    lane = threadIdx.x & 63;
    wm = (threadIdx.x >> 6) & 1;
    wn = threadIdx.x >> 7;
  }
  __device__ __forceinline__ int m(int e) const { return acc_m(wm, e >> 4, e & 15, lane); }
  __device__ __forceinline__ int n(int j) const { return acc_n(wn, j, lane); }
  // A token is shared by the halves of a wave and by two waves, which meet in LDS behind the loop.  merge(i, x, y): value i of two
  // shares put together.  True in the lanes that hold the result.
  template <int N, class Merge>
  __device__ __forceinline__ bool gather(float (&v)[N], char* smem, Merge&& merge) const {
    float* const box = (float*)smem + wn * N * 32 + (lane & 31);
    float o[N];
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = __shfl_xor(v[i], 32, 64);
    merge(v, o);
    __syncthreads();                                 // (every wave has read its last fragments, and its last loads have landed)
    if (wm == 1 && lane < 32)
#pragma unroll
      for (int i = 0; i < N; ++i) box[32 * i] = v[i];
    __syncthreads();
    if (wm == 1 || lane >= 32) return false;
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = box[32 * i];
    merge(v, o);
    return true;
  }
  // dz (dz_chunk): entries 16 p .. + 15 of column j are pieces of four rows, piece q at rows 8 q + 4 (lane / 32) of 32;
  // pieces u and u + 2 are a lane's 16 bytes (u = 0, 1)
  static constexpr int PAIR = 2;
  __device__ __forceinline__ int64_t dz_at(int ldz, int n0, int m0, int j, int p, int u) const {
    return dz_chunk(ldz, (n0 >> 6) + wn, ((m0 + wm * 32 * MI) >> 5) + p, 2 * j + ((lane >> 4) & 1), 16 * (2 * u + (lane >> 5)) + (lane & 15));
  }
};
struct StripGeo {        // 192 x 256 tile of four waves (kd_strip.hpp)
  static constexpr int NC = StripCfg::NB, NE = StripCfg::MB * 4;
  static constexpr bool IN_LDS = true;
  int wave, lane;
  __device__ StripGeo() {
    lane = threadIdx.x & 63;
    wave = threadIdx.x >> 6;
  }
  __device__ __forceinline__ int m(int e) const { return StripCfg::acc_m(e >> 2, e & 3, lane); }
  __device__ __forceinline__ int n(int j) const { return StripCfg::acc_n(j, lane, wave); }
  template <int N, class Merge>
  __device__ __forceinline__ bool gather(float (&v)[N], char*, Merge&& merge) const {      // lanes 16 and 32 apart hold the same token
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
      float o[N];
#pragma unroll
      for (int i = 0; i < N; ++i) o[i] = __shfl_xor(v[i], off, 64);
      merge(v, o);
    }
    return lane < 16;
  }
  // dz (dz_chunk): entries 16 p .. + 15 of column j are four rows of each of four blocks; two neighbouring blocks are a
  // lane's 16 bytes, a wave's stores whole KiB
  static constexpr int PAIR = 1;
  __device__ __forceinline__ int64_t dz_at(int ldz, int n0, int m0, int j, int p, int u) const {
    return dz_chunk(ldz, (n0 >> 6) + wave, (m0 >> 5) + 2 * p + u, j, lane);
  }
};

struct AddUp {
  template <int N>
  __device__ __forceinline__ void operator()(float (&v)[N], const float (&o)[N]) const {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += o[i];
  }
};

// Drives an epilogue (template on the geometry, one column at a time) from tile_loop.
template <class Epi>
struct TileEpi {
  Epi& epi;
  float ts;
  __device__ TileEpi(Epi& e, float t_scale) : epi(e), ts(t_scale) {}
  __device__ void begin_item(const WorkItem& it) { epi.begin_item(it.m0, it.n0, BM); }
  __device__ void end_item(const WorkItem& it, AccTile& accS, AccTile& accT) {
    if (ts != 1.f) {     // fp8 teacher: the accumulator holds the product of the e4m3 codes; bring it to logits
#pragma unroll
      for (int mt = 0; mt < MI; ++mt)
#pragma unroll
        for (int nt = 0; nt < NI; ++nt)
#pragma unroll
          for (int r = 0; r < 16; ++r) accT[mt][nt][r] *= ts;
    }
    // Rows of A beyond the vocabulary (last tile only) must not contribute: give them a huge negative logit in
    // both accumulators (their exp is 0, their difference is 0).
    if (it.a_rows != BM) {
#pragma unroll
      for (int mt = 0; mt < MI; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool ok = epi.geo.m(16 * mt + r) < it.a_rows;
#pragma unroll
          for (int nt = 0; nt < NI; ++nt) {
            accS[mt][nt][r] = ok ? accS[mt][nt][r] : NEG_BIG;
            accT[mt][nt][r] = ok ? accT[mt][nt][r] : NEG_BIG;
          }
        }
    }
    static_for<0, NI>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      float S[TileGeo::NE], T[TileGeo::NE];
#pragma unroll
      for (int mt = 0; mt < MI; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) { S[16 * mt + r] = accS[mt][j][r]; T[16 * mt + r] = accT[mt][j][r]; }
      epi.column(jc, S, T);
    });
  }
};
// ... and from strip_loop.
template <class Epi>
struct StripEpi {
  static constexpr bool WHOLE = false;
  Epi& epi;
  __device__ StripEpi(Epi& e) : epi(e) {}
  __device__ void begin_item(const StripItem& it) { epi.begin_item(it.m0, it.n0, it.out_rows); }
  __device__ float pad(int) const { return NEG_BIG; }
  template <class J, int NM>
  __device__ __forceinline__ void column(const StripItem&, J jc, f32x4 (&S4)[NM], f32x4 (&T4)[NM]) {
    float S[4 * NM], T[4 * NM];
#pragma unroll
    for (int e = 0; e < 4 * NM; ++e) { S[e] = S4[e >> 2][e & 3]; T[e] = T4[e >> 2][e & 3]; }
    epi.column(jc, S, T);
  }
};

// Online log-sum-exp of both models plus the cross term of FKL / RKL.
//   FKL: X = sum_v 2^(a_t - m_t) (z_t - z_s)      RKL: X = sum_v 2^(a_s - m_s) (z_s - z_t)
template <int KIND>
struct StatsEpi {
  static constexpr int NV = KIND == 6 ? 6 : 5;     // values per token and part (AKL keeps both cross terms)
  static constexpr int NC = TileGeo::NC;
  TileGeo geo;
  float m_t[NC], S_t[NC], m_s[NC], S_s[NC], X[NC], X2[NC];
  float c;
  __device__ StatsEpi(float c_) : c(c_) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      m_t[j] = M_FLOOR; m_s[j] = M_FLOOR; S_t[j] = 0.f; S_s[j] = 0.f; X[j] = 0.f; X2[j] = 0.f;
    }
  }
  __device__ void begin_item(int, int, int) {}
  template <class J, int NE>
  __device__ __forceinline__ void column(J, const float (&S)[NE], const float (&T)[NE]) {
    constexpr int j = J::value;
    float tmax = NEG_BIG, smax = NEG_BIG;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      tmax = fmaxf(tmax, T[e]);
      smax = fmaxf(smax, S[e]);
    }
    const float nmt = fmaxf(m_t[j], tmax * c);
    const float nms = fmaxf(m_s[j], smax * c);
    const float sct = fexp2(m_t[j] - nmt);
    const float scs = fexp2(m_s[j] - nms);
    float st = S_t[j] * sct, ss = S_s[j] * scs;
    float x = X[j] * ((KIND == 0 || KIND == 6) ? sct : scs);
    float x2 = X2[j] * scs;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const float zt = T[e], zs = S[e];
      const float et = fexp2(fmaf(zt, c, -nmt));
      const float es = fexp2(fmaf(zs, c, -nms));
      st += et;
      ss += es;
      if (KIND == 0 || KIND == 6) x = fmaf(et, zt - zs, x);
      if (KIND == 1) x = fmaf(es, zs - zt, x);
      if (KIND == 6) x2 = fmaf(es, zs - zt, x2);
    }
    m_t[j] = nmt; m_s[j] = nms; S_t[j] = st; S_s[j] = ss; X[j] = x; X2[j] = x2;
  }
  __device__ void write(const LogitArgs& a, char* smem, int tt, int split) {
    float v[NC * NV];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const float own[6] = {m_t[j], S_t[j], m_s[j], S_s[j], X[j], X2[j]};
#pragma unroll
      for (int i = 0; i < NV; ++i) v[NV * j + i] = own[i];
    }
    const bool mine = geo.gather(v, smem, [](float (&v)[NC * NV], const float (&o)[NC * NV]) {
#pragma unroll
      for (int j = 0; j < NC * NV; j += NV) {
        const float mt = fmaxf(v[j], o[j]), ms = fmaxf(v[j + 2], o[j + 2]);
        const float vt = fexp2(v[j] - mt), ot = fexp2(o[j] - mt), vs = fexp2(v[j + 2] - ms), os = fexp2(o[j + 2] - ms);
        v[j] = mt; v[j + 2] = ms;
        v[j + 1] = fmaf(v[j + 1], vt, o[j + 1] * ot);
        v[j + 3] = fmaf(v[j + 3], vs, o[j + 3] * os);
        v[j + 4] = KIND == 1 ? fmaf(v[j + 4], vs, o[j + 4] * os) : fmaf(v[j + 4], vt, o[j + 4] * ot);
        if constexpr (NV == 6) v[j + 5] = fmaf(v[j + 5], vs, o[j + 5] * os);
      }
    });
    if (!mine) return;
    float* const p = a.partials + (int64_t)split * NV * a.T_pad + tt * BN;
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int i = 0; i < NV; ++i) p[(int64_t)i * a.T_pad + geo.n(j)] = v[NV * j + i];
  }
};

// The same on the strip loop, whose lanes have no registers for what lasts from tile to tile: 20 of them, held by every lane for
// its own rows, were spilled to memory, and each reload waited for every load in flight, four times a tile.  They live in LDS,
// [token][8], one copy for the four lanes of a token, which merge what a tile adds to them; a token belongs to one wave, so there is
// no barrier.  T = 4096, V = 151936, H = 4096 / 1024: statistics 4.33 -> 4.16 ms; with the gradient kernels' rows there, too, a step of
// T = 4096 1.057 -> 1.062 (JSD 1.070) times the speed of the same earlier state, forward pass alone at T = 1003 1.004 -> 1.022.
__device__ __forceinline__ float quad_max(float x) {          // over the lanes of a token, 16 and 32 apart
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float quad_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
template <int KIND>
struct StripStatsEpi {
  static constexpr int NV = KIND == 6 ? 6 : 5;
  StripGeo geo;
  float* state;            // m_t, S_t, m_s, S_s, X, X2 of this lane's token of column 0
  float c;
  __device__ StripStatsEpi(float c_, char* smem) : c(c_) {
    float* const all = (float*)(smem + StripCfg::STATE_AT);
    float* const own = all + threadIdx.x * 8;                 // (thread i: token i of the tile, its wave's)
    *(f32x4*)own = f32x4{M_FLOOR, 0.f, M_FLOOR, 0.f};
    own[4] = own[5] = 0.f;
    state = all + geo.n(0) * 8;
  }
  __device__ void begin_item(int, int, int) {}
  template <class J, int NE>
  __device__ __forceinline__ void column(J, const float (&S)[NE], const float (&T)[NE]) {
    constexpr int j = J::value;
    float* const at = state + 16 * 8 * j;
    const f32x4 old = *(const f32x4*)at;
    float tmax = NEG_BIG, smax = NEG_BIG;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      tmax = fmaxf(tmax, T[e]);
      smax = fmaxf(smax, S[e]);
    }
    const float nmt = fmaxf(old[0], quad_max(tmax) * c);
    const float nms = fmaxf(old[2], quad_max(smax) * c);
    float st = 0.f, ss = 0.f, x = 0.f, x2 = 0.f;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const float zt = T[e], zs = S[e];
      const float et = fexp2(fmaf(zt, c, -nmt));
      const float es = fexp2(fmaf(zs, c, -nms));
      st += et;
      ss += es;
      if (KIND == 0 || KIND == 6) x = fmaf(et, zt - zs, x);
      if (KIND == 1) x = fmaf(es, zs - zt, x);
      if (KIND == 6) x2 = fmaf(es, zs - zt, x2);
    }
    const float sct = fexp2(old[0] - nmt), scs = fexp2(old[2] - nms);
    *(f32x4*)at = f32x4{nmt, fmaf(old[1], sct, quad_sum(st)), nms, fmaf(old[3], scs, quad_sum(ss))};
    if (KIND != 2) at[4] = fmaf(at[4], KIND == 1 ? scs : sct, quad_sum(x));
    if (KIND == 6) at[5] = fmaf(at[5], scs, quad_sum(x2));
  }
  __device__ void write(const LogitArgs& a, char* smem, int tt, int split) {
    const float* const own = (const float*)(smem + StripCfg::STATE_AT) + threadIdx.x * 8;
    float* p = a.partials + (int64_t)split * NV * a.T_pad + tt * BN + threadIdx.x;
#pragma unroll
    for (int i = 0; i < NV; ++i) p[(int64_t)i * a.T_pad] = own[i];
  }
};

// Divergences whose row value needs both log-sum-exps first (JSD, TVD, skewed KL) share one
// scheme.  With D a function of the student probabilities and c = dD/dp_s, the gradient through the
// softmax is  dD/dz_s = p_s (c - R) / tau,  R = sum_v p_s c.  A row pass over the logit tiles
// accumulates two sums (a1, a2) per token, from which the row loss and R follow; the gradient pass
// evaluates c element by element.  lt, ls are base-2 log-probabilities, w is beta (JSD) or the skew
// weight alpha.
//   JSD       M = w p_t + (1-w) p_s    a1 = sum p_t (lt - lm)   a2 = sum p_s (ls - lm)
//             loss = ln2 (w a1 + (1-w) a2)     c = (1-w) ln2 (ls - lm)          R = (1-w) ln2 a2
//   TVD       d = p_s - p_t            a1 = sum |d|             a2 = sum p_s sign(d)
//             loss = a1 / 2                    c = sign(d) / 2                  R = a2 / 2
//   skew FKL  M = w p_t + (1-w) p_s    a1 = sum p_t (lt - lm)   a2 = sum p_s p_t / M
//             loss = ln2 a1                    c = -(1-w) p_t / M               R = -(1-w) a2
//   skew RKL  M = (1-w) p_t + w p_s    a1 = sum p_s (ls - lm)   a2 = sum p_s c
//             loss = ln2 a1                    c = ln2 (ls - lm) + 1 - w p_s / M   R = a2
template <int KIND>
struct RowTerm {
  // c for one element; also adds the element's contribution to (a1, a2) when ACC is set
  template <bool ACC>
  static __device__ __forceinline__ float eval(float lt, float ls, float w, float& a1, float& a2) {
    const float pt = fexp2(lt), ps = fexp2(ls);
    if (KIND == 3) {
      const float d = ps - pt;
      const float sg = (d > 0.f ? 1.f : 0.f) - (d < 0.f ? 1.f : 0.f);
      if (ACC) { a1 += fabsf(d); a2 = fmaf(ps, sg, a2); }
      return 0.5f * sg;
    }
    const float wt = (KIND == 5) ? 1.f - w : w;          // weight of p_t in the mixture
    // log M is taken relative to the larger of the two probabilities: with d = ls - lt and q = 2^-|d| <= 1,
    //   p_t >= p_s:  M / p_t = wt + (1-wt) q      p_t < p_s:  M / p_s = wt q + (1-wt)
    // so the logarithm's argument lies in [min(wt, 1-wt), 1]: no large logarithms are subtracted from one
    // another (the hardware log of M itself, of size log2 V, is half an ulp short on average, which
    // showed as a bias of 3e-7 in small losses), and nothing degenerates where p_t and p_s underflow.
    const float d = ls - lt;
    const bool t_big = d <= 0.f;
    const float q = fexp2(t_big ? d : -d);
    const float mix = t_big ? fmaf(1.f - wt, q, wt) : fmaf(wt, q, 1.f - wt);
    const float lmix = flog2(mix);
    const float lt_lm = t_big ? -lmix : -d - lmix;       // lt - lm
    const float ls_lm = t_big ? d - lmix : -lmix;        // ls - lm
    const float inv = __builtin_amdgcn_rcpf(mix);
    if (KIND == 2) {
      if (ACC) { a1 = fmaf(pt, lt_lm, a1); a2 = fmaf(ps, ls_lm, a2); }
      return (1.f - w) * LN2 * ls_lm;
    }
    if (KIND == 4) {
      const float r = t_big ? inv : q * inv;             // p_t / M
      if (ACC) { a1 = fmaf(pt, lt_lm, a1); a2 = fmaf(ps, r, a2); }
      return -(1.f - w) * r;
    }
    const float r = t_big ? q * inv : inv;               // p_s / M
    const float cc = fmaf(LN2, ls_lm, 1.f - w * r);
    if (ACC) { a1 = fmaf(ps, ls_lm, a1); a2 = fmaf(ps, cc, a2); }
    return cc;
  }
};

// AKL (KIND 6) uses the same pass for its gaps:  a1 = sum over the head of |p_t - p_s|,  a2 = the same over
// the tail, the head being the entries whose teacher log-probability reaches the token's threshold.
template <int KIND, class Geo>
struct RowsEpi {
  static constexpr int NC = Geo::NC;
  Geo geo;
  float A1[NC], A2[NC], Lt[NC], Ls[NC], Thr[NC];
  float c, w;
  __device__ RowsEpi(const LogitArgs& a, int tt) : c(a.c), w(a.beta) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int t = tt * BN + geo.n(j);
      const f32x4 ri = a.rowinfo[t];
      Lt[j] = ri[0]; Ls[j] = ri[1]; A1[j] = 0.f; A2[j] = 0.f;
      Thr[j] = 0.f;
      if (KIND == 6)    // the top entry is head whatever its mass
        Thr[j] = fminf(a.akl[AKL_HI * a.T_pad + t], a.akl[AKL_LTMAX * a.T_pad + t] - AKL_TOP_EPS);
    }
  }
  __device__ void begin_item(int, int, int) {}
  template <class J, int NE>
  __device__ __forceinline__ void column(J, const float (&S)[NE], const float (&T)[NE]) {
    constexpr int j = J::value;
    float a1 = A1[j], a2 = A2[j];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const float lt = fmaf(T[e], c, -Lt[j]);
      const float ls = fmaf(S[e], c, -Ls[j]);
      if constexpr (KIND == 6) {
        const float gap = fabsf(fexp2(lt) - fexp2(ls));
        const bool head = lt >= Thr[j];
        a1 += head ? gap : 0.f;
        a2 += head ? 0.f : gap;
      } else {
        (void)RowTerm<KIND>::template eval<true>(lt, ls, w, a1, a2);
      }
    }
    A1[j] = a1; A2[j] = a2;
  }
  __device__ void write(const LogitArgs& a, char* smem, int tt, int split) {
    float v[2 * NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) { v[2 * j] = A1[j]; v[2 * j + 1] = A2[j]; }
    if (!geo.gather(v, smem, AddUp())) return;
    float* const p = a.partials + (int64_t)split * 2 * a.T_pad + tt * BN;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      p[geo.n(j)] = v[2 * j];
      p[a.T_pad + geo.n(j)] = v[2 * j + 1];
    }
  }
};

// dL/dz_s tile.  rowinfo = {lse2_t, lse2_s, s = mask/(n tau), R}
//   FKL: dz = s (p_s - p_t)
//   RKL: dz = s p_s (ln2 (l_s - l_t) - R),   R = row loss
//   JSD, TVD, skewed KL: dz = s p_s (c - R)  (RowTerm above)
//   AKL: dz = s (w_f (p_s - p_t) + w_r p_s (ln2 (l_s - l_t) - RKL)) = s (p_s (w_r ln2 (l_s - l_t) + R) - w_f p_t),
//        R = w_f - w_r RKL, the weights being constants for the gradient
// Vocabulary entries that do not exist carry the logit NEG_BIG in both models: their dz comes out 0 in every
// kind, and that is what the chunk buffer holds from its last valid column to the end of a 64-column step.
template <int KIND, class Geo>
struct GradEpi {
  static constexpr int NC = Geo::NC;
  Geo geo;
  const LogitArgs& a;
  // Of the lane's tokens, in registers; on the strip loop, which has none for them (spills whose reloads waited for every load in
  // flight, at the start of each phase), in LDS, [token] of rowinfo and behind them [token] of w_r.  A token belongs to one
  // wave, and a workgroup stays with its token tile but for a few changes.
  float Lt[Geo::IN_LDS ? 1 : NC], Ls[Geo::IN_LDS ? 1 : NC], sc[Geo::IN_LDS ? 1 : NC], R[Geo::IN_LDS ? 1 : NC], Wr[Geo::IN_LDS ? 1 : NC];
  f32x4* info;
  int m0, n0, out_rows;
  __device__ GradEpi(const LogitArgs& a_, char* smem) : a(a_), n0(-1) {
    info = (f32x4*)(smem + (Geo::IN_LDS ? StripCfg::STATE_AT : 0));
  }
  __device__ void begin_item(int m0_, int n0_, int out_rows_) {
    out_rows = out_rows_;
    m0 = m0_ - a.v0;                           // vocabulary offset inside the chunk
    if constexpr (Geo::IN_LDS) {
      if (n0 != n0_) {
        info[threadIdx.x] = a.rowinfo[n0_ + threadIdx.x];
        if (KIND == 6) ((float*)(info + BN))[threadIdx.x] = a.akl[AKL_WR * a.T_pad + n0_ + threadIdx.x];
      }
      n0 = n0_;
      return;
    }
    n0 = n0_;
#pragma unroll
    for (int j = 0; j < (Geo::IN_LDS ? 0 : NC); ++j) {
      const f32x4 ri = a.rowinfo[n0 + geo.n(j)];
      Lt[j] = ri[0]; Ls[j] = ri[1]; sc[j] = ri[2]; R[j] = ri[3];
      Wr[j] = 0.f;
      if (KIND == 6) Wr[j] = a.akl[AKL_WR * a.T_pad + n0 + geo.n(j)];
    }
  }
  template <bool ADD, class J, int NE>
  __device__ __forceinline__ void emit(J, const float (&S)[NE], const float (&T)[NE]) {
    constexpr int j = J::value;
    const float c = a.c, w = a.beta;
    float Lt_, Ls_, s, R_, Wr_ = 0.f;
    if constexpr (Geo::IN_LDS) {
      const f32x4 ri = info[geo.n(j)];
      Lt_ = ri[0]; Ls_ = ri[1]; s = ri[2]; R_ = ri[3];
      if (KIND == 6) Wr_ = ((const float*)(info + BN))[geo.n(j)];
    } else {
      Lt_ = Lt[j]; Ls_ = Ls[j]; s = sc[j]; R_ = R[j]; Wr_ = Wr[j];
    }
#pragma unroll
    for (int p = 0; p < NE / 16; ++p) {
      bf16x4 o[4];
      if (64 * p >= out_rows) break;             // (whole entries of 64 rows: only the strip loop's last tile has fewer)
      if (ADD)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const bf16x8 v = *(const bf16x8*)(a.dz + geo.dz_at(a.ldz, n0, m0, j, p, u));
          o[Geo::PAIR == 1 ? 2 * u : u] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
          o[Geo::PAIR == 1 ? 2 * u + 1 : u + 2] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
        }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        // (KIND 5 has finite gradients beside teacher entries at minus infinity.  The rest of the last token tile are tokens of zeros,
        // whose entries there are 0 x infinity, NaN, and would stay NaN in 0 x g: this gives the number.  A token that counts and has a
        // NaN keeps it through R.  The last valid token again instead of zeros, which cost no energy, is slower everywhere: T = 4096
        // 10290 -> 10337 us, evaluation at T = 1003 1193 -> 1220.)
        const float lt = KIND == 5 ? fmaxf(fmaf(T[16 * p + e], c, -Lt_), -1.0e38f) : fmaf(T[16 * p + e], c, -Lt_);
        const float ls = fmaf(S[16 * p + e], c, -Ls_);
        const float ps = fexp2(ls);
        float g;
        if (KIND == 0) {
          g = ps - fexp2(lt);
        } else if (KIND == 1) {
          g = ps * fmaf(LN2, ls - lt, -R_);
        } else if (KIND == 6) {
          g = fmaf(ps, fmaf(Wr_ * LN2, ls - lt, R_), -(1.f - Wr_) * fexp2(lt));
        } else {
          float u1, u2;
          g = ps * (RowTerm<KIND>::template eval<false>(lt, ls, w, u1, u2) - R_);
        }
        const float d = s * g;
        o[e >> 2][e & 3] = (bf16_t)(ADD ? (float)o[e >> 2][e & 3] + d : d);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
        *(bf16x8*)(a.dz + geo.dz_at(a.ldz, n0, m0, j, p, u)) =
            __builtin_shufflevector(o[Geo::PAIR == 1 ? 2 * u : u], o[Geo::PAIR == 1 ? 2 * u + 1 : u + 2], 0, 1, 2, 3, 4, 5, 6, 7);
      __builtin_amdgcn_sched_barrier(0);       // (or all of a column is computed before anything is stored: spills)
    }
  }
  // (two bodies: a shared one would wait for the loads of the adding one, and for everything older, on both paths)
  template <class J, int NE>
  __device__ __forceinline__ void column(J jc, const float (&S)[NE], const float (&T)[NE]) {
    if (a.dz_accumulate) emit<true>(jc, S, T);
    else emit<false>(jc, S, T);
  }
};

// AKL threshold search on the eight-wave loop, one pass: for AKL_K thresholds spread evenly inside the token's current interval
// (LO, HI), the teacher mass of the entries at or above each threshold.
template <class Geo>
struct SearchEpi {
  static constexpr int NC = Geo::NC;
  Geo geo;
  float Lt[NC], th0[NC], step[NC];
  float mass[NC * AKL_K];
  float c;
  __device__ SearchEpi(const LogitArgs& a, int tt) : c(a.c) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int t = tt * BN + geo.n(j);
      Lt[j] = a.rowinfo[t][0];
      const float lo = a.akl[AKL_LO * a.T_pad + t], hi = a.akl[AKL_HI * a.T_pad + t];
      step[j] = (hi - lo) * (1.f / (AKL_K + 1));
      th0[j] = lo + step[j];
#pragma unroll
      for (int k = 0; k < AKL_K; ++k) mass[AKL_K * j + k] = 0.f;
    }
  }
  __device__ void begin_item(int, int, int) {}
  // T alone: the teacher's logits (entries that do not exist are NEG_BIG: below every threshold)
  template <class J, int NE>
  __device__ __forceinline__ void column(J, const float (&)[NE], const float (&T)[NE]) {
    constexpr int j = J::value;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const float lt = fmaf(T[e], c, -Lt[j]);
      const float p = fexp2(lt);
#pragma unroll
      for (int k = 0; k < AKL_K; ++k) mass[AKL_K * j + k] += (lt >= fmaf((float)k, step[j], th0[j])) ? p : 0.f;
    }
  }
  __device__ void write(const LogitArgs& a, char* smem, int tt, int split) {
    if (!geo.gather(mass, smem, AddUp())) return;
    float* const p = a.partials + (int64_t)split * AKL_K * a.T_pad + tt * BN;
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int k = 0; k < AKL_K; ++k) p[(int64_t)k * a.T_pad + geo.n(j)] = mass[AKL_K * j + k];
  }
};

// ... and on the strip loop, which has one accumulator here and so LDS to spare: the mass of the entries inside the interval by
// AKL_BINS bins in LDS, [bin][token].  What lies above the interval is known from the pass before.  A token belongs to one wave: no
// barrier.  Its four lanes may meet in one bin, and in no stated order, so the sums are whole numbers, of units of 2^-56: the same
// in any order.  (An entry loses less than a unit: 2^-32 in all at 2^24 entries, where a sum in fp32 is 2^-25 off by its last addition
// alone.)
// A compare, a select and an addition for each of 16 thresholds were 52 instructions per logit, 0.4 of the time that its MFMAs take
// and hidden by nothing; a bin takes 21, and past the first pass hardly any entry lies in the interval.
struct BinsEpi {
  static constexpr int NC = StripGeo::NC;
  static constexpr int BINS_AT = StripCfg::NST * StripCfg::STAGE_BYTES;      // in LDS, where other passes park student blocks
  static constexpr int SMEM_BYTES = BINS_AT + AKL_BINS * BN * 8;
  static_assert(SMEM_BYTES <= 160 * 1024, "LDS of a gfx950 CU");
  static constexpr float FIRST = 0x1p24f, SECOND = 0x1p32f, UNIT = 0x1p-56f;       // upper and lower word of a mass in units
  StripGeo geo;
  float Lt[NC], low[NC], cell[NC];             // of the lane's tokens: log-sum-exp and grid; the first cell above the lowest bin,
  float above[NC], first[NC], scale[NC];       // the lowest bin's lower edge, bins per unit of log-probability
  uint64_t* bins;          // of this lane's token of column 0
  // (The atomic is inline assembly: in front of the compiler's stands a wait for the loads into LDS, which it might alias
  // (4 % of the search).  The strip loop's prologue and its end order it against the bins' first and last accesses.)
  uint32_t bins_lds;
  float c, width;
  __device__ BinsEpi(const LogitArgs& a, int tt, char* smem) : c(a.c), width(a.akl_width) {
    bins = (uint64_t*)(smem + BINS_AT) + geo.n(0);
    bins_lds = (uint32_t)(uintptr_t)(lds_void_t*)bins;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int t = tt * BN + geo.n(j);
      Lt[j] = a.rowinfo[t][0];
      low[j] = a.akl[AKL_HI * a.T_pad + t];
      cell[j] = akl_cell(low[j], a.akl[AKL_LTMAX * a.T_pad + t]);
      const float lo = a.akl[AKL_LO * a.T_pad + t];
      first[j] = akl_edge(lo, low[j], cell[j]);
      above[j] = lo + width;
      scale[j] = 1.f / (width * cell[j]);
    }
    for (int k = geo.lane >> 4; k < AKL_BINS; k += 4)
#pragma unroll
      for (int j = 0; j < NC; ++j) bins[k * BN + 16 * j] = 0;
  }
  __device__ void begin_item(int, int, int) {}
  // T alone: the teacher's logits (entries that do not exist are NEG_BIG: below the interval).
  // k: floor of the entry's place in units of bins, less 1/4: more than its rounding in the narrowest bins (edges of size 24 are
  // 1e-6 off, a tenth of the smallest cell), so it is the bin's number or one less, and the comparison with the edge above says which.
  template <class J, int NE>
  __device__ __forceinline__ void column(J, const float (&)[NE], const float (&T)[NE]) {
    constexpr int j = J::value;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const float lt = fmaf(T[e], c, -Lt[j]);
      float k = floorf(fmaf(lt - first[j], scale[j], -0.25f));
      if (lt >= akl_edge(fmaf(k, width, above[j]), low[j], cell[j])) k += 1.f;
      if (k >= 0.f && k < (float)AKL_BINS) {
        const uint32_t at = bins_lds + (uint32_t)k * (BN * 8);
        const float p = fexp2(lt) * FIRST;
        const uint32_t hi = (uint32_t)p, lo = (uint32_t)((p - (float)hi) * SECOND);
        asm volatile("ds_add_u64 %0, %1 offset:%2" ::"v"(at), "v"((uint64_t)hi << 32 | lo), "n"(128 * j));
      }
    }
  }
  __device__ void write(const LogitArgs& a, int tt, int split) {
    float* p = a.partials + (int64_t)split * AKL_BINS * a.T_pad + tt * BN + geo.n(0);
    for (int k = geo.lane >> 4; k < AKL_BINS; k += 4)
#pragma unroll
      for (int j = 0; j < NC; ++j) p[(int64_t)k * a.T_pad + 16 * j] = (float)bins[k * BN + 16 * j] * UNIT;
  }
};

// AKL's row pass on the strip loop.  The search has left an interval of AKL_BINS cells per token, which hardly any entry lies in
// (tens of 150000), so this pass finds the border's cell by itself, where a third search pass took a seventh of a step (T = 2048, H = 4096 /
// 1024, V = 151936: a step 14.32 -> 12.47 ms, this pass 2.31 -> 2.54): the gaps above and below the interval are summed as ever, an entry inside adds its mass and its gap to its
// cell in memory, and the merge takes the cells up to the border to the tail.  Those sums are whole numbers, as the search's are, so
// their order does not matter.  What a token needs lies in LDS, [token][8], like the state of the statistics.
// A token tile in which a token has too many entries in the interval (AKL_CROWD: equal logits would meet in one word) goes through a
// third search pass first: its interval is empty here and AKL_HI the border.
struct AklRowsEpi {
  static constexpr int NC = StripGeo::NC;
  StripGeo geo;
  float* state;            // Lt, Ls, upper edge, first cell, lowest edge, largest log-probability, sums above and below; of the lane's
                           // token of column 0
  unsigned long long* fine;
  float c;
  __device__ AklRowsEpi(const LogitArgs& a, int tt, bool crowded, char* smem) : c(a.c) {
    float* const all = (float*)(smem + StripCfg::STATE_AT);
    float* const own = all + threadIdx.x * 8;                 // (thread i: token i of the tile, its wave's)
    const int t = tt * BN + threadIdx.x;
    const f32x4 ri = a.rowinfo[t];
    const float hi = a.akl[AKL_HI * a.T_pad + t], lo = a.akl[AKL_LO * a.T_pad + t], ltmax = a.akl[AKL_LTMAX * a.T_pad + t];
    own[0] = ri[0]; own[1] = ri[1];
    own[2] = crowded ? fminf(hi, ltmax - AKL_TOP_EPS) : akl_edge(lo + AKL_BINS, hi, akl_cell(hi, ltmax));
    own[3] = crowded ? 0.f : lo;
    own[4] = crowded ? own[2] : hi;                           // (crowded: the first cell's lower edge is the border, too)
    own[5] = ltmax;
    own[6] = own[7] = 0.f;
    state = all + geo.n(0) * 8;
    fine = a.akl_fine + (int64_t)(tt * BN + geo.n(0)) * AKL_BINS * 2;
  }
  __device__ void begin_item(int, int, int) {}
  static __device__ __forceinline__ unsigned long long units(float x) {        // of 2^-56
    const float p = x * 0x1p24f;
    const uint32_t hi = (uint32_t)p, lo = (uint32_t)((p - (float)hi) * 0x1p32f);
    return (unsigned long long)hi << 32 | lo;
  }
  template <class J, int NE>
  __device__ __forceinline__ void column(J, const float (&S)[NE], const float (&T)[NE]) {
    constexpr int j = J::value;
    float* const at = state + 16 * 8 * j;
    const f32x4 own = *(const f32x4*)at;
    const float low = at[4], ltmax = at[5], cell = akl_cell(low, ltmax), first = akl_edge(own[3], low, cell);
    float a1 = 0.f, a2 = 0.f;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const float lt = fmaf(T[e], c, -own[0]), pt = fexp2(lt);
      const float gap = fabsf(pt - fexp2(fmaf(S[e], c, -own[1])));
      const bool above = lt >= own[2], below = lt < first;
      a1 = fmaf((float)above, gap, a1);
      a2 = fmaf((float)below, gap, a2);
      asm volatile("" : "+v"(a1), "+v"(a2));                  // (or all the column's comparisons are kept for sums at its end)
      // (One branch an entry and no other: past 1100 blocks the compiler stops inlining, and the loop's state goes to memory.)
      if (!(above | below)) {
        // (its cell's number or one less, and the comparison with the edge above says which: see BinsEpi)
        float k = fmaxf(floorf(fmaf(lt - first, __builtin_amdgcn_rcpf(cell), -0.25f)), 0.f);
        k = fminf(k + (float)(lt >= akl_edge(own[3] + k + 1.f, low, cell)), (float)(AKL_BINS - 1));
        unsigned long long* const to = fine + (16 * j * AKL_BINS + (int)k) * 2;
        const float head = (float)(lt >= ltmax - AKL_TOP_EPS) * gap;          // the top entry, whatever its mass, which counts in its cell
        a1 += head;
        __hip_atomic_fetch_add(to, units(pt), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(to + 1, units(gap - head), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    at[6] += quad_sum(a1);
    at[7] += quad_sum(a2);
  }
  __device__ void write(const LogitArgs& a, char* smem, int tt, int split) {
    const float* const own = (const float*)(smem + StripCfg::STATE_AT) + threadIdx.x * 8;
    float* p = a.partials + (int64_t)split * 2 * a.T_pad + tt * BN + threadIdx.x;
    p[0] = own[6];
    p[a.T_pad] = own[7];
  }
};
// Whether a token of tile tt is crowded (AklRowsEpi); every wave asks for itself.
__device__ __forceinline__ bool akl_crowded(const float* akl, int T_pad, int tt) {
  const f32x4 v = *(const f32x4*)(akl + (int64_t)AKL_CROWD * T_pad + tt * BN + 4 * (threadIdx.x & 63));
  return __ballot(v[0] != 0.f || v[1] != 0.f || v[2] != 0.f || v[3] != 0.f) != 0;
}

// measurement aid, off unless asked for
struct LoopClock {
  long long c0 = 0, r0 = 0;
  __device__ LoopClock(const LogitArgs& a) {
    if (a.clock_out) { c0 = clock64(); r0 = wall_clock64(); }
  }
  __device__ void stop(const LogitArgs& a) {
    if (a.clock_out && blockIdx.x == 0 && threadIdx.x == 0) {
      a.clock_out[0] = clock64() - c0;
      a.clock_out[1] = wall_clock64() - r0;
    }
  }
};

// ------------------------------------------------------------------------------------------
// launching
// ------------------------------------------------------------------------------------------
inline int largest_divisor_le(int n, int cap) {
  for (int d = cap; d > 1; --d)
    if (n % d == 0) return d;
  return 1;
}

inline LogitArgs make_logit_args(const Problem& p) {
  LogitArgs a{};
  a.W_s = (const bf16_t*)p.W_s; a.h_s = (const bf16_t*)p.h_s;
  a.W_t = (const bf16_t*)p.W_t; a.h_t = (const bf16_t*)p.h_t;
  a.T = p.T; a.V = p.V; a.H_s = p.K_s; a.H_t = p.K_t;
  a.ld_s = p.w_hv_inplace ? p.V : p.prep_Ws ? p.K_s : p.H_s;
  a.ld_t = p.w_hv_inplace ? p.V : p.prep_Wt ? p.K_t : p.H_t;
  a.meta = p.meta;
  a.c = 1.4426950408889634f / p.tau;
  a.beta = p.beta;
  a.t_scale = p.t_fp8 ? p.t_scale : 1.f;
  a.T_pad = p.T_pad;
  a.rowinfo = (const f32x4*)p.rowinfo;
  a.akl = p.akl;
  a.akl_fine = p.akl_fine;
  return a;
}
// The strip loop's kernels for heads kept as [H][V] (kd_strip_hv.hip), by the divergence of `p`.
hipError_t launch_strip_hv_stats(const Problem& p, const LogitArgs& a, int grid, hipStream_t st);
hipError_t launch_strip_hv_rows(const Problem& p, const LogitArgs& a, int grid, hipStream_t st);
hipError_t launch_strip_hv_grad(const Problem& p, const LogitArgs& a, int grid, hipStream_t st);
hipError_t launch_strip_hv_search(const LogitArgs& a, int grid, hipStream_t st);

// Those of the eight-wave loop for at most kFewTokens tokens (kd_few.hip): a pair of waves has 64 of the 256 tokens of a tile.
constexpr int kFewTokens = 192;
inline bool few_tokens(const Problem& p) { return !p.strip && p.T <= kFewTokens; }
hipError_t launch_few_stats(const Problem& p, const LogitArgs& a, int grid, hipStream_t st);
hipError_t launch_few_rows(const Problem& p, const LogitArgs& a, int grid, hipStream_t st);
hipError_t launch_few_grad(const Problem& p, const LogitArgs& a, int grid, hipStream_t st);
hipError_t launch_few_search(const Problem& p, const LogitArgs& a, int grid, hipStream_t st);

}  // namespace kd
