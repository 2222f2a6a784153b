// gfx950 kernels of libkdloss and their launchers.
//
// Pass structure (one call of kd_loss_fwd_bwd):
//   stats    : logit tiles (student then teacher) -> online max / sum-exp / cross term per token
//   combine  : merge partial statistics -> log-sum-exps, FKL / RKL row losses
//   rows     : (JSD, TVD, skewed KL, AKL) logit tiles again -> two row sums per token (RowTerm)
//   akl search : (AKL) teacher logit tiles only, a few times -> the teacher probability that splits head from tail
//   finalize : n = sum mask, loss, per-row gradient scale mask/(n tau)
//   per vocabulary chunk:
//     grad   : logit tiles again -> dL/dz_s tile in bf16, stored once in the order of dz_chunk (kd_common.hpp)
//     the backward products: grad_W_s[chunk] = dz^T . h_s     and     grad_h_s += dz . W_s[chunk]     (kd_products.hip)
//   gradh_finish : fp32 partial sums -> grad_h_s (kd_products.hip)
// All logarithms inside the kernels are base 2: a = z * log2(e)/tau.
#include "kd_eight.hpp"

namespace kd {

// ------------------------------------------------------------------------------------------
// logit kernels: the strip loop for bf16 operands where it is ahead (strips_ahead in kd_api.hip; heads read in place as
// [H][V]: kd_strip_hv.hip); the eight-wave tile loop for the others (k-major fragments come from LDS by transposing reads)
// and where the teacher is fp8
// ------------------------------------------------------------------------------------------
template <int KIND>
KD_STRIP_KERNEL void stats_strip_kernel(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  StripWork<false> work(a, meta_get(a.meta, META_N_SPLIT));
  StripStatsEpi<KIND> epi(a.c, smem);
  StripEpi<StripStatsEpi<KIND>> drive(epi);
  LoopClock clk(a);
  strip_loop<2, true>(work, drive, smem);
  clk.stop(a);
  if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
}

template <int KIND>
KD_STRIP_KERNEL void rows_strip_kernel(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  StripWork<false> work(a, meta_get(a.meta, META_N_SPLIT));
  if constexpr (KIND == 6) {
    AklRowsEpi epi(a, work.tt, akl_crowded(a.akl, a.T_pad, work.tt), smem);
    StripEpi<AklRowsEpi> drive(epi);
    strip_loop<2, true>(work, drive, smem);
    if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
  } else {
    RowsEpi<KIND, StripGeo> epi(a, work.tt);
    StripEpi<RowsEpi<KIND, StripGeo>> drive(epi);
    strip_loop<2, true>(work, drive, smem);
    if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
  }
}

KD_STRIP_KERNEL void akl_search_strip_kernel(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  StripWork<false> work(a, meta_get(a.meta, META_N_SPLIT));
  if (a.akl_width == 1.f && !akl_crowded(a.akl, a.T_pad, work.tt)) return;
  BinsEpi epi(a, work.tt, smem);
  StripEpi<BinsEpi> drive(epi);
  strip_loop<1, true>(work, drive, smem);
  if (work.cnt > 0) epi.write(a, work.tt, work.split);
}

template <int KIND>
KD_STRIP_KERNEL void grad_strip_kernel(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  StripWork<false> work(a, meta_get(a.meta, a.last_chunk ? META_G_SPLIT_LAST : META_G_SPLIT));
  GradEpi<KIND, StripGeo> epi(a, smem);
  StripEpi<GradEpi<KIND, StripGeo>> drive(epi);
  strip_loop<2, false>(work, drive, smem);
}

// ------------------------------------------------------------------------------------------
// small kernels
// ------------------------------------------------------------------------------------------

// One workgroup.  Compacts the valid tokens (mask != 0; all of them when mask is null) to the front:
// rowmap[j] = index of the j-th valid token, inv[t] = its compacted index or -1, and writes the
// device-side plan that depends on how many there are.  Every later kernel works on the compacted
// token axis, so masked tokens cost nothing.
//
// Vocabulary ranges per token tile: the number s that finishes soonest when ceil(n_tt s / n_cu) rounds of workgroups
// walk ceil(units / s) units each, in tiles of `per_tile` units and a rest.  A rest of at most `short_units` costs
// 0.45 of a tile, a workgroup 0.33 of one to fill and drain its pipeline; the fewest ranges among equals, and at
// least eight (the blocks of group_decode) where there are that many; 0 where striding over whole tiles
// (StripWork) is better.  29 token tiles x 128256 rows: 26 ranges in
// three rounds, where eight leave 24 of 256 CUs idle; one token tile x 151936 rows: 256 ranges of three tiles and at most
// a short one, where whole tiles would take four.
struct SplitChoice { int units, per_tile, short_units, most, strided; };
struct RowmapArgs {
  const uint8_t* mask;
  int T, T_pad, n_cu;
  SplitChoice stats, grad, grad_last;
  int *rowmap, *inv, *meta;
};
__device__ __forceinline__ void make_rowmap(const RowmapArgs& a) {
  const uint8_t* const mask = a.mask;
  const int T = a.T, T_pad = a.T_pad, n_cu = a.n_cu;
  int *const rowmap = a.rowmap, *const inv = a.inv, *const meta = a.meta;
  constexpr int PER = 4;                           // rows of 1024 tokens at a time
  __shared__ int s_wave[2][PER][16];               // valid tokens of each wave; two sets, so that one barrier a time does
  __shared__ unsigned long long s_best[3];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (tid < 3) s_best[tid] = ~0ull;
  // (Counted by ballots and sums over the waves; as a scan in LDS, twenty barriers per 1024 tokens, a step of T = 32768, H = 256 / 256, V = 8000
  // took 1072 us against 1045, T = 3000, H = 1024 / 512, V = 32000 670 / 663.)
  int n = 0;
  for (int base = 0, set = 0; base < T; base += 1024 * PER, set ^= 1) {
    unsigned long long on[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int t = base + 1024 * i + tid;
      on[i] = __ballot(t < T && (mask == nullptr || mask[t] != 0));
    }
    if (lane == 0)
#pragma unroll
      for (int i = 0; i < PER; ++i) s_wave[set][i][wave] = __popcll(on[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int t = base + 1024 * i + tid;
      int before = 0, all = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        const int c = s_wave[set][i][w];
        before += w < wave ? c : 0;
        all += c;
      }
      if (t < T) {
        const bool mine = on[i] >> lane & 1;
        const int j = n + before + __popcll(on[i] & ((1ull << lane) - 1));
        if (mine) rowmap[j] = t;
        inv[t] = mine ? j : -1;
      }
      n += all;
    }
  }
  __syncthreads();                                  // (the row map is read below, s_best is set)
  const int last = n > 0 ? rowmap[n - 1] : 0;
  __syncthreads();
  for (int j = n + tid; j < T_pad; j += 1024) rowmap[j] = last;   // never dereferenced for results
  const int n_tt = max((n + BN - 1) / BN, 1);
  if (const int k = tid >> 8; k < 3) {               // 256 threads per choice
    const SplitChoice c = k == 0 ? a.stats : k == 1 ? a.grad : a.grad_last;
    for (int sp = (tid & 255) + 1; sp <= c.most; sp += 256) {
      if (c.strided && sp == 1) {                    // (n_split 0; dearer by a hair: 2 % slower at equal counts)
        const int r = (n_tt * ((c.units + c.per_tile - 1) / c.per_tile) + n_cu - 1) / n_cu;
        atomicMin(&s_best[k], ((unsigned long long)(((float)r + 0.4f) * 16.f) << 16));
      }
      if (sp < 8 && sp < c.most) continue;
      const int rounds = (n_tt * sp + n_cu - 1) / n_cu, u = (c.units + sp - 1) / sp, rest = u % c.per_tile;
      const float tiles = (float)(u / c.per_tile) + (rest == 0 ? 0.f : rest <= c.short_units ? 0.45f : 1.f) + 0.33f;
      atomicMin(&s_best[k], ((unsigned long long)((float)rounds * tiles * 16.f) << 16) | (unsigned)sp);
    }
  }
  __syncthreads();
  if (tid == 0) {
    meta[META_N_VALID] = n;
    meta[META_N_TT] = n_tt;
    meta[META_T_EFF] = max((n + 63) / 64, 1) * 64;      // what grad_W_s contracts: whole k-steps (the rest of the tile is 0)
    meta[META_N_SPLIT] = (int)(s_best[0] & 0xffff);
    meta[META_G_SPLIT] = (int)(s_best[1] & 0xffff);
    meta[META_G_SPLIT_LAST] = (int)(s_best[2] & 0xffff);
  }
}

// Merging the partial sums.  Every workgroup (one per token tile and vocabulary range) leaves its values as [range][value][T_pad], and
// with few tokens there are many ranges (256 at T <= 256; the eight-wave loop's four lanes of a token put theirs
// together first: a step of T = 200, H = 2048 / 512, V = 32000 148 -> 133 us, AKL at T = 150, H = 1024 / 512 347 -> 291).  A merge is bound by the latency of its loads:
// one thread walking all the parts of a token took 658 us at T = 256 and 47 us at T = 4096.  So a workgroup owns TX
// tokens and NT / TX threads share the parts of each: lanes run along the tokens (TX = 8: 32-byte runs, TX = 32:
// whole lines), the rest of the lanes and the waves along the parts; partial results meet by shuffles, then through
// LDS, in a fixed order.  Measured: combine_kernel 658 -> 23 us at T = 256, 47 -> 9 us at 128 parts, 6 us at 32 (T = 4096),
// one search merge of AKL 536 -> 15 us at T = 2048.
struct MergeSum {
  static __device__ __forceinline__ float op(float a, float b) { return a + b; }
};
struct MergeMax {
  static __device__ __forceinline__ float op(float a, float b) { return fmaxf(a, b); }
};
// v[i] of every thread -> the merged value of the thread's token, in every thread of that token
template <int TX, int NT, int NV, class Op>
__device__ __forceinline__ void merge_parts(float (&v)[NV], float* lds) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tx = lane % TX;
#pragma unroll
  for (int off = TX; off < 64; off <<= 1)
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = Op::op(v[i], __shfl_xor(v[i], off, 64));
  __syncthreads();                       // the values of an earlier merge have been read
  if (lane < TX)
#pragma unroll
    for (int i = 0; i < NV; ++i) lds[(wave * NV + i) * TX + tx] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    float r = lds[i * TX + tx];
#pragma unroll
    for (int w = 1; w < NW; ++w) r = Op::op(r, lds[(w * NV + i) * TX + tx]);
    v[i] = r;
  }
}

// Merge the partial statistics of one (compacted) token; write log-sum-exps and, for FKL / RKL, the
// row loss.
template <int TX, int NT>
__global__ __launch_bounds__(NT) void combine_kernel(const float* partials, const int* meta, int T_pad, int kind, int strip, float c, float least,
                                                     f32x4* rowinfo, float* row_loss, float* akl) {
  __shared__ float lds[NT / 64 * 4 * TX];
  const int t = blockIdx.x * TX + threadIdx.x % TX, g = threadIdx.x / TX;
  const int n_valid = meta[META_N_VALID], n_parts = meta[META_N_SPLIT];
  const int nv = kind == 6 ? 6 : 5;
  if ((int)(blockIdx.x * TX) >= n_valid && g > 0) return;     // a whole workgroup of padding rows
  if (t >= n_valid && g == 0) {   // padding rows: probabilities evaluate to 0, gradient scale 0
    rowinfo[t] = f32x4{1.0e30f, 1.0e30f, 0.f, 0.f};
    row_loss[t] = 0.f;
    if (kind == 6)
      for (int i = 0; i < AKL_ROWS; ++i) akl[i * T_pad + t] = 0.f;
  }
  if ((int)(blockIdx.x * TX) >= n_valid) return;
  const int64_t stride = (int64_t)nv * T_pad;
  const float* const q0 = partials + t;          // t < T_pad: allocated, whatever the row holds
  float m[2] = {M_FLOOR, M_FLOOR};
#pragma unroll 4
  for (int p = g; p < n_parts; p += NT / TX) {
    m[0] = fmaxf(m[0], q0[p * stride]);
    m[1] = fmaxf(m[1], q0[p * stride + 2 * T_pad]);
  }
  merge_parts<TX, NT, 2, MergeMax>(m, lds);
  const float Mt = m[0], Ms = m[1];
  float v[4] = {0.f, 0.f, 0.f, 0.f};             // S_t, S_s, X, X2
#pragma unroll 4
  for (int p = g; p < n_parts; p += NT / TX) {
    const float* q = q0 + p * stride;
    const float wt = fexp2(q[0] - Mt), ws = fexp2(q[2 * T_pad] - Ms);
    v[0] = fmaf(q[1 * T_pad], wt, v[0]);
    v[1] = fmaf(q[3 * T_pad], ws, v[1]);
    v[2] = fmaf(q[4 * T_pad], (kind == 0 || kind == 6) ? wt : ws, v[2]);
    if (kind == 6) v[3] = fmaf(q[5 * T_pad], ws, v[3]);
  }
  merge_parts<TX, NT, 4, MergeSum>(v, lds);
  if (g != 0 || t >= n_valid) return;
  const float St = v[0], Ss = v[1], X = v[2], X2 = v[3];
  // The row loss is a difference of quantities of size log2 V, far larger than itself when the two
  // distributions are close: this last step is done in double (one thread per token, so it costs nothing).
  const double Ltd = (double)Mt + log2((double)St), Lsd = (double)Ms + log2((double)Ss);
  double lossd = 0.0;
  if (kind == 0) lossd = (double)c * X / St - Ltd + Lsd;   // kinds >= 2: filled in by combine_rows_kernel
  if (kind == 1) lossd = (double)c * X / Ss - Lsd + Ltd;
  const float loss = (float)(0.6931471805599453 * lossd);
  rowinfo[t] = f32x4{(float)Ltd, (float)Lsd, 0.f, loss};
  row_loss[t] = loss;
  if (kind == 6) {      // both KLs, and the first search interval: no further than 2^-40 of the largest teacher probability
    const double fkl = (double)c * X / St - Ltd + Lsd, rkl = (double)c * X2 / Ss - Lsd + Ltd;
    const float ltmax = (float)((double)Mt - Ltd);
    akl[AKL_FKL * T_pad + t] = (float)(0.6931471805599453 * fkl);
    akl[AKL_RKL * T_pad + t] = (float)(0.6931471805599453 * rkl);
    // (the strip loop's grid may start higher: less than 1 - mu lies below `least`)
    akl[AKL_LO * T_pad + t] = strip ? 0.f : ltmax - 40.f;
    akl[AKL_HI * T_pad + t] = strip ? fmaxf(ltmax - 40.f, least) : ltmax + 1.0e-3f;         // (1e-3: above every entry)
    akl[AKL_LTMAX * T_pad + t] = ltmax;
    akl[AKL_WR * T_pad + t] = akl[AKL_CROWD * T_pad + t] = 0.f;
  }
}

// AKL: merge one search pass.  mass_k = teacher mass at or above threshold k (decreasing in k); the new
// interval is the pair of neighbouring thresholds between which the mass drops to mu or below.
template <int TX, int NT>
__global__ __launch_bounds__(NT) void akl_search_combine_kernel(const float* partials, const int* meta, int T_pad,
                                                                float mu, float* akl) {
  __shared__ float lds[NT / 64 * AKL_K * TX];
  const int t = blockIdx.x * TX + threadIdx.x % TX, g = threadIdx.x / TX;
  const int n_valid = meta[META_N_VALID], n_parts = meta[META_N_SPLIT];
  if ((int)(blockIdx.x * TX) >= n_valid) return;
  float m[AKL_K];
#pragma unroll
  for (int k = 0; k < AKL_K; ++k) m[k] = 0.f;
  for (int p = g; p < n_parts; p += NT / TX) {
    const float* q = partials + (int64_t)p * AKL_K * T_pad + t;
#pragma unroll
    for (int k = 0; k < AKL_K; ++k) m[k] += q[(int64_t)k * T_pad];
  }
  merge_parts<TX, NT, AKL_K, MergeSum>(m, lds);
  if (g != 0 || t >= n_valid) return;
  const float lo = akl[AKL_LO * T_pad + t], hi = akl[AKL_HI * T_pad + t];
  const float step = (hi - lo) * (1.f / (AKL_K + 1)), th0 = lo + step;
  float new_lo = lo, new_hi = hi;
  bool found = false;
#pragma unroll
  for (int k = 0; k < AKL_K; ++k) {
    const float th = fmaf((float)k, step, th0);     // the very expression the search kernel compares with
    if (!found) {
      if (m[k] <= mu) { new_hi = th; found = true; }
      else new_lo = th;
    }
  }
  akl[AKL_LO * T_pad + t] = new_lo;
  akl[AKL_HI * T_pad + t] = new_hi;
}

// The same for the strip loop's bins of `width` cells: the interval becomes the bin in which the mass from the top on passes mu, or
// the lowest one.  The pass by bins of kAklBins cells is the last one for most: the row pass does the rest (AklRowsEpi), whose sums
// are cleared here.  Where more entries than AKL_FEW lie in a token's interval (at most its mass over its lowest probability), its
// token tile takes a third pass, by single cells, behind which the upper edge of the bin is the threshold.  (Two additions to
// memory an entry: 1024 of them for every token cost about what the third pass does.)
constexpr float AKL_FEW = 1024.f;
// A thread sums one bin of one token over the parts, 32 bytes of each.  (With a thread's share of the parts in all bins, 82 registers of 44
// sums were spilled: T = 2048 31 -> 13 us a merge.)
__global__ __launch_bounds__(512) void akl_bins_combine_kernel(const float* partials, const int* meta, int T_pad, float mu, float width,
                                                               float* akl, unsigned long long* fine) {
  constexpr int TX = 8;
  __shared__ float m[AKL_BINS][TX];
  const int t0 = blockIdx.x * TX, tx = threadIdx.x % TX, bin_of = threadIdx.x / TX, t = t0 + tx;
  const int n_valid = meta[META_N_VALID], n_parts = meta[META_N_SPLIT];
  if (t0 >= n_valid) return;
  if (width == 1.f && !akl_crowded(akl, T_pad, t0 / BN)) return;
  if (width == (float)AKL_BINS)
    for (int i = threadIdx.x; i < TX * AKL_BINS * 2; i += 512) fine[(int64_t)t0 * AKL_BINS * 2 + i] = 0;
  if (bin_of < AKL_BINS) {
    const float* const q = partials + (int64_t)bin_of * T_pad + t;
    float sum = 0.f;
#pragma unroll 16
    for (int p = 0; p < n_parts; ++p) sum += q[(int64_t)p * AKL_BINS * T_pad];
    m[bin_of][tx] = sum;
  }
  __syncthreads();
  if (bin_of != 0 || t >= n_valid) return;
  float above = akl[AKL_WR * T_pad + t], bin = 0.f, mass = m[0][tx];
  bool found = false;
#pragma unroll
  for (int k = AKL_BINS - 1; k > 0; --k) {
    const float mk = m[k][tx];
    if (!found && above + mk > mu) { bin = (float)k; mass = mk; found = true; }
    if (!found) above += mk;
  }
  const float lo = fmaf(bin, width, akl[AKL_LO * T_pad + t]), low = akl[AKL_HI * T_pad + t];
  const float cell = akl_cell(low, akl[AKL_LTMAX * T_pad + t]);
  akl[AKL_LO * T_pad + t] = lo;
  if (width == (float)AKL_BINS) akl[AKL_CROWD * T_pad + t] = mass > AKL_FEW * fexp2(akl_edge(lo, low, cell)) ? 1.f : 0.f;
  if (width == 1.f) akl[AKL_HI * T_pad + t] = akl_edge(lo + 1.f, low, cell);
  akl[AKL_WR * T_pad + t] = above;
}

// The two row sums (a1, a2) of a token, in every thread of the token.
template <int TX, int NT>
__device__ __forceinline__ void merge_row_sums(const float* partials, int n_parts, int T_pad, int t, int g, float* lds,
                                               float (&a)[2]) {
  a[0] = a[1] = 0.f;
#pragma unroll 4
  for (int p = g; p < n_parts; p += NT / TX) {
    const float* q = partials + (int64_t)p * 2 * T_pad + t;
    a[0] += q[0];
    a[1] += q[T_pad];
  }
  merge_parts<TX, NT, 2, MergeSum>(a, lds);
}

// AKL: gaps -> weights, row loss and the row term of the gradient (see GradEpi).  With `fine`, the strip loop's row pass has left the
// interval's entries by cells: the border is the cell in which the mass from the top on passes mu, or the lowest one, and the cells
// above it are head.  (In a crowded tile they are all 0: the third search pass has found the border.)
template <int TX, int NT>
__global__ __launch_bounds__(NT) void akl_weights_kernel(const float* partials, const int* meta, int T_pad, float mu,
                                                         const unsigned long long* fine, f32x4* rowinfo, float* row_loss, float* akl) {
  __shared__ float lds[NT / 64 * 2 * TX];
  const int t = blockIdx.x * TX + threadIdx.x % TX, g = threadIdx.x / TX;
  const int n_valid = meta[META_N_VALID], n_parts = meta[META_N_SPLIT];
  if ((int)(blockIdx.x * TX) >= n_valid) return;
  float a[2];
  merge_row_sums<TX, NT>(partials, n_parts, T_pad, t, g, lds, a);
  if (g != 0 || t >= n_valid) return;
  if (fine) {
    const unsigned long long* const own = fine + (int64_t)t * AKL_BINS * 2;
    const float above = akl[AKL_WR * T_pad + t];
    unsigned long long mass = 0, head = 0, tail = 0;
    bool found = false;
#pragma unroll 4
    for (int k = AKL_BINS - 1; k >= 0; --k) {
      mass += own[2 * k];
      found = found || k == 0 || above + (float)mass * 0x1p-56f > mu;
      (found ? tail : head) += own[2 * k + 1];
    }
    a[0] += (float)head * 0x1p-56f;
    a[1] += (float)tail * 0x1p-56f;
  }
  const float gt = a[1], tot = a[0] + a[1];
  const float wr = tot > 0.f ? gt / tot : 0.5f, wf = 1.f - wr;
  const float fkl = akl[AKL_FKL * T_pad + t], rkl = akl[AKL_RKL * T_pad + t];
  f32x4 ri = rowinfo[t];
  ri[3] = wf - wr * rkl;
  rowinfo[t] = ri;
  row_loss[t] = wf * fkl + wr * rkl;
  akl[AKL_WR * T_pad + t] = wr;
}

// JSD / TVD / skewed KL: merge the row sums into the row loss and R (see RowTerm).
template <int TX, int NT>
__global__ __launch_bounds__(NT) void combine_rows_kernel(const float* partials, const int* meta, int T_pad, int kind,
                                                          float w, f32x4* rowinfo, float* row_loss) {
  __shared__ float lds[NT / 64 * 2 * TX];
  const int t = blockIdx.x * TX + threadIdx.x % TX, g = threadIdx.x / TX;
  const int n_valid = meta[META_N_VALID], n_parts = meta[META_N_SPLIT];
  if ((int)(blockIdx.x * TX) >= n_valid) return;
  float a[2];
  merge_row_sums<TX, NT>(partials, n_parts, T_pad, t, g, lds, a);
  if (g != 0 || t >= n_valid) return;
  const float A1 = a[0], A2 = a[1];
  float loss, R;
  if (kind == 2) { loss = LN2 * (w * A1 + (1.f - w) * A2); R = (1.f - w) * LN2 * A2; }
  else if (kind == 3) { loss = 0.5f * A1; R = 0.5f * A2; }
  else if (kind == 4) { loss = LN2 * A1; R = -(1.f - w) * A2; }
  else { loss = LN2 * A1; R = A2; }
  f32x4 ri = rowinfo[t];
  ri[3] = R;
  rowinfo[t] = ri;
  row_loss[t] = loss;
}

// The token operand of grad_W_s: h_s of the compacted rows transposed, as [16 hidden rows][32-token sub-step][lane][8], lane l
// holding tokens 8 (l / 16) .. + 7 of hidden row l mod 16; zero beyond the valid tokens.  Block (r0, c0) of 64 tokens x 64
// hidden rows through LDS, by 16 waves.
template <class E>
__device__ __forceinline__ void pack_columns(const E* src, int C, bf16_t* dst, int T_pad, const int* rowmap, int n_valid, int r0,
                                             int c0, bf16_t (*tile)[66]) {
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int c = c0 + tx, cc = min(c, C - 1);
  E v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)            // (rowmap holds a valid row for every r < T_pad: the loads need no test)
    v[i] = src[(int64_t)rowmap[r0 + ty + 16 * i] * C + cc];
#pragma unroll
  for (int i = 0; i < 4; ++i) tile[ty + 16 * i][tx] = r0 + ty + 16 * i < n_valid && c < C ? (bf16_t)v[i] : (bf16_t)0.f;
  __syncthreads();
  const int sub = ty >> 2, blk = ty & 3;                             // a wave: 16 hidden rows x 32 tokens, 1 KiB
  if (sub > 1 || c0 + 16 * blk >= C) return;
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = tile[32 * sub + 8 * (tx >> 4) + e][16 * blk + (tx & 15)];
  *(bf16x8*)(dst + ((int64_t)(c0 / 16 + blk) * (T_pad / 32) + r0 / 32 + sub) * 512 + tx * 8) = o;
}

struct PackColumnsArgs {
  const void* src;
  bf16_t* dst;
  const int* rowmap;
  int src_f32, C, T_pad;
};

// Workgroup 0: loss = sum of the valid rows' losses / n (fixed-order fp64 tree), per-row gradient
// scale 1 / (n tau), and the caller's per-token losses (0 for masked tokens).
// `weight` scales what leaves the call (teacher weight, optional tau^2); with `accumulate` the loss
// outputs are added to (further teachers of a multi-teacher call).
// The others, if there is a backward pass: h_s transposed and packed (pack_columns), beside it (a launch, 4 to 6 us).
__global__ __launch_bounds__(1024) void finalize_kernel(const int* meta, const int* inv, const float* row_loss, int T, float tau,
                                                        float weight, int accumulate, f32x4* rowinfo, float* loss_out,
                                                        float* per_token_out, const PackColumnsArgs pc) {
  __shared__ double s_sum[1024];
  __shared__ bf16_t tile[64][66];
  if (flat_group() > 0) {
    const int b = (int)(flat_group() - 1), wide = pc.T_pad / 64, by = b / wide, r0 = (b - by * wide) * 64, c0 = by * 64;
    if (c0 >= pc.C) return;
    const int n = meta[META_N_VALID];
    if (pc.src_f32) pack_columns((const float*)pc.src, pc.C, pc.dst, pc.T_pad, pc.rowmap, n, r0, c0, tile);
    else pack_columns((const bf16_t*)pc.src, pc.C, pc.dst, pc.T_pad, pc.rowmap, n, r0, c0, tile);
    return;
  }
  const int tid = threadIdx.x;
  const int n = meta[META_N_VALID];
  double acc = 0.0;
  for (int j = tid; j < n; j += 1024) acc += (double)row_loss[j];
  s_sum[tid] = acc;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (tid < s) s_sum[tid] += s_sum[tid + s];
    __syncthreads();
  }
  if (tid == 0) {
    const float l = n > 0 ? weight * (float)(s_sum[0] / (double)n) : 0.f;
    *loss_out = accumulate ? *loss_out + l : l;
  }
  const float scale = n > 0 ? weight / ((float)n * tau) : 0.f;
  for (int j = tid; j < n; j += 1024) rowinfo[j][2] = scale;
  if (per_token_out)
    for (int t = tid; t < T; t += 1024) {
      const int j = inv[t];
      const float l = j >= 0 ? weight * row_loss[j] : 0.f;
      per_token_out[t] = accumulate ? per_token_out[t] + l : l;
    }
}

// dst[c][r] = src[r][c] for r < R, zero for R <= r < R_pad;  c < C.  64 x 64 tiles through LDS.
template <class E>
__global__ void transpose_kernel(const E* src, int64_t ld_src, int R, int C, E* dst, int64_t ld_dst, int R_pad) {
  __shared__ E tile[64][66];
  const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int r = r0 + i, c = c0 + tx;
    tile[i][tx] = (r < R && c < C) ? src[(int64_t)r * ld_src + c] : E(0);
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int c = c0 + i, r = r0 + tx;
    if (c < C && r < R_pad) dst[(int64_t)c * ld_dst + r] = tile[tx][i];
  }
}

// The token operand of the strip loop: the compacted rows (row j = row rowmap[j] of src for j < n_valid, zero
// beyond) in the order in which its waves load them: [64-token panel][32-element sub-step][16-token block][lane][8],
// lane l holding elements 8 (l / 16) .. + 7 of token l mod 16.  fp32 rows become [hi | lo | hi] (see
// prepare).  A block of 256 threads writes 4 KiB; bound by its reads, 64-byte pieces of each row.
// dz_order (bf16 only): elements 4 (l / 16) .. + 3 and 16 + 4 (l / 16) .. + 3 instead, the order in which transposing reads
// bring the heads kept as [H][V] (A_KMAJOR_DZ in kd_strip.hpp).
__device__ __forceinline__ void pack_rows(int block, int tid, const void* src, int src_f32, int dz_order, int R, int H, bf16_t* dst, int K,
                                          const int* rowmap, const int* meta) {
  const int lane = tid & 63, blk = tid >> 6;
  const int panel = block / (K / 32), kb = block - panel * (K / 32);
  if (panel * 64 >= R) return;
  const int j = panel * 64 + 16 * blk + (lane & 15), k0 = 32 * kb + 8 * (lane >> 4);
  bf16x8 v;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (bf16_t)0.f;
  if (j < meta[META_N_VALID]) {
    const int64_t row = (int64_t)rowmap[j] * H;
    if (!src_f32) {
      if (dz_order) {                              // (H is a multiple of 64)
        const bf16_t* x = (const bf16_t*)src + row + 32 * kb + 4 * (lane >> 4);
        const bf16x4 lo = *(const bf16x4*)x, hi = *(const bf16x4*)(x + 16);
        v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      } else if (k0 < H) {
        v = *(const bf16x8*)((const bf16_t*)src + row + k0);
      }
    } else if (k0 < 3 * H) {
      const int part = k0 / H;                     // H is a multiple of 8: the eight values are of one part
      const f32x4* x = (const f32x4*)((const float*)src + row + (k0 - part * H));
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float f = x[i >> 2][i & 3];
        const bf16_t hi = (bf16_t)f;
        v[i] = part == 1 ? (bf16_t)(f - (float)hi) : hi;
      }
    }
  }
  *(bf16x8*)(dst + ((((int64_t)panel * (K / 32) + kb) * 4 + blk) * 64 + lane) * 8) = v;
}

// Re-pack one operand as bf16 [R][K]: plain copy (bf16 source) or the high / low bf16 parts of an
// fp32 source laid side by side along K, zero-padded up to K.
//   split_mode 1 (heads):         [hi | hi | lo]
//   split_mode 2 (hidden states): [hi | lo | hi]
// so that sum_k A'[m][k] B'[n][k] = hi.hi + hi.lo + lo.hi.
// With a row map, destination row j takes source row rowmap[j] for j < n_valid and is zero beyond:
// the compacted copy of the hidden states.
// Bound by memory: a thread makes 16 bytes of four rows (lanes along K, so that reads and writes are whole lines,
// and four independent loads in flight); element by element, with two 64-bit divisions each, the heads of
// V = 50264, H = 1000 and 520 took 124 and 70 us; two micro-batches of 777 tokens went from 1545 to 1396 us.
__device__ __forceinline__ void prepare(int block, int tid, const void* src, int src_f32, int R, int H, bf16_t* dst, int K,
                                        int split_mode, const int* rowmap, const int* meta) {
  const int wide = (R + 15) / 16, by = block / wide, bx = block - by * wide;
  const int k0 = (by * 64 + (tid & 63)) * 8;
  if (k0 >= K) return;
  const int part = src_f32 ? k0 / H : 0, col = k0 - part * H;      // H is a multiple of 8: eight values of one part
  const bool lo = (split_mode == 1 && part == 2) || (split_mode == 2 && part == 1);
  const bool pad = src_f32 ? part > 2 : k0 >= H;
  const int n = rowmap ? meta[META_N_VALID] : R;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = bx * 16 + (tid >> 6) + 4 * i;
    if (r >= R) return;
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (bf16_t)0.f;
    if (r < n && !pad) {
      const int64_t at = (int64_t)(rowmap ? rowmap[r] : r) * H + col;
      if (!src_f32) {
        v = *(const bf16x8*)((const bf16_t*)src + at);
      } else {
        const f32x4* x = (const f32x4*)((const float*)src + at);
        const f32x4 x0 = x[0], x1 = x[1];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float f = e < 4 ? x0[e & 3] : x1[e & 3];
          const bf16_t hi = (bf16_t)f;
          v[e] = lo ? (bf16_t)(f - (float)hi) : hi;
        }
      }
    }
    *(bf16x8*)(dst + (int64_t)r * K + k0) = v;
  }
}

// The same for a head kept as [H][R]: element (r, c) lies at c * R + r.  64 x 64 tiles through LDS.
__global__ __launch_bounds__(256) void prepare_transposed_kernel(const void* src, int src_f32, int R, int H, bf16_t* dst,
                                                                 int K) {
  __shared__ float tile[64][65];
  const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64, tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int c = min(c0 + ty + 4 * i, H - 1), r = min(r0 + tx, R - 1);
    const int64_t at = (int64_t)c * R + r;
    tile[ty + 4 * i][tx] = src_f32 ? ((const float*)src)[at] : (float)((const bf16_t*)src)[at];
  }
  __syncthreads();
  const int c = c0 + tx;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = r0 + ty + 4 * i;
    if (r >= R) break;
    const float x = tile[tx][ty + 4 * i];
    const bf16_t hi = (bf16_t)x;
    bf16_t* const row = dst + (int64_t)r * K;
    if (!src_f32) {
      if (c < K) row[c] = c < H ? hi : (bf16_t)0.f;
    } else {
      if (c < H) {                     // [hi | hi | lo]
        row[c] = hi;
        row[H + c] = hi;
        row[2 * H + c] = (bf16_t)(x - (float)hi);
      }
      if (3 * H + c < K && c < K - 3 * H) row[3 * H + c] = (bf16_t)0.f;      // the padding is shorter than 64
    }
  }
}

// The common case of the above, 16 bytes per thread: bf16 (or byte) rows that only have to be gathered
// (K == H, H a multiple of 8).  Row j of dst is row rowmap[j] of src for j < n_valid, zero beyond.
__device__ __forceinline__ void gather_rows(int block, int tid, const u32x4* src, u32x4* dst, int R, int chunks_per_row,
                                            const int* rowmap, const int* meta) {
  const int64_t i = (int64_t)block * 256 + tid;
  if (i >= (int64_t)R * chunks_per_row) return;
  const int j = (int)(i / chunks_per_row), c = (int)(i % chunks_per_row);
  u32x4 v = {0u, 0u, 0u, 0u};
  if (j < meta[META_N_VALID]) v = src[(int64_t)rowmap[j] * chunks_per_row + c];
  dst[i] = v;
}

// The row map and the operand copies of a call (pack_rows, prepare, gather_rows) share launches: each is small or independent
// of the others, and a launch costs 4 us.  Copies that do not look at the row map go with it, in the first launch; those that
// do, in a second.  Workgroups of 1024 threads (what the row map wants) work as four blocks of 256; a job's blocks are
// rounded up to whole workgroups.  T = 128, V = 4096, fp32 (four copies): five launches, 23 us -> one.
struct OperandJob {
  int kind;                // 0: prepare, 1: pack_rows, 2: gather_rows
  int groups;              // workgroups
  int R, H, K, mode;       // mode: split_mode of prepare, dz_order of pack_rows
  int src_f32;
  const int* rowmap;
  const void* src;
  bf16_t* dst;
};
struct OperandArgs {
  RowmapArgs rm;
  int with_rowmap, n;
  OperandJob job[4];
};
__global__ __launch_bounds__(1024) void operands_kernel(const OperandArgs a) {
  int64_t b = flat_group();
  if (a.with_rowmap) {
    if (b == 0) {
      make_rowmap(a.rm);
      return;
    }
    --b;
  }
  int i = 0;
  while (i + 1 < a.n && b >= a.job[i].groups) b -= a.job[i++].groups;
  const OperandJob& q = a.job[i];
  if (b >= q.groups) return;
  const int block = 4 * (int)b + (int)(threadIdx.x >> 8), tid = threadIdx.x & 255;
  if (q.kind == 0) prepare(block, tid, q.src, q.src_f32, q.R, q.H, q.dst, q.K, q.mode, q.rowmap, a.rm.meta);
  else if (q.kind == 1) pack_rows(block, tid, q.src, q.src_f32, q.mode, q.R, q.H, q.dst, q.K, a.rm.rowmap, a.rm.meta);
  else gather_rows(block, tid, (const u32x4*)q.src, (u32x4*)q.dst, q.R, q.K / 8, q.rowmap, a.rm.meta);
}

// Measurement aid: what the matrix pipe sustains with nothing else going on.  Same occupancy as the
// logit kernels (one workgroup of 8 waves per CU, forced by the LDS request), 8 independent 32x32x16
// accumulators per wave, operands taken from the caller's buffer (the shader clock under MFMA load
// depends on the operand values, so they should look like real data).
__global__ __launch_bounds__(512) void mfma_probe_kernel(const bf16x8* operands, int iters, float* sink,
                                                         long long* clock_out) {
  const long long c0 = clock64(), r0 = wall_clock64();
  const int lane_id = (blockIdx.x * 512 + threadIdx.x) & 2047;      // 2048 x 4 x 16 B = 128 KiB of operands
  bf16x8 a0 = operands[lane_id * 4 + 0], a1 = operands[lane_id * 4 + 1];
  bf16x8 b0 = operands[lane_id * 4 + 2], b1 = operands[lane_id * 4 + 3];
  f32x16 c[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) c[i][r] = 0.f;
  for (int it = 0; it < iters; ++it) {
    c[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, c[0], 0, 0, 0);
    c[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b1, c[1], 0, 0, 0);
    c[2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b0, c[2], 0, 0, 0);
    c[3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, c[3], 0, 0, 0);
    c[4] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0, a0, c[4], 0, 0, 0);
    c[5] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1, a0, c[5], 0, 0, 0);
    c[6] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0, a1, c[6], 0, 0, 0);
    c[7] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1, a1, c[7], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) s += c[i][r];
  sink[blockIdx.x * 512 + threadIdx.x] = s;
  if (clock_out && blockIdx.x == 0 && threadIdx.x == 0) {
    clock_out[0] = clock64() - c0;
    clock_out[1] = wall_clock64() - r0;
  }
}

// OCP e4m3 (4 exponent bits, bias 7, 3 mantissa bits, no infinities, 0x7f = NaN, largest 448):
// round to nearest even, magnitudes beyond 448 saturate to 448.
__device__ __forceinline__ uint32_t f32_to_e4m3(float x) {
  const uint32_t u = __float_as_uint(x);
  const uint32_t sign = (u >> 24) & 0x80u;
  const float a = fabsf(x);
  if (!(a == a)) return sign | 0x7fu;
  if (a >= 448.f) return sign | 0x7eu;
  if (a < 0.015625f) return sign | (uint32_t)__builtin_rintf(a * 512.f);   // steps of 2^-9; 8 = smallest normal
  const uint32_t ua = u & 0x7fffffffu;
  const uint32_t m = ua & 0x7fffffu, rem = m & 0xfffffu;
  uint32_t code = (((ua >> 23) - 120u) << 3) | (m >> 20);                   // exponent re-biased 127 -> 7
  if (rem > 0x80000u || (rem == 0x80000u && (code & 1u))) ++code;           // a carry moves into the exponent
  return sign | code;
}

// dst[i] = e4m3(src[i] * inv_scale), 8 values per thread
__global__ void quantize_e4m3_kernel(const void* src, int src_f32, int64_t n, float inv_scale, uint8_t* dst) {
  const int64_t i0 = (flat_group() * blockDim.x + threadIdx.x) * 8;
  if (i0 >= n) return;
  uint32_t w[2] = {0u, 0u};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int64_t i = i0 + k;
    float x = 0.f;
    if (i < n) x = src_f32 ? ((const float*)src)[i] : (float)((const bf16_t*)src)[i];
    w[k >> 2] |= f32_to_e4m3(x * inv_scale) << (8 * (k & 3));
  }
  if (i0 + 8 <= n) {
    *(uint2*)(dst + i0) = make_uint2(w[0], w[1]);
  } else {
    for (int k = 0; i0 + k < n; ++k) dst[i0 + k] = (uint8_t)(w[k >> 2] >> (8 * (k & 3)));
  }
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
hipError_t launch_stats(const Problem& p, hipStream_t st) {
  LogitArgs a = make_logit_args(p);
  a.v0 = 0; a.v_end = p.V; a.n_vt = p.n_vt;
  a.partials = p.partials;
  a.clock_out = p.clock_out;
  const int grid = p.n_tt * p.n_split;      // worst case; workgroups beyond the device-side plan exit
#define KD_STATS(K) (few_tokens(p) ? launch_few_stats(p, a, grid, st) : p.strip && p.w_hv_inplace ? launch_strip_hv_stats(p, a, grid, st) \
                     : p.strip ? launch_big<stats_strip_kernel<K>>(grid, StripCfg::NT, StripCfg::STATE_SMEM_BYTES, st, &a) \
                     : p.t_fp8 ? launch_big<stats_kernel<K, true, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                     : p.w_hv_inplace ? launch_big<stats_kernel<K, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                               : launch_big<stats_kernel<K, false, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a))
  switch (p.kind) {
    case 0: return KD_STATS(0);
    case 1: return KD_STATS(1);
    case 6:                        // both cross terms (AKL; never with the fp8 teacher)
      return few_tokens(p) ? launch_few_stats(p, a, grid, st) : p.strip && p.w_hv_inplace ? launch_strip_hv_stats(p, a, grid, st)
             : p.strip ? launch_big<stats_strip_kernel<6>>(grid, StripCfg::NT, StripCfg::STATE_SMEM_BYTES, st, &a)
             : p.w_hv_inplace ? launch_big<stats_kernel<6, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a)
                              : launch_big<stats_kernel<6, false, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a);
    default: return KD_STATS(2);   // log-sum-exps only
  }
#undef KD_STATS
}

hipError_t launch_rows(const Problem& p, hipStream_t st) {
  LogitArgs a = make_logit_args(p);
  a.v0 = 0; a.v_end = p.V; a.n_vt = p.n_vt;
  a.partials = p.partials;
  const int grid = p.n_tt * p.n_split;
#define KD_ROWS(K) (few_tokens(p) ? launch_few_rows(p, a, grid, st) : p.strip && p.w_hv_inplace ? launch_strip_hv_rows(p, a, grid, st) \
                     : p.strip ? launch_big<rows_strip_kernel<K>>(grid, StripCfg::NT, StripCfg::SMEM_BYTES, st, &a) \
                     : p.t_fp8 ? launch_big<rows_kernel<K, true, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                     : p.w_hv_inplace ? launch_big<rows_kernel<K, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                               : launch_big<rows_kernel<K, false, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a))
  switch (p.kind) {
    case 2: return KD_ROWS(2);
    case 3: return KD_ROWS(3);
    case 4: return KD_ROWS(4);
    case 6:
      return few_tokens(p) ? launch_few_rows(p, a, grid, st) : p.strip && p.w_hv_inplace ? launch_strip_hv_rows(p, a, grid, st)
             : p.strip ? launch_big<rows_strip_kernel<6>>(grid, StripCfg::NT, StripCfg::STATE_SMEM_BYTES, st, &a)
             : p.w_hv_inplace ? launch_big<rows_kernel<6, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a)
                              : launch_big<rows_kernel<6, false, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a);
    default: return KD_ROWS(5);
  }
#undef KD_ROWS
}

// Shape of the merges: 8 tokens x 128 threads each where a token may have 128 parts or more, else 32 tokens x 8
// threads each (see merge_parts).  128 parts, T = 128: combine_kernel 10.4 -> 5.8 us by the first.
static bool many_parts(const Problem& p) { return p.n_split >= 128; }

// AKL: one pass of the threshold search (teacher logit tiles only) and its merge.
hipError_t launch_akl_search(const Problem& p, int pass, hipStream_t st) {
  LogitArgs a = make_logit_args(p);
  a.v0 = 0; a.v_end = p.V; a.n_vt = p.n_vt;
  a.partials = p.partials;
  a.akl_width = pass == 0 ? kAklBins * kAklBins : pass == 1 ? kAklBins : 1;
  const int grid = p.n_tt * p.n_split;
  hipError_t e = few_tokens(p) ? launch_few_search(p, a, grid, st)
           : p.strip && p.w_hv_inplace ? launch_strip_hv_search(a, grid, st)
           : p.strip ? launch_big<akl_search_strip_kernel>(grid, StripCfg::NT, BinsEpi::SMEM_BYTES, st, &a)
           : p.w_hv_inplace ? launch_big<akl_search_kernel<true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a)
                            : launch_big<akl_search_kernel<false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a);
  if (e != hipSuccess) return e;
  if (p.strip) {
    hipLaunchKernelGGL(akl_bins_combine_kernel, dim3(p.T_pad / 8), dim3(512), 0, st, p.partials, p.meta, p.T_pad, p.beta,
                       a.akl_width, p.akl, p.akl_fine);
    return hipGetLastError();
  }
  if (many_parts(p))
    hipLaunchKernelGGL((akl_search_combine_kernel<8, 1024>), dim3(p.T_pad / 8), dim3(1024), 0, st, p.partials, p.meta,
                       p.T_pad, p.beta, p.akl);
  else
    hipLaunchKernelGGL((akl_search_combine_kernel<32, 256>), dim3(p.T_pad / 32), dim3(256), 0, st, p.partials, p.meta,
                       p.T_pad, p.beta, p.akl);
  return hipGetLastError();
}

hipError_t launch_akl_weights(const Problem& p, hipStream_t st) {
  if (many_parts(p))
    hipLaunchKernelGGL((akl_weights_kernel<8, 1024>), dim3(p.T_pad / 8), dim3(1024), 0, st, p.partials, p.meta,
                       p.T_pad, p.beta, p.strip ? p.akl_fine : nullptr,
                       (f32x4*)p.rowinfo, p.row_loss, p.akl);
  else
    hipLaunchKernelGGL((akl_weights_kernel<32, 256>), dim3(p.T_pad / 32), dim3(256), 0, st, p.partials, p.meta,
                       p.T_pad, p.beta, p.strip ? p.akl_fine : nullptr,
                       (f32x4*)p.rowinfo, p.row_loss, p.akl);
  return hipGetLastError();
}

static RowmapArgs rowmap_args(const Problem& p) {
  // units: 64 vocabulary rows for the strip loop, tiles for the eight-wave one (whose gradient kernel strides)
  const int last = p.V - (p.V - 1) / p.V_c * p.V_c;      // width of the last chunk
  SplitChoice stats{p.n_vt, 1, 0, p.n_split, 0}, grad{1, 1, 0, 1, 0}, grad_last = grad;
  if (p.strip) {
    const int per = StripCfg::BM / 64, sh = StripCfg::SHORT / 64, full = p.V < p.V_c ? p.V : p.V_c;
    auto choice = [&](int rows, int most, int short_units, int strided) {
      const int units = (rows + 63) / 64;
      return SplitChoice{units, per, short_units, most < units ? most : units, strided};
    };
    stats = choice(p.V, p.n_split, sh, 0);
    grad = choice(full, p.g_split, 0, 1);
    grad_last = choice(last, p.g_split, 0, 1);
  }
  return RowmapArgs{p.mask, p.T, p.T_pad, p.n_cu, stats, grad, grad_last, p.rowmap, p.inv, p.meta};
}

hipError_t launch_operands(const Problem& p, bool rowmap, bool student, bool teacher, hipStream_t st) {
  OperandArgs first{}, second{};       // what does not look at the row map, and what does
  first.rm = second.rm = rowmap_args(p);
  first.with_rowmap = rowmap;
  int64_t groups_first = rowmap ? 1 : 0, groups_second = 0;
  auto add = [&](bool mapped, OperandJob j, int64_t blocks) {
    j.groups = (int)((blocks + 3) / 4);
    OperandArgs& to = mapped ? second : first;
    to.job[to.n++] = j;
    (mapped ? groups_second : groups_first) += j.groups;
  };
  // hidden states: packed for the strip loop; else copied where they are gathered, split or padded
  auto hidden = [&](const void* src, int H, void* dst, int K, bool fp8) {
    OperandJob j{};
    j.src = src; j.dst = (bf16_t*)dst; j.src_f32 = p.in_f32 && !fp8;
    j.R = p.T; j.H = H; j.K = K;
    if (fp8) { j.H /= 2; j.K /= 2; }      // rows of bytes as rows of two-byte words
    j.rowmap = p.mask ? p.rowmap : nullptr;
    if (p.strip) {
      j.kind = 1; j.mode = p.w_hv_inplace; j.R = p.T_pad;
      add(true, j, (int64_t)(p.T_pad / 64) * (K / 32));
    } else if (!j.src_f32 && j.K == j.H && p.mask) {
      j.kind = 2;
      add(true, j, ((int64_t)j.R * j.K / 8 + 255) / 256);
    } else {
      j.mode = 2;
      add(p.mask != nullptr, j, (int64_t)((j.R + 15) / 16) * ((j.K + 511) / 512));
    }
  };
  auto head = [&](const void* src, int H, void* dst, int K) {
    OperandJob j{};
    j.src = src; j.dst = (bf16_t*)dst; j.src_f32 = p.in_f32;
    j.R = p.V; j.H = H; j.K = K; j.mode = 1;
    add(false, j, (int64_t)((j.R + 15) / 16) * ((j.K + 511) / 512));
  };
  if (teacher && p.prep_ht) hidden(p.user_h_t, p.H_t, const_cast<void*>(p.h_t), p.K_t, p.t_fp8);
  if (student && p.prep_hs) hidden(p.user_h_s, p.H_s, const_cast<void*>(p.h_s), p.K_s, false);
  if (teacher && p.prep_Wt && !p.w_hv) head(p.user_W_t, p.H_t, const_cast<void*>(p.W_t), p.K_t);
  if (student && p.prep_Ws && !p.w_hv) head(p.user_W_s, p.H_s, const_cast<void*>(p.W_s), p.K_s);
  auto launch = [&](int64_t groups, const OperandArgs& a) {
    const FlatGrid g = flat_grid(groups);
    if (groups) hipLaunchKernelGGL(operands_kernel, dim3(g.x, g.y), dim3(1024), 0, st, a);
  };
  launch(groups_first, first);
  launch(groups_second, second);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !p.w_hv) return e;
  // heads kept as [H][V] that are not read in place: transposed copies
  auto turned = [&](const void* src, int H, void* dst, int K) {
    hipLaunchKernelGGL(prepare_transposed_kernel, dim3((p.V + 63) / 64, ((p.in_f32 ? H : K) + 63) / 64), dim3(256), 0, st, src,
                       p.in_f32, p.V, H, (bf16_t*)dst, K);
  };
  if (teacher && p.prep_Wt && p.t_fp8)      // e4m3 bytes
    hipLaunchKernelGGL(transpose_kernel<uint8_t>, dim3((p.K_t + 63) / 64, (p.V + 63) / 64), dim3(256), 0, st,
                       (const uint8_t*)p.user_W_t, (int64_t)p.V, p.H_t, p.V, (uint8_t*)const_cast<void*>(p.W_t), (int64_t)p.K_t, p.K_t);
  else if (teacher && p.prep_Wt)
    turned(p.user_W_t, p.H_t, const_cast<void*>(p.W_t), p.K_t);
  if (student && p.prep_Ws) turned(p.user_W_s, p.H_s, const_cast<void*>(p.W_s), p.K_s);
  return hipGetLastError();
}

// Where AKL's search on the strip loop starts at the lowest: entries below log2((1 - mu) / V) hold less than 1 - mu (one more for
// the rounding of the sums).
static float akl_least(const Problem& p) { return p.kind == 6 ? std::log2((1.f - p.beta) / (float)p.V) - 1.f : 0.f; }

hipError_t launch_combine(const Problem& p, hipStream_t st) {
  if (many_parts(p))
    hipLaunchKernelGGL((combine_kernel<8, 1024>), dim3(p.T_pad / 8), dim3(1024), 0, st, p.partials, p.meta,
                       p.T_pad, p.kind, p.strip, 1.4426950408889634f / p.tau, akl_least(p), (f32x4*)p.rowinfo, p.row_loss, p.akl);
  else
    hipLaunchKernelGGL((combine_kernel<32, 256>), dim3(p.T_pad / 32), dim3(256), 0, st, p.partials, p.meta,
                       p.T_pad, p.kind, p.strip, 1.4426950408889634f / p.tau, akl_least(p), (f32x4*)p.rowinfo, p.row_loss, p.akl);
  return hipGetLastError();
}

hipError_t launch_combine_rows(const Problem& p, hipStream_t st) {
  if (many_parts(p))
    hipLaunchKernelGGL((combine_rows_kernel<8, 1024>), dim3(p.T_pad / 8), dim3(1024), 0, st, p.partials, p.meta,
                       p.T_pad, p.kind, p.beta, (f32x4*)p.rowinfo, p.row_loss);
  else
    hipLaunchKernelGGL((combine_rows_kernel<32, 256>), dim3(p.T_pad / 32), dim3(256), 0, st, p.partials, p.meta,
                       p.T_pad, p.kind, p.beta, (f32x4*)p.rowinfo, p.row_loss);
  return hipGetLastError();
}

hipError_t launch_finalize(const Problem& p, bool pack_h_s, hipStream_t st) {
  const PackColumnsArgs pc{p.user_h_s, (bf16_t*)p.h_sT, p.rowmap, p.in_f32, p.H_s, p.T_pad};
  const FlatGrid g = flat_grid(1 + (pack_h_s ? (int64_t)(p.T_pad / 64) * ((p.H_s + 63) / 64) : 0));
  hipLaunchKernelGGL(finalize_kernel, dim3(g.x, g.y), dim3(1024), 0, st, p.meta, p.inv, p.row_loss, p.T, p.tau,
                     p.out_weight, p.accumulate_loss, (f32x4*)p.rowinfo, p.loss, p.per_token_loss, pc);
  return hipGetLastError();
}

hipError_t launch_grad_chunk(const Problem& p, int v0, int width, bool accumulate, hipStream_t st) {
  LogitArgs a = make_logit_args(p);
  a.dz_accumulate = accumulate ? 1 : 0;
  a.v0 = v0; a.v_end = v0 + width;
  a.n_vt = (width + BM - 1) / BM;
  a.bb = largest_divisor_le(a.n_vt, 16);
  a.last_chunk = v0 + width >= p.V;
  a.dz = (bf16_t*)p.dz; a.ldz = p.V_c;
  const int tiles = p.n_tt * a.n_vt;
  // strip loop: one workgroup per (token tile, range), surplus ones exit; eight-wave loop: persistent workgroups
  const int grid = p.strip ? p.n_tt * p.g_split : tiles < p.n_cu ? tiles : p.n_cu;
#define KD_GRAD(K) (few_tokens(p) ? launch_few_grad(p, a, grid, st) : p.strip && p.w_hv_inplace ? launch_strip_hv_grad(p, a, grid, st) \
                     : p.strip ? launch_big<grad_strip_kernel<K>>(grid, StripCfg::NT, StripCfg::STATE_SMEM_BYTES, st, &a) \
                     : p.t_fp8 ? launch_big<grad_kernel<K, true, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                     : p.w_hv_inplace ? launch_big<grad_kernel<K, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                               : launch_big<grad_kernel<K, false, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a))
  switch (p.kind) {
    case 0: return KD_GRAD(0);
    case 1: return KD_GRAD(1);
    case 2: return KD_GRAD(2);
    case 3: return KD_GRAD(3);
    case 4: return KD_GRAD(4);
    case 6:
      return few_tokens(p) ? launch_few_grad(p, a, grid, st) : p.strip && p.w_hv_inplace ? launch_strip_hv_grad(p, a, grid, st)
             : p.strip ? launch_big<grad_strip_kernel<6>>(grid, StripCfg::NT, StripCfg::STATE_SMEM_BYTES, st, &a)
             : p.w_hv_inplace ? launch_big<grad_kernel<6, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a)
                              : launch_big<grad_kernel<6, false, false>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a);
    default: return KD_GRAD(5);
  }
#undef KD_GRAD
}

hipError_t launch_mfma_probe(const void* operands, int iters, float* sink, long long* clock_out, int n_cu,
                             hipStream_t st) {
  struct { const bf16x8* o; int it; float* s; long long* c; } a{(const bf16x8*)operands, iters, sink, clock_out};
  hipError_t e = hipFuncSetAttribute((const void*)mfma_probe_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     LCfg::SMEM_BYTES);
  if (e != hipSuccess) return e;
  void* params[] = {&a.o, &a.it, &a.s, &a.c};
  return hipLaunchKernel((const void*)mfma_probe_kernel, dim3(n_cu), dim3(512), params, LCfg::SMEM_BYTES, st);
}

hipError_t launch_quantize_e4m3(const void* src, int src_f32, int64_t n, float inv_scale, void* dst, hipStream_t st) {
  const FlatGrid g = flat_grid(((n + 7) / 8 + 255) / 256);
  hipLaunchKernelGGL(quantize_e4m3_kernel, dim3(g.x, g.y), dim3(256), 0, st, src, src_f32, n,
                     inv_scale, (uint8_t*)dst);
  return hipGetLastError();
}

#define KD_STR2(...) #__VA_ARGS__
#define KD_STR(...) KD_STR2(__VA_ARGS__)
const char* build_info() {
  static_assert(StripCfg::BM == 192 && StripCfg::NT == 256 && StripCfg::NST == 3, "as named below");
  return "logit tile cfg (MI,NI,WN,BK,NST) = " KD_STR(KD_LOGIT_CFG) "; strip loop = 192 x 256 tiles, 4 waves, 3 stages"
         "; ablation = 0";
}

}  // namespace kd
