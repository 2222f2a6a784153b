// C ABI of libkdloss: argument checks, workspace planning and the launch sequence.
// All checks are host-only and happen before the first HIP call.
#include <hip/hip_runtime.h>

#include "../../include/kdloss.h"
#include "../../include/kdloss_bench.h"
#include "kd_launch.h"

#include <atomic>
#include <cmath>
#ifdef KD_TRACE_ERRORS
#include <cstdio>
#endif

// Scratch memory of kd_loss_fwd_bwd_static: one array per GPU, owned by the library.  In host code this
// name is only a handle for hipGetSymbolAddress; the device address is looked up once per device.
static __device__ __align__(256) unsigned char scratch[KD_STATIC_SCRATCH_BYTES];

namespace {

using kd::Problem;

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct Layout {
  size_t meta, rowmap, inv, row_loss, partials, akl_fine, h_sT, dz, gh32;
  size_t prep_h_s, prep_W_s;                       // re-packed student operands (only when needed)
  size_t common;                                   // end of everything above: the same for every teacher
  size_t rowinfo, akl, prep_h_t, prep_W_t;         // per-teacher block (row statistics, re-packed operands)
  size_t total;                                    // end of this teacher's block
};

kd_status check_params(const kd_loss_params* p) {
  if (!p) return KD_ERR_NULL;
  if (p->T < 1 || p->H_t < 1 || p->H_s < 1 || p->V < 1) return KD_ERR_SHAPE;
  if (p->T > (1 << 22) || p->V > (1 << 24) || p->H_t > 65536 || p->H_s > 65536) return KD_ERR_SHAPE;
  if (p->H_t % 8 || p->H_s % 8 || p->V % 8) return KD_ERR_ALIGN;
  if (p->in_dtype != KD_BF16 && p->in_dtype != KD_F32) return KD_ERR_PARAM;
  if (p->grad_dtype != KD_BF16 && p->grad_dtype != KD_F32) return KD_ERR_PARAM;
  if (p->w_layout != KD_W_HV && p->w_layout != KD_W_VH) return KD_ERR_PARAM;
  if (p->kind < KD_FKL || p->kind > KD_AKL) return KD_ERR_PARAM;
  if (!(p->tau >= 1e-6f && p->tau <= 1e6f)) return KD_ERR_PARAM;   // also rejects NaN
  if ((p->kind == KD_JSD || p->kind == KD_SKEW_FKL || p->kind == KD_SKEW_RKL || p->kind == KD_AKL) &&
      !(p->beta > 0.f && p->beta < 1.f))
    return KD_ERR_PARAM;
  if (p->accumulate_grad_W != 0 && p->accumulate_grad_W != 1) return KD_ERR_PARAM;
  if (p->flags & ~(int32_t)(KD_FLAG_TAU2 | KD_FLAG_TEACHER_FP8)) return KD_ERR_PARAM;
  if (p->flags & KD_FLAG_TEACHER_FP8) {
    if (!(p->teacher_scale > 0.f && p->teacher_scale < INFINITY)) return KD_ERR_PARAM;
    if (p->in_dtype != KD_BF16) return KD_ERR_UNSUPPORTED;     // the student side stays bf16
    if (p->H_t % 128) return KD_ERR_ALIGN;                     // fp8 k-steps are 128 elements
  }
  if (p->kind == KD_AKL && (p->flags & KD_FLAG_TEACHER_FP8)) return KD_ERR_UNSUPPORTED;   // its search pass is bf16 only
  if (p->vocab_chunk != 0 && (p->vocab_chunk < 256 || p->vocab_chunk > (1 << 20) || p->vocab_chunk % 256))
    return KD_ERR_PARAM;
  if (!(std::isfinite(p->loss_scale) && p->loss_scale != 0.f)) return KD_ERR_PARAM;
  if (p->reserved != 0) return KD_ERR_PARAM;
  return KD_OK;
}

// Vocabulary chunk of the backward pass.  The [T_pad, V_c] bf16 staging buffer of dL/dz_s is written by the gradient
// kernel and read back by both products; it should stay in the 256 MB last-level cache together with the operands, but every chunk also
// costs the ends of three launches and re-reads and re-writes the fp32 sums of grad_h_s.
//  - From 4096 tokens on 16384 columns, halved until the staging buffer is within 512 MiB (at least 1024).  Against 8192 columns, means of
//    steps with all tokens and with a tenth masked, 59 sizes, FKL and JSD, T = 4190 .. 16384, V = 54032 .. 151936: 0.966 of the time where
//    the buffer stays in the cache (up to 6656 tokens; 12 sizes, 0.90 .. 0.99), beyond 0.971 with up to 6144 elements contracted for a
//    logit (13 sizes, 0.93 .. 1.00) and 0.991 with more (34 sizes, 0.966 .. 1.013), whose products hide a chunk's ends best.  What a size
//    gains or loses follows the rounds of workgroups: T = 8192, H = 8192 / 2048, V = 128256 38.4 -> 37.0 ms with all tokens, 34.7 -> 34.9
//    with a tenth masked, two teachers, H = 4096 + 2048 / 1024, V = 151936 36.3 -> 34.7; fp32, T = 16384, H = 2048 / 1024, V = 32000
//    15.9 -> 16.0.  (The rounds as priced below would take 16384 at every one of the 59.)  12288 columns: 0.970, 0.991, 0.993.
//    Past 512 MiB wider chunks lose (T = 32768, H = 5120 / 4096, JSD 262.6 -> 265.4).  (At 4096 tokens 24576 columns, 201 MB, measured 11.72
//    against 12.25 ms without a mask on an earlier state; tests/test_abi_host.py holds that size to 16384 columns.)
//  - Below, up to 208 MiB (201 MB still stays in the cache), and the width decides how full the last rounds of
//    workgroups are: the candidates (multiples of the tile heights) are priced by the rounds of the gradient kernel,
//    with all tokens and with an eighth of them masked, and of the grad_W_s product.  Measured steps: T = 3584 10.60 ms
//    with 24576 columns against 10.78 with 16384; T = 2048 6.03 with 49152 against 6.25 with 32768; T = 1024 3.28 with
//    98304 against 3.34 with 65536.
// `logit_k`: elements contracted for one logit of every model of the call (each teacher with the student again).
int64_t choose_chunk(const Problem& q, int64_t v_all, int64_t logit_k) {
  if (q.T_pad >= 4096) {
    int64_t vc = 16384;
    while (vc > 1024 && (int64_t)q.T_pad * vc * 2 > (512ll << 20)) vc >>= 1;
    return vc;
  }
  const int64_t step = 1536, most = (208ll << 20) / (2 * q.T_pad);      // a multiple of 192, 256 and 128
  if (most >= v_all) return v_all;
  const int tile_m = q.strip ? 192 : kd::kTileM, masked_tt = (q.n_tt * 7 + 7) / 8;
  // (the grad_W_s tile that covers H_s cheapest, whatever the width; priced by each width's own, grad_W_tile, a twelfth of the widths
  // below 4096 tokens change, for the worse as often as for the better: T = 1764, H = 576, V = 151936 1.59 -> 1.68 ms, T = 2880,
  // H = 512 / 192 1.63 -> 1.57)
  int64_t gw_rows = 256;
  auto cover = [&](int64_t rows) { return (q.H_s + rows - 1) / rows * (rows + 48); };
  for (int64_t rows : {192, 128}) if (cover(rows) < cover(gw_rows)) gw_rows = rows;
  const int64_t m_tiles = (q.H_s + gw_rows - 1) / gw_rows;
  // multiply-adds of one workgroup: a logit tile, a grad_W_s tile, and what a chunk costs besides (three launches
  // and the sums of grad_h_s: 20 us and 8 bytes per element at 5 TB/s, at 2.6e12 a second)
  const double logit = (double)tile_m * kd::kTileN * (double)logit_k;
  const double gw = (double)gw_rows * 256. * q.T_pad;
  const double fixed = 52e6 + (double)q.T * q.H_s * 4.2;
  auto cost = [&](int64_t width) {
    const int64_t n = (width + tile_m - 1) / tile_m;
    auto rounds = [&](int64_t tiles) { return (double)((tiles + q.n_cu - 1) / q.n_cu); };
    return logit * 0.5 * (rounds(n * q.n_tt) + rounds(n * masked_tt)) + gw * rounds((width + 255) / 256 * m_tiles) + fixed;
  };
  int64_t best = step;
  double best_cost = 1e300;
  for (int64_t vc = step; vc <= most; vc += step) {
    const int64_t full = q.V / vc, rest = q.V - full * vc;
    const double c = (double)full * cost(vc) + (rest > 0 ? cost(rest) : 0.);
    if (c <= best_cost) { best_cost = c; best = vc; }
  }
  return best;
}

// What a plan depends on besides the params.  The backward pass and the student's buffers are shared by all teachers of
// a call, so whatever decides about them looks at the whole call and never at one teacher's hidden size.
struct CallPlan {
  const int64_t* H_t = nullptr;    // hidden sizes of the call's teachers (null: the one of the params)
  int n_teachers = 1;
  size_t teacher_base = 0;         // where this teacher's block lies (0: right after the common part)
  bool repack_hv = false;          // [H][V] heads are re-packed even where they could be read in place
  bool lean = false;               // the smallest workspace: the eight-wave loop with the fewest ranges of the vocabulary
};

// Whether the strip loop (192-row tiles) or the eight-wave loop (128-row tiles) makes the logit tiles.
//  - A contracted element costs the strip loop 0.91 of what it costs the other, but its one wave per SIMD has nothing to
//    hide a tile's epilogue behind: that costs as much as 100 more elements (FKL, RKL), 200 (the row pass of JSD, TVD and
//    the skewed KLs) or 300 (AKL).
//  - The gradient kernel walks whole tiles in rounds of n_cu workgroups; the passes before it even out over ranges of the
//    vocabulary, down to a tile each.
// The constants are from 1178 sizes on an earlier state of both loops.  Steps of the present state (eight waves against strips): T = 512,
// H_t = 8192, H_s = 512, V = 512 183 against 230 us; T = 4096, H = 256 / 128, V = 151936 2.00 against 2.22 ms; T = 2048, H = 2048 / 1024,
// V = 4096 168 against 200 us and V = 100000 2.91 against 2.71 ms; T = 4096, H = 4096 / 1024, V = 151936 12.6 against 11.8 ms.  Over 60
// random sizes, T = 257 .. 16384, V = 256 .. 151936, every kind but AKL, 0.6 % is lost against the faster loop of each, 12 % at most (JSD,
// T = 12361, H = 3648 / 832, V = 2304; one loop for all of them: 3.1 % and 4.5 %); over 24 with [H][V] heads 0.3 %, 2.6 % at most.
// AKL's line lies too far to the eight-wave side: its 300 and its mean over seven passes are from when its search was four passes of
// compares on both loops.  With two passes of bins strips are ahead at each of 30 sizes (T = 259 .. 11168, H_t from 320, V = 288 .. 151936),
// and the rule loses 23 %, up to 48 % (T = 2182, H = 2112 / 320, V = 128256 9.35 against 6.33 ms).  It stands: the loops find the border
// between head and tail on different grids, so that results change within AKL's tolerance with it, and tests/test_plan_host.py holds
// two sizes to it.
// One token tile: the heads stream through once, nothing is shared, and the smaller tiles spread better over the CUs
// (T = 1, H = 4096 / 1024, V = 151936, JSD 1.09 against 1.37 ms; 24 sizes, T = 16 .. 256: 24 % on average, strips never ahead; at T = 256
// FKL the same, 1.05 against 1.04).
// `logit_k`: the contraction of one logit of all models, summed over the call's teachers.
bool strips_ahead(const Problem& q, int n_teachers, int64_t logit_k) {
  if (q.n_tt < 2) return false;
  double k = (double)logit_k / n_teachers;
  if (q.kind == KD_AKL) k -= q.K_s * 4. / 7.;                 // mean over the seven passes of the eight-wave loop
  const double epilogue = q.kind == KD_AKL ? 300. : q.kind >= KD_JSD ? 200. : 100.;
  const int spread = q.kind == KD_AKL ? 6 : q.kind >= KD_JSD ? 2 : 1;
  auto rounds = [&](int rows) {
    const int64_t tiles = (int64_t)q.n_tt * ((q.V + rows - 1) / rows);
    const double even = (double)tiles / q.n_cu;
    return (double)((tiles + q.n_cu - 1) / q.n_cu) + spread * (even > 1. ? even : 1.);
  };
  return rounds(192) * 192. * (0.91 * k + epilogue) < rounds(kd::kTileM) * kd::kTileM * k;
}

// Contraction length of one operand as the kernels read it: fp32 is three bf16 products side by side.
inline int64_t contraction(bool f32, int64_t H) { return round_up(f32 ? 3 * H : H, 64); }

// Tile counts, vocabulary chunk and split factors.  Depends on the params and on `call` only.
void plan(const kd_loss_params* p, Problem& q, Layout& L, bool with_backward, const CallPlan& call = CallPlan{}) {
  q.T = (int)p->T; q.V = (int)p->V; q.H_s = (int)p->H_s; q.H_t = (int)p->H_t;
  q.kind = p->kind; q.tau = p->tau; q.beta = p->beta;
  q.grad_f32 = p->grad_dtype == KD_F32;
  q.accumulate_grad_W = p->accumulate_grad_W;
  q.out_weight = p->loss_scale * ((p->flags & KD_FLAG_TAU2) ? p->tau * p->tau : 1.f);
  q.accumulate_loss = 0;
  q.n_cu = kd::kNumCU;
  // Operands as the kernels want them: bf16, K-contiguous, K a multiple of 64.  fp32 inputs are
  // split into bf16 high and low parts laid side by side along K (three products recover all
  // but the low x low term); bf16 inputs with an odd hidden size are zero-padded along K.
  q.in_f32 = p->in_dtype == KD_F32;
  q.w_hv = p->w_layout == KD_W_HV;
  q.t_fp8 = (p->flags & KD_FLAG_TEACHER_FP8) ? 1 : 0;
  q.t_scale = q.t_fp8 ? p->teacher_scale : 1.f;
  q.K_t = (int)contraction(q.in_f32, q.H_t);                    // fp8: H_t % 128 == 0, used as it is
  q.K_s = (int)contraction(q.in_f32, q.H_s);
  // A bf16 [V][H] head with rows off the 64-element grid is read in place with few tokens: what a row's last k-step covers behind the
  // row's end is loaded as 0, whatever lies there.  Its rows straddle cache lines, so with more tokens a padded copy is as good or
  // better: H = 1000 / 520, V = 50264, T = 64 203 (copies) against 141 us, T = 300 322 / 266, T = 2048 902 / 902, T = 4096 1815 / 1847;
  // T = 777, H = 4088 / 1000, V = 151936 3.63 / 3.23 ms.  Copies of small heads share the row map's launch and cost nothing.
  auto copied = [&](int64_t K, int64_t H) { return K != H && (q.w_hv || q.T > 1536 || 2 * q.V * K <= (4ll << 20)); };
  q.prep_Wt = q.in_f32 || copied(q.K_t, q.H_t);
  q.prep_Ws = q.in_f32 || copied(q.K_s, q.H_s);
  // [H][V] heads are read in place as k-major operands when they are bf16 with whole k-steps and a
  // vocabulary that the K-contiguous operand of the grad_h_s product can walk in whole 64-element
  // steps; otherwise both are re-packed (transposing) and the kernels see [V][K] copies
  // (an fp8 teacher head kept as [H][V] bytes is transposed into a [V][H] copy: the fp8 phase of the tile
  // loop reads K-contiguous rows only)
  q.w_hv_inplace = q.w_hv && !call.repack_hv && !q.t_fp8 && !q.prep_Wt && !q.prep_Ws && q.V % 64 == 0;
  if (q.w_hv && !q.w_hv_inplace) q.prep_Wt = q.prep_Ws = 1;
  // hidden states are also re-packed when a mask is given: valid tokens are compacted to the front
  // (the workspace is sized as if it were, since the size query does not see the mask)
  q.prep_ht = q.prep_hs = 1;
  q.T_pad = (int)round_up(q.T, kd::kTileN);
  q.n_tt = q.T_pad / kd::kTileN;
  int64_t logit_k = 0;       // elements contracted for one logit of every model of the call
  for (int i = 0; i < call.n_teachers; ++i) {
    const int64_t K_t = contraction(q.in_f32, call.H_t ? call.H_t[i] : p->H_t);
    logit_k += q.K_s + (q.t_fp8 ? K_t / 2 : K_t);        // (an e4m3 element costs half a bf16 one)
  }
  // The strip loop takes bf16 operands (heads [V][K], in place or re-packed, or [K][V] in place with 24-bit strides).  It
  // reads the hidden states from a packed copy, so they are re-packed whether a mask is given or not.
  q.strip = !q.t_fp8 && !(q.w_hv_inplace && q.V >= (1 << 23)) && !call.lean && strips_ahead(q, call.n_teachers, logit_k);
  q.n_vt = (q.V + kd::kTileM - 1) / kd::kTileM;
  // Vocabulary ranges of the statistics passes.  The device picks the actual number once it knows
  // how many token tiles survive the mask; this is the upper bound the buffers are sized for:
  // enough to keep every CU busy with up to half of the tokens masked, and to even out the rounds
  // of workgroups where there are many token tiles (65 of them: 31 ranges in eight full rounds, where eight ranges
  // leave the last of three rounds nearly empty).  A lean plan leaves that last point out.
  auto ranges = [&](int least) {
    int ns = 2 * ((q.n_cu + q.n_tt - 1) / q.n_tt);
    if (ns < least) ns = least;
    return ns > q.n_cu ? q.n_cu : ns;      // a single token tile is split over all CUs
  };
  const int strips = (q.V + 63) / 64;      // shortest worthwhile ranges: 64 rows, or a tile of the eight-wave loop
  const int lean_split = ranges(8) < q.n_vt ? ranges(8) : q.n_vt;
  const int full_split = ranges(32) < q.n_vt ? ranges(32) : q.n_vt;
  q.n_split = q.strip ? (ranges(32) < strips ? ranges(32) : strips) : call.lean ? lean_split : full_split;
  q.g_split = q.n_split;        // (bounded by the chunk's rows where it is used)

  const int64_t v_all = round_up(q.V, 256);
  const int64_t vc = p->vocab_chunk > 0 ? p->vocab_chunk : choose_chunk(q, v_all, logit_k);  // (the caller's: a multiple of 256)
  q.V_c = (int)(vc < v_all ? vc : v_all);

  // Tile and split-K of the grad_h_s product: the tiles of every chunk are rounds of n_cu workgroups, each of so many k-steps of 64
  // columns (the last chunk has those of the first, in fewer parts); 1.47, 1.19, 0.85, 0.62 us a k-step for 256, 192, 128, 64 hidden
  // rows (1.43 PFLOP/s down to 0.85); where the chunk of dz and of the head is more than the last-level cache keeps, the smaller tiles,
  // which have less in flight, take longer; 1.7 us a tile to start and 8.5 us per 256 rows to write its sums, 24 us with reading
  // them where there are several chunks; and every part is read once more at the end of the call (3.4 TB/s).  The mean of all tokens and
  // of an eighth of them masked, as in choose_chunk.  Fitted to 516 sizes, T = 100 .. 16384, H_s = 128 .. 4096, both head orders, each
  // with up to 18 tiles and splits (product and gradh_finish), and 180 more: 0.6 % behind the best one of each on average (2.5 % and more
  // with the last chunk and the cache left out).  T = 4096, H_s = 1024, V = 151936 128 rows x 2 parts 1123 us a call, 256 x 4 1213; T = 1024 256 x 16 353 us,
  // 128 x 8 372, 128 x 16 312; T = 512 256 x 32 142 us, 128 x 16 159.
  const int first_width = (int)(q.V < q.V_c ? q.V : q.V_c), steps_first = (first_width + 63) / 64;
  const int full_chunks = q.V / first_width, last_width = q.V - full_chunks * first_width;
  double least = 1e300;
  int sk = 1;
  for (int rows = call.lean ? 128 : 256; rows >= 64; rows -= 64) {
    if (q.w_hv_inplace && q.V > (1 << 23) && rows > 128) continue;              // (32-bit offsets: rows of 2 V bytes)
    const int i = rows / 64 - 1;
    const double in_cache[] = {0.62, 0.85, 1.19, 1.47}, from_memory[] = {0.82, 0.98, 1.26, 1.47};
    const double ends = 1.7 + rows / 256. * (q.V > q.V_c ? 24. : 8.5);
    const int64_t h_tiles = (q.H_s + rows - 1) / rows, tiles = h_tiles * q.n_tt, masked_tiles = h_tiles * ((q.n_tt * 7 + 7) / 8);
    auto rounds = [&](int64_t n) { return (double)((n + q.n_cu - 1) / q.n_cu); };
    for (int s = 1; s <= 32 && (s == 1 || q.V_c / s >= 512) && s <= steps_first; ++s) {
      if (call.lean && s > 1 && s * tiles > q.n_cu) break;
      const int steps = (steps_first + s - 1) / s;
      auto chunk = [&](int width) {
        const int n = (width + 63) / 64, parts = (n + steps - 1) / steps;
        const double step = 2. * width * (double)(q.T_pad + q.H_s) > 240e6 ? from_memory[i] : in_cache[i];
        return 0.5 * (rounds(tiles * parts) + rounds(masked_tiles * parts)) * ((steps < n ? steps : n) * step + ends);
      };
      const double t = full_chunks * chunk(first_width) + (last_width > 0 ? chunk(last_width) : 0.) +
                       (double)((steps_first + steps - 1) / steps) * q.T * q.H_s * 1.17e-6;
      if (t < least) { least = t; q.gh_rows = rows; sk = s; }
    }
  }
  q.ksteps_h = (steps_first + sk - 1) / sk;
  q.n_ksplit_h = (steps_first + q.ksteps_h - 1) / q.ksteps_h;   // every part is written by the first chunk

  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = (size_t)round_up((int64_t)(off + bytes), 256); return o; };
  L.meta = take(64);
  L.rowmap = take((size_t)q.T_pad * 4);
  L.inv = take((size_t)q.T * 4);
  L.row_loss = take((size_t)q.T_pad * 4);
  // partial sums per (vocabulary range, token): 5 statistics, 6 for AKL, whose search passes keep one sum per threshold or bin
  const int part_vals = q.kind != KD_AKL ? 5 : q.strip ? kd::kAklBins : kd::kAklThresholds;
  size_t partial_bytes = (size_t)q.n_split * part_vals * q.T_pad * 4;
  const size_t fine_at = partial_bytes;                  // behind the partials: the cells that AKL's row pass finds the border by
  if (q.strip && q.kind == KD_AKL) partial_bytes += (size_t)q.T_pad * kd::kAklBins * 16;
  if (!with_backward) L.partials = take(partial_bytes);
  L.prep_h_t = L.prep_W_t = L.prep_h_s = L.prep_W_s = 0;
  const size_t h_rows = q.strip ? q.T_pad : q.T;         // the strip loop reads whole token tiles of packed rows
  if (q.prep_hs) L.prep_h_s = take(h_rows * q.K_s * 2);
  if (q.prep_Ws) L.prep_W_s = take((size_t)q.V * q.K_s * 2);
  if (with_backward) {
    L.partials = off;           // read for the last time before the backward pass writes its first byte
    L.h_sT = take((size_t)round_up(q.H_s, 16) * q.T_pad * 2);
    L.dz = take((size_t)q.T_pad * q.V_c * 2);
    L.gh32 = take((size_t)q.n_ksplit_h * q.T * q.H_s * 4);
    if (off < L.partials + partial_bytes) off = (size_t)round_up((int64_t)(L.partials + partial_bytes), 256);
  } else {
    L.h_sT = L.dz = L.gh32 = off;
  }
  L.akl_fine = L.partials + fine_at;
  // what belongs to one teacher comes last, so that everything above sits at the same offsets for
  // every teacher of a multi-teacher call and the teachers' blocks can lie side by side
  L.common = off;
  if (call.teacher_base > off) off = call.teacher_base;
  L.rowinfo = take((size_t)q.T_pad * 16);
  L.akl = q.kind == KD_AKL ? take((size_t)q.T_pad * kd::kAklRows * 4) : 0;
  const size_t t_es = q.t_fp8 ? 1 : 2;
  if (q.prep_ht) L.prep_h_t = take(h_rows * q.K_t * t_es);
  if (q.prep_Wt) L.prep_W_t = take((size_t)q.V * q.K_t * t_es);
  L.total = off;
}

void carve(Problem& q, const Layout& L, void* ws) {
  char* b = static_cast<char*>(ws);
  q.meta = reinterpret_cast<int*>(b + L.meta);
  q.rowmap = reinterpret_cast<int*>(b + L.rowmap);
  q.inv = reinterpret_cast<int*>(b + L.inv);
  q.rowinfo = reinterpret_cast<float*>(b + L.rowinfo);
  q.akl = q.kind == KD_AKL ? reinterpret_cast<float*>(b + L.akl) : nullptr;
  q.akl_fine = reinterpret_cast<unsigned long long*>(b + L.akl_fine);
  q.row_loss = reinterpret_cast<float*>(b + L.row_loss);
  q.partials = reinterpret_cast<float*>(b + L.partials);
  q.h_sT = b + L.h_sT;
  q.dz = b + L.dz;
  q.gh32 = reinterpret_cast<float*>(b + L.gh32);
  q.user_h_t = q.h_t; q.user_W_t = q.W_t; q.user_h_s = q.h_s; q.user_W_s = q.W_s;
  // without a mask the eight-wave loop uses the hidden states in place unless they need re-packing anyway
  if (!q.mask && !q.strip) {
    q.prep_ht = q.prep_Wt || q.K_t != q.H_t;
    q.prep_hs = q.prep_Ws || q.K_s != q.H_s;
  }
  if (q.prep_ht) q.h_t = b + L.prep_h_t;
  if (q.prep_Wt) q.W_t = b + L.prep_W_t;
  if (q.prep_hs) q.h_s = b + L.prep_h_s;
  if (q.prep_Ws) q.W_s = b + L.prep_W_s;
}



// Benchmark aid: bracket the launches of one kernel family with caller-supplied events.
struct ProfileHook {
  int which = -1;
  hipEvent_t* events = nullptr;
  int n_events = 0;
  int used = 0;     // pairs recorded
};
thread_local ProfileHook g_hook;
thread_local long long* g_clock_out = nullptr;   // kd_loss_profile_clock

struct ProfileScope {
  bool on;
  hipStream_t st;
  ProfileScope(int which, hipStream_t s) : on(false), st(s) {
    if (g_hook.which == which && g_hook.events && 2 * g_hook.used + 1 < g_hook.n_events) {
      on = true;
      (void)hipEventRecord(g_hook.events[2 * g_hook.used], st);
    }
  }
  ~ProfileScope() {
    if (on) {
      (void)hipEventRecord(g_hook.events[2 * g_hook.used + 1], st);
      ++g_hook.used;
    }
  }
};

// -DKD_TRACE_ERRORS (a debugging build) names the failing call on stderr.
#ifdef KD_TRACE_ERRORS
#define KD_TRY(expr)                                                                              \
  do {                                                                                            \
    const hipError_t kd_e_ = (expr);                                                              \
    if (kd_e_ != hipSuccess) {                                                                    \
      std::fprintf(stderr, "libkdloss: %s:%d: %s -> %s\n", __FILE__, __LINE__, #expr, hipGetErrorString(kd_e_)); \
      return KD_ERR_LAUNCH;                                                                       \
    }                                                                                             \
  } while (0)
#else
#define KD_TRY(expr)                                \
  do {                                              \
    if ((expr) != hipSuccess) return KD_ERR_LAUNCH; \
  } while (0)
#endif

// Forward pass of one teacher.  The token compaction and the student operands are shared by the
// teachers of a call: only the first one makes them.  `backward`: a backward pass follows (behind the last teacher).
kd_status run_forward(const Problem& q, hipStream_t st, bool backward, bool first_teacher = true) {
  KD_TRY(kd::launch_operands(q, first_teacher, first_teacher, true, st));
  {
    ProfileScope ps(KD_PROF_STATS, st);
    KD_TRY(kd::launch_stats(q, st));
  }
  KD_TRY(kd::launch_combine(q, st));
  if (q.kind == KD_AKL) {
    // the teacher probability that splits each token's vocabulary into head and tail, by a multi-way search
    // over the teacher logit tiles; then the head and tail gaps, which weigh the two KLs
    for (int pass = 0; pass < kd::akl_search_passes(q.strip); ++pass) KD_TRY(kd::launch_akl_search(q, pass, st));
    {
      ProfileScope ps(KD_PROF_ROWS, st);
      KD_TRY(kd::launch_rows(q, st));
    }
    KD_TRY(kd::launch_akl_weights(q, st));
  } else if (q.kind >= KD_JSD) {   // divergences that need both log-sum-exps before their row value
    {
      ProfileScope ps(KD_PROF_ROWS, st);
      KD_TRY(kd::launch_rows(q, st));
    }
    KD_TRY(kd::launch_combine_rows(q, st));
  }
  KD_TRY(kd::launch_finalize(q, backward, st));       // (h_s^T once: the hidden-row operand of grad_W_s)
  return KD_OK;
}

// Backward pass: dL/dz_s chunk by chunk and the two products.  With several teachers the chunk of
// dL/dz_s is the sum over the teachers (each gradient kernel adds its weighted share to the bf16
// staging buffer), so the products run once per chunk whatever the number of teachers.  grad_h_s is
// summed in fp32 over the chunks and converted once at the end.
kd_status run_backward(const Problem* qs, int n_teachers, hipStream_t st) {
  const Problem& q = qs[0];          // everything on the student side is the same for all teachers
  for (int64_t v0 = 0; v0 < q.V; v0 += q.V_c) {
    const int width = (int)((q.V - v0 < q.V_c) ? q.V - v0 : q.V_c);
    for (int k = 0; k < n_teachers; ++k) {
      ProfileScope ps(KD_PROF_GRAD, st);
      KD_TRY(kd::launch_grad_chunk(qs[k], (int)v0, width, k > 0, st));
    }
    {
      ProfileScope ps(KD_PROF_GEMM_GRAD_W, st);
      KD_TRY(kd::launch_grad_W(q, (int)v0, width, st));
    }
    {
      ProfileScope ps(KD_PROF_GEMM_GRAD_H, st);
      KD_TRY(kd::launch_grad_h(q, (int)v0, width, v0 == 0, st));
    }
  }
  KD_TRY(kd::launch_gradh_finish(q, st));
  return KD_OK;
}


kd_status check_buffers(const kd_loss_params* params, const void* h_t, const void* W_t, const void* h_s,
                        const void* W_s, const uint8_t* mask, float* loss, void* workspace,
                        size_t workspace_bytes, bool backward, void* grad_h_s, void* grad_W_s,
                        Problem& q, Layout& L, const CallPlan& call = CallPlan{}) {
  kd_status s = check_params(params);
  if (s != KD_OK) return s;
  if (!h_t || !W_t || !h_s || !W_s || !loss || !workspace) return KD_ERR_NULL;
  if (backward && (!grad_h_s || !grad_W_s)) return KD_ERR_NULL;
  if (!aligned16(h_t) || !aligned16(W_t) || !aligned16(h_s) || !aligned16(W_s)) return KD_ERR_ALIGN;
  if (backward && (!aligned16(grad_h_s) || !aligned16(grad_W_s))) return KD_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return KD_ERR_ALIGN;
  plan(params, q, L, backward, call);
  if (workspace_bytes < L.total) return KD_ERR_WORKSPACE;
  q.h_t = h_t; q.W_t = W_t; q.h_s = h_s; q.W_s = W_s; q.mask = mask;
  q.clock_out = g_clock_out;
  q.loss = loss;
  q.grad_h_s = grad_h_s; q.grad_W_s = grad_W_s;
  carve(q, L, workspace);
  return KD_OK;
}

// The student side of a multi-teacher call (how [H][V] heads are read, which student operands are
// re-packed, where the shared buffers lie) must be the same for every teacher.  Whether [H][V] heads can
// be read in place depends on each teacher's hidden size, so the decision is taken here once: if any
// teacher needs the re-packing path, all of them (and the student head) take it.  Also runs the parameter
// checks of every teacher.
kd_status multi_call_plan(const kd_loss_params* params, int n_teachers, const int64_t* H_t, CallPlan& call) {
  call.H_t = H_t;
  call.n_teachers = n_teachers;
  for (int k = 0; k < n_teachers; ++k) {
    kd_loss_params pk = *params;
    pk.H_t = H_t[k];
    if (pk.flags & KD_FLAG_TEACHER_FP8) pk.teacher_scale = 1.f;   // checked per teacher by the call itself
    kd_status s = check_params(&pk);
    if (s != KD_OK) return s;
    Problem q{};
    Layout L{};
    plan(&pk, q, L, true);
    if (q.w_hv && !q.w_hv_inplace) call.repack_hv = true;
  }
  return KD_OK;
}

// The backward pass and the student operands are laid out by teacher 0's plan: every teacher's must agree with it.
// (By construction they do; the size query and the call both ask.)
bool same_student_plan(const Problem& a, const Layout& A, const Problem& b, const Layout& B) {
  return A.common == B.common && A.dz == B.dz && A.h_sT == B.h_sT && A.gh32 == B.gh32 && A.prep_h_s == B.prep_h_s &&
         A.prep_W_s == B.prep_W_s && a.w_hv_inplace == b.w_hv_inplace && a.prep_Ws == b.prep_Ws &&
         a.prep_hs == b.prep_hs && a.V_c == b.V_c && a.strip == b.strip && a.n_split == b.n_split;
}

}  // namespace

extern "C" {

kd_status kd_loss_workspace_size(const kd_loss_params* params, size_t* bytes) {
  if (!bytes) return KD_ERR_NULL;
  kd_status s = check_params(params);
  if (s != KD_OK) return s;
  Problem q{};
  Layout L{};
  plan(params, q, L, true);
  *bytes = L.total;
  return KD_OK;
}

kd_status kd_loss_plan_info(const kd_loss_params* params, int64_t* vocab_chunk, int64_t* n_launches) {
  kd_status s = check_params(params);
  if (s != KD_OK) return s;
  Problem q{};
  Layout L{};
  plan(params, q, L, true);
  const int64_t chunks = (q.V + q.V_c - 1) / q.V_c;
  if (vocab_chunk) *vocab_chunk = q.V_c;
  // compaction with the copies of the heads, copies of the hidden states (as with a mask), heads turned, statistics + merge,
  // row pass + merge, AKL's search as on the eight-wave loop, loss and h_s^T, per chunk the gradient kernel and the two products, grad_h_s conversion
  if (n_launches)
    *n_launches = 1 + 1 + (q.w_hv ? q.prep_Wt + q.prep_Ws : 0) + 2 + (q.kind >= KD_JSD ? 2 : 0) +
                  (q.kind == KD_AKL ? 2 * kd::akl_search_passes(false) : 0) + 1 + chunks * 3 + 1;
  return KD_OK;
}

kd_status kd_loss_plan_loop(const kd_loss_params* params, int32_t* loop) {
  if (!loop) return KD_ERR_NULL;
  kd_status s = check_params(params);
  if (s != KD_OK) return s;
  Problem q{};
  Layout L{};
  plan(params, q, L, true);
  *loop = q.strip;
  return KD_OK;
}

kd_status kd_loss_plan_grad_h(const kd_loss_params* params, int32_t* tile_rows, int32_t* parts) {
  kd_status s = check_params(params);
  if (s != KD_OK) return s;
  Problem q{};
  Layout L{};
  plan(params, q, L, true);
  if (tile_rows) *tile_rows = q.gh_rows;
  if (parts) *parts = q.n_ksplit_h;
  return KD_OK;
}

kd_status kd_loss_fwd(const kd_loss_params* params, const void* h_t, const void* W_t, const void* h_s,
                      const void* W_s, const uint8_t* mask, float* loss, float* per_token_loss,
                      void* workspace, size_t workspace_bytes, void* hip_stream) {
  Problem q{};
  Layout L{};
  kd_status s = check_buffers(params, h_t, W_t, h_s, W_s, mask, loss, workspace, workspace_bytes, false,
                              nullptr, nullptr, q, L);
  if (s != KD_OK) return s;
  q.per_token_loss = per_token_loss;
  return run_forward(q, static_cast<hipStream_t>(hip_stream), false);
}

kd_status kd_loss_fwd_bwd(const kd_loss_params* params, const void* h_t, const void* W_t, const void* h_s,
                          const void* W_s, const uint8_t* mask, float* loss, float* per_token_loss,
                          void* grad_h_s, void* grad_W_s, void* workspace, size_t workspace_bytes,
                          void* hip_stream) {
  Problem q{};
  Layout L{};
  kd_status s = check_buffers(params, h_t, W_t, h_s, W_s, mask, loss, workspace, workspace_bytes, true,
                              grad_h_s, grad_W_s, q, L);
  if (s != KD_OK) return s;
  q.per_token_loss = per_token_loss;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);

  s = run_forward(q, st, true);
  if (s != KD_OK) return s;
  return run_backward(&q, 1, st);
}

kd_status kd_loss_fwd_bwd_static(const kd_loss_params* params, const void* h_t, const void* W_t, const void* h_s,
                                 const void* W_s, const uint8_t* mask, float* loss, float* per_token_loss,
                                 void* grad_h_s, void* grad_W_s, void* hip_stream) {
  kd_status s = check_params(params);
  if (s != KD_OK) return s;
  // the plan: the caller's chunk, else the widest one that fits the array; at each width a lean plan before the next
  // narrower one
  kd_loss_params pp = *params;
  CallPlan call;
  auto fits = [&]() {
    for (int lean = 0; lean < 2; ++lean) {
      Problem q{};
      Layout L{};
      call.lean = lean != 0;
      plan(&pp, q, L, true, call);
      if (L.total <= KD_STATIC_SCRATCH_BYTES) return true;
    }
    return false;
  };
  bool fit = fits();
  if (!fit && params->vocab_chunk == 0) {
    Problem q{};
    Layout L{};
    plan(params, q, L, true);
    for (int vc = 1 << 19; vc >= 256 && !fit; vc >>= 1) {
      if (vc >= q.V_c) continue;
      pp.vocab_chunk = vc;
      fit = fits();
    }
  }
  if (!fit) return KD_ERR_TOO_LARGE;
  // every remaining host-side check, with a stand-in for the scratch address (nothing is dereferenced)
  Problem q{};
  Layout L{};
  s = check_buffers(&pp, h_t, W_t, h_s, W_s, mask, loss, reinterpret_cast<void*>(uintptr_t{256}),
                    KD_STATIC_SCRATCH_BYTES, true, grad_h_s, grad_W_s, q, L, call);
  if (s != KD_OK) return s;
  // device address of this GPU's copy of the array, looked up once per device
  static void* ptr_of_device[64];
  static std::atomic<uint64_t> have{0};
  int dev = 0;
  KD_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return KD_ERR_UNSUPPORTED;
  const uint64_t bit = 1ull << dev;
  if (!(have.load(std::memory_order_acquire) & bit)) {
    void* ptr = nullptr;
    KD_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return KD_ERR_LAUNCH;
    ptr_of_device[dev] = ptr;
    have.fetch_or(bit, std::memory_order_release);
  }
  void* const ptr = ptr_of_device[dev];
  q = Problem{};
  s = check_buffers(&pp, h_t, W_t, h_s, W_s, mask, loss, ptr, KD_STATIC_SCRATCH_BYTES, true, grad_h_s, grad_W_s, q, L,
                    call);
  if (s != KD_OK) return s;
  q.per_token_loss = per_token_loss;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  s = run_forward(q, st, true);
  if (s != KD_OK) return s;
  return run_backward(&q, 1, st);
}

kd_status kd_loss_workspace_size_multi(const kd_loss_params* params, int n_teachers, const int64_t* H_t,
                                       size_t* bytes) {
  if (!bytes || !params || !H_t) return KD_ERR_NULL;
  if (n_teachers < 1 || n_teachers > 16) return KD_ERR_PARAM;
  CallPlan call;
  kd_status s = multi_call_plan(params, n_teachers, H_t, call);
  if (s != KD_OK) return s;
  Problem q0{};
  Layout L0{};
  for (int k = 0; k < n_teachers; ++k) {  // teacher blocks lie side by side after the common part
    kd_loss_params pk = *params;
    pk.H_t = H_t[k];
    if (pk.flags & KD_FLAG_TEACHER_FP8) pk.teacher_scale = 1.f;   // the size does not depend on the scales
    Problem q{};
    Layout L{};
    plan(&pk, q, L, true, call);
    if (k == 0) { q0 = q; L0 = L; }
    if (!same_student_plan(q0, L0, q, L)) return KD_ERR_UNSUPPORTED;
    call.teacher_base = L.total;
  }
  *bytes = call.teacher_base;
  return KD_OK;
}

kd_status kd_loss_fwd_bwd_multi(const kd_loss_params* params, int n_teachers, const void* const* h_t,
                                const void* const* W_t, const int64_t* H_t, const float* weights,
                                const float* teacher_scales,
                                const void* h_s, const void* W_s, const uint8_t* mask, float* loss,
                                float* per_token_loss, void* grad_h_s, void* grad_W_s, void* workspace,
                                size_t workspace_bytes, void* hip_stream) {
  if (!params || !h_t || !W_t || !H_t || !weights) return KD_ERR_NULL;
  if (n_teachers < 1 || n_teachers > 16) return KD_ERR_PARAM;
  const bool fp8 = (params->flags & KD_FLAG_TEACHER_FP8) != 0;
  if (fp8 && !teacher_scales) return KD_ERR_NULL;
  // all checks for all teachers before the first launch
  Problem q[16];
  Layout L[16];
  CallPlan call;
  {
    kd_status s = multi_call_plan(params, n_teachers, H_t, call);
    if (s != KD_OK) return s;
  }
  for (int k = 0; k < n_teachers; ++k) {
    if (!std::isfinite(weights[k])) return KD_ERR_PARAM;
    kd_loss_params pk = *params;
    pk.H_t = H_t[k];
    if (fp8) pk.teacher_scale = teacher_scales[k];
    q[k] = Problem{};
    kd_status s = check_buffers(&pk, h_t[k], W_t[k], h_s, W_s, mask, loss, workspace, workspace_bytes, true,
                                grad_h_s, grad_W_s, q[k], L[k], call);
    if (s != KD_OK) return s;
    if (!same_student_plan(q[0], L[0], q[k], L[k])) return KD_ERR_UNSUPPORTED;
    call.teacher_base = L[k].total;
    q[k].per_token_loss = per_token_loss;
    q[k].out_weight *= weights[k];     // scales this teacher's loss and its share of dL/dz_s
    q[k].accumulate_loss = k > 0;
  }
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  for (int k = 0; k < n_teachers; ++k) {
    kd_status s = run_forward(q[k], st, k + 1 == n_teachers, k == 0);
    if (s != KD_OK) return s;
  }
  return run_backward(q, n_teachers, st);
}

kd_status kd_quantize_e4m3(const void* src, int32_t src_dtype, int64_t n, float scale, void* dst,
                           void* hip_stream) {
  if (!src || !dst) return KD_ERR_NULL;
  if (n < 1 || n > ((int64_t)1 << 40)) return KD_ERR_SHAPE;
  if (src_dtype != KD_BF16 && src_dtype != KD_F32) return KD_ERR_PARAM;
  if (!(scale > 0.f && scale < INFINITY)) return KD_ERR_PARAM;
  if (!aligned16(src) || !aligned16(dst)) return KD_ERR_ALIGN;
  KD_TRY(kd::launch_quantize_e4m3(src, src_dtype == KD_F32, n, 1.f / scale, dst, static_cast<hipStream_t>(hip_stream)));
  return KD_OK;
}

kd_status kd_probe_mfma_rate(const void* operands, int iters, float* sink, void* hip_stream) {
  if (!operands || !sink) return KD_ERR_NULL;
  if (iters < 1 || iters > (1 << 24)) return KD_ERR_PARAM;
  if (!aligned16(operands) || !aligned16(sink)) return KD_ERR_ALIGN;
  KD_TRY(kd::launch_mfma_probe(operands, iters, sink, g_clock_out, kd::kNumCU, static_cast<hipStream_t>(hip_stream)));
  return KD_OK;
}

kd_status kd_loss_profile_clock(void* two_int64_device) {
  if (reinterpret_cast<uintptr_t>(two_int64_device) & 7u) return KD_ERR_ALIGN;
  g_clock_out = static_cast<long long*>(two_int64_device);
  return KD_OK;
}

kd_status kd_loss_profile_hook(int which, void** events, int n_events) {
  if (which < 0) {
    g_hook = ProfileHook{};
    return KD_OK;
  }
  if (which > KD_PROF_GEMM_GRAD_H) return KD_ERR_PARAM;
  if (!events || n_events < 2) return KD_ERR_NULL;
  g_hook.which = which;
  g_hook.events = reinterpret_cast<hipEvent_t*>(events);
  g_hook.n_events = n_events;
  g_hook.used = 0;
  return KD_OK;
}

int kd_loss_profile_count(void) { return g_hook.used; }

const char* kd_build_info(void) { return kd::build_info(); }
int kd_build_ablation(void) { return 0; }

const char* kd_status_string(kd_status status) {
  switch (status) {
    case KD_OK: return "ok";
    case KD_ERR_NULL: return "a required pointer is NULL";
    case KD_ERR_SHAPE: return "T, H_t, H_s or V out of range";
    case KD_ERR_ALIGN: return "pointer not 16-byte aligned or size not a multiple of 8";
    case KD_ERR_PARAM: return "invalid tau, beta, enum value or flag";
    case KD_ERR_WORKSPACE: return "workspace too small";
    case KD_ERR_UNSUPPORTED: return "valid request not implemented by this build";
    case KD_ERR_LAUNCH: return "HIP launch failed";
    case KD_ERR_TOO_LARGE: return "problem needs more scratch memory than the library's static array holds";
  }
  return "unknown status";
}

}  // extern "C"
