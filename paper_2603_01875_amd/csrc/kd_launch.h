// Host-side interface between the C ABI layer and the kernel launchers.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

namespace kd {

constexpr int kNumCU = 256;            // MI355X: 8 XCDs x 32 CUs; persistent grids are sized for it
constexpr int kTileM = 128;            // vocabulary rows per logit tile of the eight-wave loop
constexpr int kTileN = 256;            // token rows per logit tile

// Hidden rows per tile of grad_W_s (beside 256 vocabulary columns) for a chunk of `width` columns: of 128, 192, 256 the number whose
// tiles finish soonest on n_cu workgroups, a tile's price being its rows and 64 more.  Over 90 sizes (T = 64 .. 16384, H_s = 64 .. 4032,
// chunks of 800 to 152000 columns) 0.4 % behind the fastest on average, 7 % at most; by the hidden rows alone, without the rounds of
// workgroups, it was 18 % (T = 4096, H_s = 448, V = 10640, 84 tiles of 256 rows 75 us, 168 of 128 rows 53; T = 12271, H_s = 512, V = 151936
// 4.38 ms with 256, 2.89 with 128).
inline int grad_W_tile(int64_t H_s, int64_t width, int n_cu) {
  int best = 256;
  int64_t low = INT64_MAX;
  for (int rows = 256; rows >= 128; rows -= 64) {
    const int64_t tiles = (width + 255) / 256 * ((H_s + rows - 1) / rows);
    const int64_t price = (tiles + n_cu - 1) / n_cu * (rows + 64);
    if (price < low) { low = price; best = rows; }
  }
  return best;
}

// Shape of a grid of `groups` workgroups of up to 1024 threads that are numbered in a row (kernels: flat_group).  A grid has fewer
// than 2^32 threads along one axis, so beyond 2^21 workgroups it takes a second one, and the last row has some too many.
struct FlatGrid { uint32_t x, y; };
inline FlatGrid flat_grid(int64_t groups) {
  const int64_t most = (int64_t)1 << 21;
  return groups <= most ? FlatGrid{(uint32_t)groups, 1} : FlatGrid{(uint32_t)most, (uint32_t)((groups + most - 1) / most)};
}

// Everything a launch needs, resolved by the planner in kd_api.hip.
struct Problem {
  int T, V, H_s, H_t;
  int kind;
  float tau, beta;
  int grad_f32;
  int accumulate_grad_W;
  float out_weight;        // factor on the loss and the gradients of this call (teacher weight, tau^2)
  int accumulate_loss;     // add to *loss and per_token_loss instead of overwriting them
  const void *h_t, *W_t, *h_s, *W_s;                   // bf16 [rows][K_t or K_s] as the kernels read them
  const void *user_h_t, *user_W_t, *user_h_s, *user_W_s;  // the caller's arrays
  int in_f32;                   // inputs are fp32
  int w_hv;                     // the caller's heads and grad_W_s are stored [H][V]
  int w_hv_inplace;             // ... and the kernels read the heads in that order, in place (else they are
                                // re-packed into [V][K] copies like any operand that needs re-packing)
  long long* clock_out;         // measurement aid, see kd_loss_profile_clock (null unless set)
  int t_fp8;                    // teacher operands are e4m3 bytes (K_t = H_t elements = bytes per row)
  float t_scale;                // ... and z_t = t_scale * (product of the codes)
  int prep_ht, prep_Wt, prep_hs, prep_Ws;   // which operands are re-packed into the workspace
  int K_t, K_s;                 // contraction lengths of the (re-packed) logit operands, multiples of 64
  const uint8_t* mask;
  float* loss;
  float* per_token_loss;
  void *grad_h_s, *grad_W_s;
  // plan
  int strip;                    // strip loop on packed hidden states (bf16 logit operands, heads [V][K] or [K][V]), else eight-wave loop
  int g_split;                  // strip loop: most vocabulary ranges per token tile in the gradient kernel
  int gh_rows;                  // hidden rows per tile of the grad_h_s product
  int T_pad, n_tt, n_vt, n_split, V_c, n_ksplit_h, ksteps_h, n_cu;
  // workspace carve-up
  int* meta;           // device-side plan written by the row-map kernel
  int* rowmap;         // [T_pad] compacted index -> token
  int* inv;            // [T] token -> compacted index or -1
  float* rowinfo;      // [T_pad][4]
  float* akl;          // AKL only: [kAklRows][T_pad] per-token values between its passes (null otherwise)
  unsigned long long* akl_fine;  // ... strip loop: [T_pad][kAklBins][2] sums of its row pass, behind the partials
  float* row_loss;     // [T_pad]
  float* partials;     // [n_split][values of the pass][T_pad]
  void* h_sT;          // bf16, T_pad tokens x H_s rounded up to 16, packed (pack_columns)
  void* dz;            // bf16, T_pad x V_c, in the order of dz_chunk (kd_common.hpp)
  float* gh32;         // [n_ksplit_h][T][H_s]
};

// the row map (first teacher of a call), and the operand copies of the student and of the teacher that the call needs
hipError_t launch_operands(const Problem& p, bool rowmap, bool student, bool teacher, hipStream_t st);
hipError_t launch_mfma_probe(const void* operands, int iters, float* sink, long long* clock_out, int n_cu,
                             hipStream_t st);
hipError_t launch_quantize_e4m3(const void* src, int src_f32, int64_t n, float inv_scale, void* dst, hipStream_t st);
hipError_t launch_stats(const Problem& p, hipStream_t st);
hipError_t launch_combine(const Problem& p, hipStream_t st);
hipError_t launch_rows(const Problem& p, hipStream_t st);
hipError_t launch_akl_search(const Problem& p, int pass, hipStream_t st);      // one search pass and its merge
hipError_t launch_akl_weights(const Problem& p, hipStream_t st);
// AKL's border lies on a grid of cells between a lowest base-2 log-probability and 1e-3 above a token's largest one: 17^4 of them from
// 40 below the largest on the eight-wave loop (4.8e-4 each), 44^3 from wherever less than 1 - mu can lie below on the strip loop
// (4.7e-4 at most, 1e-5 for a flat teacher).
constexpr int kAklThresholds = 16;     // eight-wave loop: four passes, 17-fold narrowing each (the kernels' AKL_K)
constexpr int kAklBins = 44;           // strip loop: passes by bins of 44^2 and 44 cells; the row pass (or a third) finds the cell
constexpr int kAklCells = kAklBins * kAklBins * kAklBins;
constexpr int kAklRows = 7;            // values kept per token (AKL_* in kd_logits.hpp)
inline int akl_search_passes(bool strip) { return strip ? 3 : 4; }
hipError_t launch_combine_rows(const Problem& p, hipStream_t st);
// ... and, for the backward pass, h_s of the compacted tokens transposed and packed for grad_W_s, from the caller's array
hipError_t launch_finalize(const Problem& p, bool pack_h_s, hipStream_t st);
hipError_t launch_grad_chunk(const Problem& p, int v0, int width, bool accumulate, hipStream_t st);
// the backward products on the chunk of `width` columns from v0; `first`: grad_h_s's parts are written, not added to
hipError_t launch_grad_W(const Problem& p, int v0, int width, hipStream_t st);
hipError_t launch_grad_h(const Problem& p, int v0, int width, bool first, hipStream_t st);
hipError_t launch_gradh_finish(const Problem& p, hipStream_t st);
const char* build_info();     // compile-time configuration of the kernels (tile shapes)
}  // namespace kd
