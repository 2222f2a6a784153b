// Device-side pieces that the kernels of several source files share.
#pragma once
#include "kd_launch.h"
#include "kd_mfma.hpp"
#include "kd_strip.hpp"

#include <atomic>

namespace kd {

// Number of this workgroup in a grid of flat_grid (kd_launch.h).
__device__ __forceinline__ int64_t flat_group() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

// Workgroups are dealt to the 8 XCDs round-robin by workgroup id.  Renumber so
// that consecutive logical ids sit on one XCD (and share its L2).
__device__ __forceinline__ int xcd_logical_id(int b, int G) {
  const int x = b % 8, q = G / 8, r = G % 8;       // XCD x holds q (+1 if x < r) of the G workgroups
  return x * q + (x < r ? x : r) + b / 8;
}

// Device-side plan, written by make_rowmap once the mask has been counted (the host never
// learns how many tokens are valid, so everything that depends on it is decided on the device).
// META_N_SPLIT: vocabulary ranges per token tile in the statistics passes; META_G_SPLIT, META_G_SPLIT_LAST: in the
// gradient kernel, for a full chunk and for the last one (strip loop).
enum { META_N_VALID = 0, META_N_TT = 1, META_N_SPLIT = 2, META_T_EFF = 3, META_G_SPLIT = 4, META_G_SPLIT_LAST = 5,
       META_WORDS = 6 };
__device__ __forceinline__ int meta_get(const int* meta, int i) { return uniform(meta[i]); }

// Index q over n_tt token tiles x n_split vocabulary splits: the token tiles in groups of at most four (of sizes
// that differ by one where four does not divide them), a group's splits one after the other.  32 consecutive
// indices, the workgroups of an XCD, then cover 4 x 8: the shape that streams the fewest rows into one L2.
__device__ __forceinline__ void group_decode(int q, int n_tt, int n_split, int& tt, int& split) {
  const int ng = (n_tt + 3) / 4, small = n_tt / ng, n_big = n_tt - small * ng;
  const int big_units = n_big * (small + 1) * n_split;
  int g = small, base = 0;
  if (q < big_units) g = small + 1;
  else { q -= big_units; base = n_big * (small + 1); }
  const int grp = q / (g * n_split), w = q - grp * g * n_split;
  tt = base + grp * g + w % g;
  split = w / g;
}

// dL/dz_s of a vocabulary chunk is kept in the order in which a lane of a finished logit tile holds it and in which the
// products read it: [64-token panel][32-column sub-step][16-token block][lane][8], lane 16 g + t with the columns
// 4 g .. + 3 and 16 + 4 g .. + 3 of token t of the block.  As the token operand of grad_h_s a lane's 16 bytes are its share of an
// MFMA (eight of the 32 columns contracted); as the column operand of grad_W_s they go through the transposing LDS reads.
// The panels are V_c columns apart.  Element offset of the 16 bytes of (panel, column sub-step, block, lane):
__device__ __forceinline__ int64_t dz_chunk(int ldz, int panel, int sub, int blk, int lane) {
  return (int64_t)panel * 64 * ldz + ((int64_t)(sub * 4 + blk) * 64 + lane) * 8;
}
// Column of row `row` (0 .. 15) of block i of an A_DZ tile (strip_loop).
__device__ __forceinline__ int dz_column(int i, int row) {
  return 32 * (i >> 1) + 16 * ((row >> 2) & 1) + 8 * (i & 1) + 4 * (row >> 3) + (row & 3);
}

#define KD_STRIP_KERNEL __global__ __launch_bounds__(StripCfg::NT, 1) __attribute__((amdgpu_waves_per_eu(1, 1)))

// Launch of a kernel that needs more dynamic LDS than the default limit.  The limit is a property of
// the kernel on a device: it is raised once per kernel and device (one flag word per instantiation,
// one bit per device), not on every launch.
template <auto Kern>
static hipError_t launch_big(int grid, int threads, int smem_bytes, hipStream_t st, const void* args_ptr) {
  static std::atomic<uint64_t> attr_done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (!(attr_done.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)Kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem_bytes);
    if (e != hipSuccess) return e;
    attr_done.fetch_or(bit, std::memory_order_release);
  }
  void* params[] = {const_cast<void*>(args_ptr)};
  return hipLaunchKernel((const void*)Kern, dim3(grid), dim3(threads), params, smem_bytes, st);
}

}  // namespace kd
