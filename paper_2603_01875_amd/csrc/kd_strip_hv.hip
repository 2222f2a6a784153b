// The strip loop's logit kernels for bf16 heads kept as [H][V] and read in place (those for [V][H] heads: kd_kernels.hip).
//
// The vocabulary is the contiguous index, so a stage of the LDS holds k-rows of a tile, and the fragments come by the transposing
// reads of the backward products, in the order of k in which dz lies (A_KMAJOR_DZ in kd_strip.hpp); pack_rows packs
// the hidden states in the same order, and nothing else differs.  Bound as the [V][H] kernels are, by the matrix pipe and the
// chip's power.  Steps against the eight-wave loop, which takes both operands through the LDS: T = 2048, H = 4096 / 1024, V = 151936
// 6.80 -> 6.19 ms (JSD 9.54 -> 8.90), T = 4096 13.33 -> 12.51, T = 512 1957 -> 1766 us, T = 1024, H = 8192 / 2048, V = 128256 5.98 -> 5.47
// ms, T = 2048, H = 8192 / 512, V = 6144 523 -> 428 us.  strips_ahead (kd_api.hip) draws the line as for [V][H] heads: beside it
// the two are as close, T = 300, V = 24576 364 -> 317 us.
#include "kd_logits.hpp"

namespace kd {

template <int KIND>
KD_STRIP_KERNEL void stats_strip_hv_kern(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  StripWork<true> work(a, meta_get(a.meta, META_N_SPLIT));
  StripStatsEpi<KIND> epi(a.c, smem);
  StripEpi<StripStatsEpi<KIND>> drive(epi);
  LoopClock clk(a);
  strip_loop<2, true, StripCfg, A_KMAJOR_DZ>(work, drive, smem);
  clk.stop(a);
  if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
}

template <int KIND>
KD_STRIP_KERNEL void rows_strip_hv_kern(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  StripWork<true> work(a, meta_get(a.meta, META_N_SPLIT));
  if constexpr (KIND == 6) {
    AklRowsEpi epi(a, work.tt, akl_crowded(a.akl, a.T_pad, work.tt), smem);
    StripEpi<AklRowsEpi> drive(epi);
    strip_loop<2, true, StripCfg, A_KMAJOR_DZ>(work, drive, smem);
    if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
  } else {
    RowsEpi<KIND, StripGeo> epi(a, work.tt);
    StripEpi<RowsEpi<KIND, StripGeo>> drive(epi);
    strip_loop<2, true, StripCfg, A_KMAJOR_DZ>(work, drive, smem);
    if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
  }
}

template <int KIND>
KD_STRIP_KERNEL void grad_strip_hv_kern(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  StripWork<true> work(a, meta_get(a.meta, a.last_chunk ? META_G_SPLIT_LAST : META_G_SPLIT));
  GradEpi<KIND, StripGeo> epi(a, smem);
  StripEpi<GradEpi<KIND, StripGeo>> drive(epi);
  strip_loop<2, false, StripCfg, A_KMAJOR_DZ>(work, drive, smem);
}

KD_STRIP_KERNEL void search_strip_hv_kern(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  StripWork<true> work(a, meta_get(a.meta, META_N_SPLIT));
  if (a.akl_width == 1.f && !akl_crowded(a.akl, a.T_pad, work.tt)) return;
  BinsEpi epi(a, work.tt, smem);
  StripEpi<BinsEpi> drive(epi);
  strip_loop<1, true, StripCfg, A_KMAJOR_DZ>(work, drive, smem);
  if (work.cnt > 0) epi.write(a, work.tt, work.split);
}

#define KD_LAUNCH(kern) launch_big<kern>(grid, StripCfg::NT, StripCfg::SMEM_BYTES, st, &a)
#define KD_LAUNCH_STATE(kern) launch_big<kern>(grid, StripCfg::NT, StripCfg::STATE_SMEM_BYTES, st, &a)

hipError_t launch_strip_hv_stats(const Problem& p, const LogitArgs& a, int grid, hipStream_t st) {
  switch (p.kind) {
    case 0: return KD_LAUNCH_STATE(stats_strip_hv_kern<0>);
    case 1: return KD_LAUNCH_STATE(stats_strip_hv_kern<1>);
    case 6: return KD_LAUNCH_STATE(stats_strip_hv_kern<6>);
    default: return KD_LAUNCH_STATE(stats_strip_hv_kern<2>);
  }
}
hipError_t launch_strip_hv_rows(const Problem& p, const LogitArgs& a, int grid, hipStream_t st) {
  switch (p.kind) {
    case 2: return KD_LAUNCH(rows_strip_hv_kern<2>);
    case 3: return KD_LAUNCH(rows_strip_hv_kern<3>);
    case 4: return KD_LAUNCH(rows_strip_hv_kern<4>);
    case 6: return KD_LAUNCH_STATE(rows_strip_hv_kern<6>);
    default: return KD_LAUNCH(rows_strip_hv_kern<5>);
  }
}
hipError_t launch_strip_hv_grad(const Problem& p, const LogitArgs& a, int grid, hipStream_t st) {
  switch (p.kind) {
    case 0: return KD_LAUNCH_STATE(grad_strip_hv_kern<0>);
    case 1: return KD_LAUNCH_STATE(grad_strip_hv_kern<1>);
    case 2: return KD_LAUNCH_STATE(grad_strip_hv_kern<2>);
    case 3: return KD_LAUNCH_STATE(grad_strip_hv_kern<3>);
    case 4: return KD_LAUNCH_STATE(grad_strip_hv_kern<4>);
    case 6: return KD_LAUNCH_STATE(grad_strip_hv_kern<6>);
    default: return KD_LAUNCH_STATE(grad_strip_hv_kern<5>);
  }
}
hipError_t launch_strip_hv_search(const LogitArgs& a, int grid, hipStream_t st) {
  return launch_big<search_strip_hv_kern>(grid, StripCfg::NT, BinsEpi::SMEM_BYTES, st, &a);
}

}  // namespace kd
