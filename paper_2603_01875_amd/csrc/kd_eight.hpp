// The logit kernels on the eight-wave tile loop (kd_mfma.hpp).  FEW: of one token tile whose last wave pairs have no token (those
// kernels are in kd_few.hip, the others in kd_kernels.hip).
#pragma once
#include "kd_logits.hpp"

namespace kd {

#define KD_LOGIT_KERNEL __global__ __launch_bounds__(LCfg::NT)

template <int KIND, bool TF8, bool WHV, bool FEW = false>
KD_LOGIT_KERNEL void stats_kernel(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  SplitWork<TF8, WHV> work(a);
  StatsEpi<KIND> epi(a.c);
  TileEpi<StatsEpi<KIND>> drive(epi, a.t_scale);
  LoopClock clk(a);
  tile_loop<2, LCfg, WHV, TF8, FEW>(work, drive, a.ld_s, a.ld_t, a.H_s, a.H_t, smem, FEW ? max(meta_get(a.meta, META_N_VALID), 1) : 0);
  clk.stop(a);
  if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
}

template <int KIND, bool TF8, bool WHV, bool FEW = false>
KD_LOGIT_KERNEL void rows_kernel(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  SplitWork<TF8, WHV> work(a);
  RowsEpi<KIND, TileGeo> epi(a, work.tt);
  TileEpi<RowsEpi<KIND, TileGeo>> drive(epi, a.t_scale);
  tile_loop<2, LCfg, WHV, TF8, FEW>(work, drive, a.ld_s, a.ld_t, a.H_s, a.H_t, smem, FEW ? max(meta_get(a.meta, META_N_VALID), 1) : 0);
  if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
}

// (one accumulator: the driver gets the teacher's tile as the first one)
template <class Epi>
struct SearchTileEpi : TileEpi<Epi> {
  using TileEpi<Epi>::TileEpi;
  __device__ void end_item(const WorkItem& it, AccTile& accT, AccTile&) { TileEpi<Epi>::end_item(it, accT, accT); }
};
template <bool WHV, bool FEW = false>
KD_LOGIT_KERNEL void akl_search_kernel(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  TeacherSplitWork<WHV> work(a);
  SearchEpi<TileGeo> epi(a, work.tt);
  SearchTileEpi<SearchEpi<TileGeo>> drive(epi, 1.f);
  tile_loop<1, LCfg, WHV, false, FEW>(work, drive, a.ld_t, a.ld_t, a.H_t, a.H_t, smem, FEW ? max(meta_get(a.meta, META_N_VALID), 1) : 0);
  if (work.cnt > 0) epi.write(a, smem, work.tt, work.split);
}

template <int KIND, bool TF8, bool WHV, bool FEW = false>
KD_LOGIT_KERNEL void grad_kernel(const LogitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  ChunkWork<TF8, WHV> work(a);
  GradEpi<KIND, TileGeo> epi(a, smem);
  TileEpi<GradEpi<KIND, TileGeo>> drive(epi, a.t_scale);
  tile_loop<2, LCfg, WHV, TF8, FEW>(work, drive, a.ld_s, a.ld_t, a.H_s, a.H_t, smem, FEW ? max(meta_get(a.meta, META_N_VALID), 1) : 0);
}

}  // namespace kd
