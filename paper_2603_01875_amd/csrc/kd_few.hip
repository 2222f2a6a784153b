// The eight-wave loop's logit kernels for at most kFewTokens tokens, so that at least one of the four wave pairs of a tile has none:
// those waves only load.  Bound by the heads, which stream through once a pass: H = 4096 / 1024, V = 151936, 1.56 GB, 305 us at the
// rate of a large copy.  Measured with all waves multiplying and so: T = 64 a step 893 -> 800 us, JSD 1263 -> 1102, T = 128 943 -> 859, T = 100 the
// statistics alone 369 -> 321, a step with the fp8 teacher 665 -> 612; T = 100, H = 512 / 256, V = 8000 60.3 -> 53.7; T = 128, H = 256 / 128, V = 4096, fp32 63.9 -> 58.0.
#include "kd_eight.hpp"

namespace kd {

#define KD_PICK(kern, K) (p.t_fp8 ? launch_big<kern<K, true, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                          : p.w_hv_inplace ? launch_big<kern<K, false, true, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                                           : launch_big<kern<K, false, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a))
// (AKL: never with the fp8 teacher)
#define KD_PICK_AKL(kern) (p.w_hv_inplace ? launch_big<kern<6, false, true, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a) \
                                          : launch_big<kern<6, false, false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a))

hipError_t launch_few_stats(const Problem& p, const LogitArgs& a, int grid, hipStream_t st) {
  switch (p.kind) {
    case 0: return KD_PICK(stats_kernel, 0);
    case 1: return KD_PICK(stats_kernel, 1);
    case 6: return KD_PICK_AKL(stats_kernel);
    default: return KD_PICK(stats_kernel, 2);
  }
}
hipError_t launch_few_rows(const Problem& p, const LogitArgs& a, int grid, hipStream_t st) {
  switch (p.kind) {
    case 2: return KD_PICK(rows_kernel, 2);
    case 3: return KD_PICK(rows_kernel, 3);
    case 4: return KD_PICK(rows_kernel, 4);
    case 6: return KD_PICK_AKL(rows_kernel);
    default: return KD_PICK(rows_kernel, 5);
  }
}
hipError_t launch_few_grad(const Problem& p, const LogitArgs& a, int grid, hipStream_t st) {
  switch (p.kind) {
    case 0: return KD_PICK(grad_kernel, 0);
    case 1: return KD_PICK(grad_kernel, 1);
    case 2: return KD_PICK(grad_kernel, 2);
    case 3: return KD_PICK(grad_kernel, 3);
    case 4: return KD_PICK(grad_kernel, 4);
    case 6: return KD_PICK_AKL(grad_kernel);
    default: return KD_PICK(grad_kernel, 5);
  }
}
hipError_t launch_few_search(const Problem& p, const LogitArgs& a, int grid, hipStream_t st) {
  return p.w_hv_inplace ? launch_big<akl_search_kernel<true, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a)
                        : launch_big<akl_search_kernel<false, true>>(grid, LCfg::NT, LCfg::SMEM_BYTES, st, &a);
}

}  // namespace kd
