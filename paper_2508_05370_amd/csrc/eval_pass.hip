// eval_pass.hip -- one evaluation pass of one variant: table mode HETSIM_MODE
// (0..2), plan layout HETSIM_HET (0 shared, 1 per class), pass HETSIM_PASS
// (0 the first pass's k_eval groups, 1 k_all, shared layout only).  The build
// compiles this file once per variant; kernels.hip dispatches at run time.
#include "launch.h"

#if !defined(HETSIM_MODE) || !defined(HETSIM_HET) || !defined(HETSIM_PASS)
#error "eval_pass.hip is built once per variant: define HETSIM_MODE, HETSIM_HET and HETSIM_PASS"
#endif
#if HETSIM_PASS != 0 && HETSIM_HET
#error "k_all is built for the shared layout only"
#endif

namespace hetsim {

// A grid of at most `cap` blocks that has a wavefront for each of n tiles.
static uint32_t tile_grid(uint32_t n, uint32_t cap) {
  const uint32_t need = (n + kEvalThreads / 64 - 1) / (kEvalThreads / 64);
  return need < 1 ? 1 : need < cap ? need : cap;
}

#if HETSIM_PASS == 0
template <int kMode, bool kHet>
hipError_t launch_group_v(const Tab& t, const EvalBufs& e, uint32_t max_tiles, int g, hipStream_t s) {
  const uint32_t grid = tile_grid(max_tiles, 4 * t.grid_eval[g]);
  const size_t lds = (kMode < 2 ? t.lds_bytes : 0) + block_lds_bytes(kHet ? 0 : plan_cols(g, false), t.K);
  if (g == 0) k_eval<0, kMode, kHet><<<grid, kEvalThreads, lds, s>>>(e.dtab, e);
  else if (g == 1) k_eval<1, kMode, kHet><<<grid, kEvalThreads, lds, s>>>(e.dtab, e);
  else if (g == 2) k_eval<2, kMode, kHet><<<grid, kEvalThreads, lds, s>>>(e.dtab, e);
  else k_eval<3, kMode, kHet><<<grid, kEvalThreads, lds, s>>>(e.dtab, e);
  return hipGetLastError();
}
template hipError_t launch_group_v<HETSIM_MODE, (bool)HETSIM_HET>(const Tab&, const EvalBufs&, uint32_t, int,
                                                                  hipStream_t);

#if !HETSIM_HET
// Grid caps come from the shared-layout kernels; the per-class-layout ones
// take the same caps (their fixed-stride loops cover any grid).
template <int kMode>
hipError_t occupancy_v(int nb[4], size_t lds, uint32_t types) {
  const void* k[4] = {(const void*)k_eval<0, kMode, false>, (const void*)k_eval<1, kMode, false>,
                      (const void*)k_eval<2, kMode, false>, (const void*)k_eval<3, kMode, false>};
  for (int i = 0; i < 4; ++i) {
    const size_t b = lds + block_lds_bytes(plan_cols(i, false), types);
    hipError_t r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb[i], k[i], kEvalThreads, b);
    if (r != hipSuccess) return r;
  }
  return hipSuccess;
}
template hipError_t occupancy_v<HETSIM_MODE>(int[4], size_t, uint32_t);
#endif

#else
template <int kMode>
hipError_t launch_all_v(const Tab& t, const EvalBufs& e, uint32_t max_tiles, bool plain, hipStream_t s) {
  const size_t lds = (kMode < 2 ? t.lds_bytes : 0) + block_lds_bytes(plan_cols(0, true), t.K);
  k_all<kMode><<<tile_grid(max_tiles, t.grid_all), kEvalThreads, lds, s>>>(e.dtab, e, plain ? 1u : 0u);
  return hipGetLastError();
}
template hipError_t launch_all_v<HETSIM_MODE>(const Tab&, const EvalBufs&, uint32_t, bool, hipStream_t);

template <int kMode>
hipError_t occupancy_all_v(int nb[1], size_t lds, uint32_t types) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb[0], (const void*)k_all<kMode>, kEvalThreads,
                                                      lds + block_lds_bytes(plan_cols(0, true), types));
}
template hipError_t occupancy_all_v<HETSIM_MODE>(int[1], size_t, uint32_t);
#endif

}  // namespace hetsim
