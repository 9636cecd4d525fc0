// launch.h -- host-side launchers of the evaluation kernels.  The first pass of
// each (table mode, plan layout) pair and k_all of each table mode are compiled
// in translation units of their own (eval_pass.hip built once per variant), so
// that the library builds in parallel; kernels.hip dispatches to them.
#pragma once
#include "device.h"

namespace hetsim {

// First pass of stage-count group g (0..3: 16-13, 12-9, 8-5, 4-1 stages) over
// at most max_tiles tiles.
template <int kMode, bool kHet>
hipError_t launch_group_v(const Tab& t, const EvalBufs& e, uint32_t max_tiles, int g, hipStream_t s);
// The plans of every other kind, and with `plain` all of them (shared layout).
template <int kMode>
hipError_t launch_all_v(const Tab& t, const EvalBufs& e, uint32_t max_tiles, bool plain, hipStream_t s);
// Blocks per CU of the shared-layout first-pass kernels (nb[0..3]) or of k_all
// (nb[0]) with `lds` bytes of table image and `types` device types.
template <int kMode>
hipError_t occupancy_v(int nb[4], size_t lds, uint32_t types);
template <int kMode>
hipError_t occupancy_all_v(int nb[1], size_t lds, uint32_t types);

#define HETSIM_EXTERN_MODE(M)                                                                                   \
  extern template hipError_t launch_group_v<M, false>(const Tab&, const EvalBufs&, uint32_t, int, hipStream_t); \
  extern template hipError_t launch_group_v<M, true>(const Tab&, const EvalBufs&, uint32_t, int, hipStream_t);  \
  extern template hipError_t launch_all_v<M>(const Tab&, const EvalBufs&, uint32_t, bool, hipStream_t);         \
  extern template hipError_t occupancy_v<M>(int[4], size_t, uint32_t);                                          \
  extern template hipError_t occupancy_all_v<M>(int[1], size_t, uint32_t);
HETSIM_EXTERN_MODE(0)
HETSIM_EXTERN_MODE(1)
HETSIM_EXTERN_MODE(2)
#undef HETSIM_EXTERN_MODE

}  // namespace hetsim
