// Instantiations of the segmented kernels: solve, order d = 2.
#include "whs_seg_launch.h"

namespace whs {
hipError_t run_seg_solve_d2(const LaunchDesc& L, hipStream_t stream) {
  return L.perdiff ? run_seg<2, false, true>(L, stream) : run_seg<2, false, false>(L, stream);
}
}  // namespace whs
