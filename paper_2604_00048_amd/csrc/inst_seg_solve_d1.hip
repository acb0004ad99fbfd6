// Instantiations of the segmented kernels: solve, order d = 1.
#include "whs_seg_launch.h"

namespace whs {
hipError_t run_seg_solve_d1(const LaunchDesc& L, hipStream_t stream) {
  return L.perdiff ? run_seg<1, false, true>(L, stream) : run_seg<1, false, false>(L, stream);
}
}  // namespace whs
