// Instantiations of the segmented kernels: backward, order d = 2.
#include "whs_seg_launch.h"

namespace whs {
hipError_t run_seg_backward_d2(const LaunchDesc& L, hipStream_t stream) {
  return L.perdiff ? run_seg<2, true, true>(L, stream) : run_seg<2, true, false>(L, stream);
}
}  // namespace whs
