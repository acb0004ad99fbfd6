// Instantiations of the segmented kernels: backward, order d = 1.
#include "whs_seg_launch.h"

namespace whs {
hipError_t run_seg_backward_d1(const LaunchDesc& L, hipStream_t stream) {
  return L.perdiff ? run_seg<1, true, true>(L, stream) : run_seg<1, true, false>(L, stream);
}
}  // namespace whs
