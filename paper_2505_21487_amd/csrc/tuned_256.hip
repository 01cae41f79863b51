// Tuned decode-attention kernels with 256 state dims.
#include "tuned_launch.hpp"

namespace gla {

int tuned_launch_256(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev) {
  return launch_tuned_shape<256, 256>(plan, d, st, ev);
}

}  // namespace gla
