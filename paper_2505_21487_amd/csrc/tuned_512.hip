// Tuned decode-attention kernels with 512 state dims.
#include "tuned_launch.hpp"

namespace gla {

int tuned_launch_512(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev) {
  return launch_tuned_shape<512, 512>(plan, d, st, ev);
}

}  // namespace gla
