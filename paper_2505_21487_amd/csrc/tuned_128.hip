// Tuned decode-attention kernels with 128 state dims (GTA: half of them in the score).
#include "tuned_launch.hpp"

namespace gla {

int tuned_launch_128(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev) {
  return launch_tuned_shape<128, 64>(plan, d, st, ev);
}

}  // namespace gla
