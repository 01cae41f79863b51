// Launches of the eight-wave decode-attention kernel (its own translation unit: built beside the others).
#include "tuned_launch.hpp"
#include "wide_main_kernel.hpp"

namespace gla {

template <int DV, bool PP>
static int launch_wide(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev) {
  using W = WideTraits<DV, PP>;
  if (plan.wpg != W::NSL || plan.ks != W::E || plan.tok != W::TT || plan.slot_floats != W::kSlotFloats) return GLA_ERR_LAUNCH;
  if (ev) (void)hipEventRecord(ev[0], st);
  const dim3 grid(plan.num_chunks * plan.mb), block(512);
  if (d.lg_page >= 3) {
    if (plan.stream) hipLaunchKernelGGL((wide_main_kernel<DV, PP, 0, true>), grid, block, 0, st, d);
    else hipLaunchKernelGGL((wide_main_kernel<DV, PP, 0, false>), grid, block, 0, st, d);
  } else {
    if (plan.stream) hipLaunchKernelGGL((wide_main_kernel<DV, PP, 1, true>), grid, block, 0, st, d);
    else hipLaunchKernelGGL((wide_main_kernel<DV, PP, 1, false>), grid, block, 0, st, d);
  }
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  if (ev) (void)hipEventRecord(ev[1], st);
  return launch_tuned_combine<DV, 1, W::NSL, W::E / 2, kTok>(plan, d, st, ev);  // (the four-wave kernel's: the same partials)
}

int wide_launch(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev) {
  return plan.dv == 256 ? launch_wide<256, true>(plan, d, st, ev) : launch_wide<512, false>(plan, d, st, ev);
}

}  // namespace gla
