// Launch of the eight-wave decode-attention kernel.
#include "tuned_host.hpp"
#include "wide_main_kernel.hpp"

namespace gla {

template <int DV, bool PP>
static int launch_wide(const TunedPlan& plan, const DevParams& d, hipStream_t st) {
  using W = WideTraits<DV, PP>;
  if (plan.rows != W::kRows || plan.slot_floats != W::kSlotFloats) return GLA_ERR_LAUNCH;
  const dim3 grid(plan.wide_chunks * plan.mb), block(512);
  if (d.lg_page >= 3) {
    if (plan.stream) hipLaunchKernelGGL((wide_main_kernel<DV, PP, 0, true>), grid, block, 0, st, d);
    else hipLaunchKernelGGL((wide_main_kernel<DV, PP, 0, false>), grid, block, 0, st, d);
  } else {
    if (plan.stream) hipLaunchKernelGGL((wide_main_kernel<DV, PP, 1, true>), grid, block, 0, st, d);
    else hipLaunchKernelGGL((wide_main_kernel<DV, PP, 1, false>), grid, block, 0, st, d);
  }
  return hipGetLastError() == hipSuccess ? GLA_OK : GLA_ERR_LAUNCH;
}

int wide_launch(const TunedPlan& plan, const DevParams& four, hipStream_t st) {
  DevParams d = four;  // (tiles of twice as many tokens)
  d.num_chunks = plan.wide_chunks;
  d.chunk_tiles = (plan.chunk_tiles + 1) / 2;
  d.setup_tiles = setup_tiles(kSetupTilesWide, plan.list_bound);
  d.fd_chunks = make_fastdiv((uint32_t)plan.wide_chunks);
  d.xcd_map = plan.wide_chunks % 8 == 0 ? 1 : 0;
  return plan.dv == 256 ? launch_wide<256, true>(plan, d, st) : launch_wide<512, false>(plan, d, st);
}

}  // namespace gla
