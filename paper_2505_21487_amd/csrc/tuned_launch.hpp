// Launches of the tuned decode-attention kernels; included by one unit (of library.hip) per state shape.
#pragma once

#include "tuned_combine_kernel.hpp"
#include "tuned_host.hpp"

namespace gla {

template <int DV, int DN, int NG, int WPG, int KS, int TOK, bool STREAM>
inline int launch_tuned_main(const DevParams& d, dim3 mgrid, dim3 mblock, hipStream_t st) {
  constexpr int STAGES = tuned_stages(DV, NG, WPG, KS), STAGES_LANE = tuned_stages(DV, NG, WPG, KS, true);
  constexpr bool kLaneFits = tuned_windows_fit(DV, NG, WPG, KS);
  if (d.lg_page == 6) {
    hipLaunchKernelGGL((tuned_main_kernel<DV, DN, 64, NG, WPG, KS, TOK, STAGES, 0, STREAM>), mgrid, mblock, 0, st, d);
  } else if (d.lg_page >= 4) {
    hipLaunchKernelGGL((tuned_main_kernel<DV, DN, 64, NG, WPG, KS, TOK, STAGES, 1, STREAM>), mgrid, mblock, 0, st, d);
  } else {
    if constexpr (kLaneFits)
      hipLaunchKernelGGL((tuned_main_kernel<DV, DN, 64, NG, WPG, KS, TOK, STAGES_LANE, 2, STREAM>), mgrid, mblock, 0, st, d);
    else  // (no LDS left for the page-id windows: kept in registers)
      hipLaunchKernelGGL((tuned_main_kernel<DV, DN, 64, NG, WPG, KS, TOK, STAGES, 3, STREAM>), mgrid, mblock, 0, st, d);
  }
  return GLA_OK;
}

template <int DV, int NG, int WPG, int KS, int TOK>
inline int launch_tuned_combine(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev) {
  // waves per merge task from the expected number of chunks per unit
  const int64_t span_est = (plan.num_chunks + std::max(1, plan.units / plan.mb) - 1) / std::max(1, plan.units / plan.mb) + 1;
  const dim3 cgrid(plan.units, NG * WPG * (DV / 32));
  if (span_est <= 2)
    hipLaunchKernelGGL((tuned_combine_kernel<DV, NG, WPG, KS, TOK, 1, 1, 2>), cgrid, dim3(64), 0, st, d);
  else if (span_est <= 6)  // (one wave with four chunks in flight: a fourth of the waves to launch, no merge through LDS)
    hipLaunchKernelGGL((tuned_combine_kernel<DV, NG, WPG, KS, TOK, 1, 1, 4>), cgrid, dim3(64), 0, st, d);
  else if (span_est <= 12)
    hipLaunchKernelGGL((tuned_combine_kernel<DV, NG, WPG, KS, TOK, 4, 1, 2>), cgrid, dim3(256), 0, st, d);
  else if (span_est <= 64)  // (a wave folds eight chunks per round trip: four waves do for fairly long lists)
    hipLaunchKernelGGL((tuned_combine_kernel<DV, NG, WPG, KS, TOK, 4, 1, 8>), cgrid, dim3(256), 0, st, d);
  else if ((int64_t)cgrid.x * cgrid.y * 4 > 4 * device_cu_count())
    hipLaunchKernelGGL((tuned_combine_kernel<DV, NG, WPG, KS, TOK, 16, 1, 4>), cgrid, dim3(1024), 0, st, d);
  else  // few tasks: each cut into quarters (see the kernel)
    hipLaunchKernelGGL((tuned_combine_kernel<DV, NG, WPG, KS, TOK, 16, 4, 4>), dim3(cgrid.x, cgrid.y * 4), dim3(1024), 0, st, d);
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  if (ev) (void)hipEventRecord(ev[2], st);
  return GLA_OK;
}

template <int DV, int DN, int NG, int WPG, int KS, int TOK>
inline int launch_tuned_variant(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev) {
  if (ev) (void)hipEventRecord(ev[0], st);
  const dim3 mgrid(plan.num_chunks * plan.mb), mblock(64 * NG * WPG * KS);
  // (plan.stream: the cache of this batch can be larger than the last-level cache: fetch it with the streaming hint)
  const int lrc = plan.stream ? launch_tuned_main<DV, DN, NG, WPG, KS, TOK, true>(d, mgrid, mblock, st)
                              : launch_tuned_main<DV, DN, NG, WPG, KS, TOK, false>(d, mgrid, mblock, st);
  if (lrc != GLA_OK) return lrc;
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  if constexpr (eight_wave_shape(DV, NG, WPG, KS)) {
    if (plan.wide_tiles > 0) {  // (one of the two kernels finds that the batch is the other's, and leaves)
      const int wrc = wide_launch(plan, d, st);
      if (wrc != GLA_OK) return wrc;
    }
  }
  if (ev) (void)hipEventRecord(ev[1], st);
  return launch_tuned_combine<DV, NG, WPG, KS, TOK>(plan, d, st, ev);
}

template <int DV, int DN>
inline int launch_tuned_shape(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev) {
  if constexpr (DV > 256) {
    switch (plan.ng * 100 + plan.wpg * 10 + plan.ks) {
      case 112: return launch_tuned_variant<DV, DN, 1, 1, 2, kTok>(plan, d, st, ev);
      case 122: return launch_tuned_variant<DV, DN, 1, 2, 2, kTok>(plan, d, st, ev);
      default: return GLA_ERR_UNSUPPORTED_SHAPE;
    }
  } else {
    switch (plan.ng * 100 + plan.wpg * 10 + plan.ks) {
      case 111: return launch_tuned_variant<DV, DN, 1, 1, 1, kTok>(plan, d, st, ev);
      case 121: return launch_tuned_variant<DV, DN, 1, 2, 1, kTok>(plan, d, st, ev);
      case 141: return launch_tuned_variant<DV, DN, 1, 4, 1, kTok>(plan, d, st, ev);
      case 211: return launch_tuned_variant<DV, DN, 2, 1, 1, kTok>(plan, d, st, ev);
      case 221: return launch_tuned_variant<DV, DN, 2, 2, 1, kTok>(plan, d, st, ev);
      case 411:
        if constexpr (DV <= 128) return launch_tuned_variant<DV, DN, 4, 1, 1, kTok>(plan, d, st, ev);
        else return GLA_ERR_UNSUPPORTED_SHAPE;
      default: return GLA_ERR_UNSUPPORTED_SHAPE;
    }
  }
}

}  // namespace gla
