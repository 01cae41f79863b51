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
  // Sets every unit has: by the mean length of a list, while the grid is no more than two workgroups per compute unit
  // (256 / 512 / 1024 workgroups: GLA-2 8 x 2048 tokens 24.1 / 23.5 / 23.3 us per call, 15 x 1024 and 1 x 65536 41.2 / 41.2 /
  // 43.3, MLA shape 53.5 / 53.6 / 55.2, GTA-4 10 sequences 20.9 / 19.1 / 18.2).  Windows of eight chunks (5 / 8 / 12: MLA shape
  // 15 x 1024 and 1 x 65536 52.5 / 53.6 / 53.4, 20 ragged sequences 33.7 / 32.8 / 33.8), at most 64; none where a unit is the
  // only one, or looked for among thousands.
  constexpr int kPanels = NG * WPG * KS * (DV / KS / 32) / 4;
  DevParams c = d;
  const int chunks = std::max(plan.num_chunks, plan.wide_chunks), seq_units = plan.units / plan.mb;
  const int list = chunks / seq_units;
  int lg = 0;
  while (lg < 4 && (2 << lg) <= list && ((int64_t)plan.units * kPanels << (lg + 1)) <= 2 * device_cu_count()) ++lg;
  c.merge_sets_lg = lg;
  c.merge_span = std::max(8, (chunks + 63) / 64);
  c.merge_windows = seq_units > 1 && seq_units <= 2048 && lg < 4 ? chunks / c.merge_span : 0;
  const int64_t blocks = (((int64_t)plan.units << lg) + (int64_t)c.merge_windows * plan.mb) * kPanels, width = 1 << 20;
  const dim3 grid((unsigned)std::min(blocks, width), (unsigned)((blocks + width - 1) / width));
  // few panels and long lists: sixteen waves per block (one sequence of 131072 tokens: 57.5 us with four)
  if (list >= 64 && lg == 4 && blocks <= device_cu_count())
    hipLaunchKernelGGL((tuned_combine_kernel<DV, NG, WPG, KS, TOK, 16>), grid, dim3(1024), 0, st, c);
  else
    hipLaunchKernelGGL((tuned_combine_kernel<DV, NG, WPG, KS, TOK, 4>), grid, dim3(256), 0, st, c);
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
