// Host side of the two projections (proj_kernels.hpp): which kernel a call runs and how its sums are cut.  Needs no GPU
// headers: the number of compute units is an argument.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "../../include/gla_decode.h"

namespace gla {

struct ProjPlan {
  int mt;          // 32-row blocks of query rows per workgroup (1, 2 or 4)
  int nt;          // 32-row blocks of output features per wave (1 or 2)
  int ksplit;      // ranges the input features of a group are cut into
  int k_per_split;
  bool direct;     // no partials: the kernel writes the result itself
  bool stream;     // fetch the weights with the streaming hint
  bool placed;     // workgroups are placed on the XCDs, each with a contiguous run of (range, block of features, row tile)
  bool rotated;    // blocks of features start at different steps of their range
  size_t part_bytes;
};

// Weights that the last-level cache cannot hold (256 MB).
constexpr int64_t kProjCacheBytes = 256ll << 20;

// The cut of the kernel with 64 output features per wave (256 per workgroup) and 32 * mt rows: as many ranges per group as
// give one workgroup per compute unit in a single round (its ring of three stages of 40 or 48 KB fills the LDS), of at least
// 512 features, of ceil(steps / ranges) steps of 64 each, the last one shorter.  Against 32 features per wave that halves the
// re-reads of the query rows (every workgroup fetches its range of them: rows x k x 2 bytes per 128 or 256 output features)
// and needs fewer partial results (output projection of the benchmark shape: 240 workgroups, 93 -> 74 us).  False where such
// a grid covers less than three quarters of the compute units.
inline bool proj_cut_64(const gla_proj_params* p, int mt, int cus, int* ranges, int* per_range) {
  const int64_t base = (int64_t)((p->n + 255) / 256) * ((p->rows + 32 * mt - 1) / (32 * mt)) * p->groups;
  const int64_t want = std::min<int64_t>(std::max(1, p->k / 512), cus / std::max<int64_t>(1, base));
  if (want < 1 || base * want * 4 < (int64_t)cus * 3) return false;
  const int steps = p->k / 64, per = (int)((steps + want - 1) / want);
  *ranges = (steps + per - 1) / per;  // (no empty range)
  *per_range = per * 64;
  return true;
}

// small: the plan of a call whose workspace is too small for the one it would get otherwise.  1: no more than 64 rows per
// workgroup, which takes fewer partials; 2: beyond 64 rows, 32 output features per wave besides.
inline int proj_plan(const gla_proj_params* p, int sum_groups, int cus, int small, ProjPlan* plan) {
  if (!p || p->rows < 0 || p->groups < 1 || p->n < 1 || p->k < 1) return GLA_ERR_INVALID_ARG;
  if (p->c_dtype != GLA_OUT_BF16 && p->c_dtype != GLA_OUT_FP32) return GLA_ERR_INVALID_ARG;
  if ((int64_t)p->rows * p->groups * p->n > (int64_t)0x7fffffff) return GLA_ERR_INVALID_ARG;
  // what the kernel assumes: whole steps of 64 input features, whole waves of 32 output features, 16-byte loads
  if (p->k % 64 || p->n % 32) return GLA_ERR_UNSUPPORTED_SHAPE;
  if (p->a_row_stride % 8 || p->a_group_stride % 8 || p->c_row_stride % 4 || p->c_group_stride % 4)
    return GLA_ERR_UNSUPPORTED_SHAPE;
  const int64_t weights = (int64_t)p->groups * p->n * p->k * 2;
  const int tiles64 = (p->rows + 63) / 64, tiles128 = (p->rows + 127) / 128;
  const int mt = p->rows <= 32 ? 1 : 2;
  int ks = 1, per = p->k;
  plan->mt = mt;
  plan->nt = 1;
  if (p->rows <= 64 || small) {
    if ((p->rows <= 64 || small < 2) && proj_cut_64(p, mt, cus, &ks, &per)) plan->nt = 2;
  } else {
    // More than 64 rows.  128 rows per workgroup halve the passes over the weights (two latent heads x 5120 x 16384, 100
    // rows: 83 us with 64 rows per workgroup, 73 with 128), but double the partials per range and compute what pads the last 128 rows.
    // The lines were drawn with workgroups in plain order.  us in the present one, the other way / the way taken (some have
    // moved: where the first figure is the smaller one the line now lies on the wrong side of the shape).  128 rows are taken
    //   up to 128 rows, but weights of less than 128 MB only where the number of blocks of 256 features is no multiple of
    //   eight.  (Else the workgroups of the two 64-row tiles of a block met on one XCD and shared the weights through its L2; placed,
    //   they do with any number.)  2 x 2048 x 8192, 100 rows 27.4 / 23.7, 6144 x 8192 32.5 / 31.1; but 2 x 5120 x 4096 28.2 / 30.3, 3 x
    //   1024 x 10752 25.9 / 30.0.  2 x 8192 x 8192, 100 rows 64.4 / 59.3;
    //   for sums of one range (and more than 128 output features, else half a workgroup has nothing to do) up to 256 rows,
    //   where 64 rows would pad about as much (128 heads x 256 x 128: 200 rows 11.7 / 11.7, 160 rows 10.9 / 9.5; 128 x 512 x 128, 100
    //   rows 12.5 / 12.3; 32 x 512 x 128, 300 rows 10.3 / 9.4);
    //   for longer sums beyond 128 rows in ranges of at least 1280 features where 64 rows would pad about as much, or where the
    //   weights are as large as the last-level cache (2 x 5120 x 8192: 256 rows 85 / 66, but 300 rows 85 / 98; 1 x 5120 x 4096,
    //   ranges of 704: 256 rows 29.5 / 27.1, 129 rows 26.2 / 21.3; 2 x 8192 x 8192: 129 rows 97.7 / 86.9).
    const bool single = p->k < 1024, as_full = 20 * tiles64 >= 36 * tiles128;  // (nine tenths of the 128-row tiles' halves have rows)
    int ranges, features;
    const bool cut4 = proj_cut_64(p, 4, cus, &ranges, &features);
    bool rows4;
    if (single) rows4 = as_full && p->rows <= 256 && p->n > 128;
    else if (p->rows <= 128) rows4 = (p->n + 255) / 256 % 8 != 0 || weights >= kProjCacheBytes / 2;
    else rows4 = features >= 1280 && (as_full || weights >= kProjCacheBytes);
    // Else 64 rows with 64 features per wave, but not in short ranges (1 x 2048 x 8192, 65 rows, ranges of 512: 16.0 / 14.2; 1 x
    // 5120 x 4096, of 704: 18.4 / 20.8; 129 rows, of 1024: 21.4 / 21.3; 2 x 2048 x 8192, of 1664: 31.0 / 28.9) nor, beyond 128
    // rows, where 128 rows per workgroup do not fill the chip (4 x 5120 x 8192, 167 rows 107 / 112); for sums of one range only with
    // one block of 256 features per group, up to 128 rows (100 rows of 128 heads x 256 x 128 7.15 / 7.5, of 64 x 512 x 128 7.5 / 7.15,
    // 122 rows of 128 x 128 x 192 6.7 / 5.6; 64 heads x 256 x 128, 200 rows 7.5 / 7.05).
    if (cut4 && rows4) {
      plan->mt = 4;
      plan->nt = 2;
    } else {
      const bool rows2 = single ? p->rows <= 128 && p->n > 128 && p->n <= 256 : cut4 || p->rows <= 128;
      if (rows2 && proj_cut_64(p, 2, cus, &ranges, &features) && (single || features >= (p->rows <= 128 ? 768 : 1152))) plan->nt = 2;
    }
    if (plan->nt == 2) {
      ks = ranges;
      per = features;
    }
  }
  plan->k_per_split = per;
  const int64_t row_tiles = (p->rows + 32 * plan->mt - 1) / (32 * plan->mt);
  if (plan->nt == 1) {
    const int64_t tiles = (int64_t)((p->n + 127) / 128) * row_tiles;
    // Ranges per group: the grid runs in rounds of as many workgroups as there are compute units.  Among
    // the cuts into ranges of at least 512 features pick the one with the least estimated time: rounds x
    // (steps per range + a fixed cost per workgroup of about four steps: start-up latency, partial store).
    double best = 1e30;
    for (int c = 1; c <= 64 && p->k / c >= 512 && (p->k / c) % 64 == 0; c *= 2) {
      const int64_t wgs = tiles * p->groups * c;
      const double t = (double)((wgs + cus - 1) / cus) * (p->k / c / 64 + 4);
      if (t < best * 0.999) { best = t; ks = c; }
    }
    plan->k_per_split = p->k / ks;
  }
  plan->ksplit = ks;
  // Weights read once, by one row tile, that would take more than half of the last-level cache and are not there any more
  // at the next step, after everything else a decode step reads: their lines then do not displace query rows and partials
  // (64 rows, without / with the hint: 335 MB 66.7 / 60.7 us, 671 MB 125 / 108, 168 to 268 MB +-1.5 %; 16 rows: 168 MB 34.2 / 32.3, 199 MB
  // 39.5 / 37.3, 268 MB 50.1 / 46.9).  A program that does nothing else between two calls with the same weights loses by it where
  // the cache can hold them (64 rows: 199 MB 39.6 / 44.5, 168 MB 37.1 / 39.0, 268 MB 50.5 / 52.5; 16 rows gain also then).
  // Smaller ones may still be there (84 MB 24.8 / 27.7).  With two row tiles it hardly matters (335 MB, 129 rows 108.9 / 108.6).
  plan->stream = plan->nt == 2 && row_tiles == 1 && weights > kProjCacheBytes / 2;
  // Placement and start offsets (what they are for: proj_kernel).  us in plain order / this way, weights not in the caches:
  //   64 features per wave, ranges of 512 features and more: placed (64 rows of 2 x 5120 x 16384 70.1 / 60.7, both with offsets,
  //   of 16 x 2048 x 1024 24.7 / 23.8; 128 rows of 8 x 4096 x 2048 46.2 / 41.6), up to 16 rows only with many groups (8 x 4096 x
  //   2048, 1 row 30.4 / 28.2; 16 x 2048 x 1024 17.9 / 17.6; 1 x 16384 x 1536, 16 rows 14.8 / 15.1, 4 x 5120 x 8192 56.5 / 58.4).
  //   Offsets where rows of weights lie more than 2 KB apart (32 rows of 2 x 8192 x 8192 77 / 48, of 128 x 512 x 2048 70 / 48,
  //   1 row of 1 x 5120 x 16384 33.4 / 30.0).  Closer rows of a block cover the channels by themselves (16 x 4096 x 512, 1 row
  //   15.3 / 15.9; 8 x 4096 x 1024, 65 rows 21.9 / 23.2), but at 2 KB large weights still gain (64 x 1024 x 1024, 134 MB, 1 row
  //   27.5 / 26.5).  Groups start alike: many of them with long rows are better off as they are (17 rows of 32 x 1024 x 8192 122 / 148,
  //   of 32 x 2048 x 8192 169 / 231; not of 64 x 1024 x 4096 134 / 94, nor of 16 x 2048 x 8192 122 / 93).
  //   32 features per wave, and short ranges: two workgroups share a compute unit at different steps, and long lists run in
  //   rounds.  Weights of more than the last-level cache with rows more than 2 KB apart: as above (64 rows of 1 x 128256 x 8192 474 / 364,
  //   of 32 x 8192 x 2048 250 / 212; the other way 16 x 7168 x 7168 331 / 343).  (One block of 32 rows and features has neither: offsets
  //   alone would gain where rows lie a multiple of 4 KB apart, 1 x 128256 x 8192, 1 row 464 / 403, and cost short sums 2 %.)
  //   Else beyond 64 rows, where the workgroups in between two row tiles of a block read more weights than the L2s hold (32 MB:
  //   129 rows of 1 x 128256 x 1024 132 / 94; 300 rows of 8 x 5120 x 2048, 21 MB 92.7 / 97.9), or where few blocks put a block's
  //   row tiles on different XCDs (128 heads x 256 x 128, 65 rows 8.5 / 7.0; 32 x 256 x 128, 129 rows 4.85 / 4.6; 128 x 256 x 1024,
  //   256 rows 58 / 36), but not in short sums of few groups or on part of the chip (16 x 512 x 128, 129 rows 4.47 / 4.60, 200
  //   rows 4.78 / 4.93).  With eight blocks and more they mostly share one anyway, and the writes suffer (32 x 7168 x 64, 65 rows 24.9 /
  //   28.9; 4 x 1024 x 2048, 256 rows 14.3 / 16.3; 16 x 5120 x 128, 200 rows 23.4 / 24.4; the other way 1 x 4096 x 2048, 256 rows 15.8 /
  //   14.2, 32 x 1536 x 192 21.0 / 18.6).
  //   33 to 64 rows: one round of workgroups with long ranges (1 x 1024 x 16384, 64 rows 15.7 / 14.2; 2 x 16384 x 512 11.9 / 11.6),
  //   not short sums (128 x 256 x 128, 64 rows 5.37 / 5.55), few weights (2 x 4096 x 1024 9.2 / 9.5) nor several rounds (8 x
  //   5120 x 2048 39.6 / 42.9).
  const int64_t blocks = (p->n + 128 * plan->nt - 1) / (128 * plan->nt), slices = (int64_t)p->groups * ks;
  const int64_t list = blocks * row_tiles * slices;
  const int64_t l2s = 32ll << 20;
  if (plan->nt == 2 && plan->k_per_split >= 512) {
    const bool alike = p->groups >= 32 && p->k >= 8192 && weights >= 2 * kProjCacheBytes;
    plan->placed = !alike && (p->rows > 16 || p->groups >= 8);
    plan->rotated = !alike && (p->k > 1024 || (p->k == 1024 && weights >= kProjCacheBytes / 2));
  } else {
    const bool large = p->k > 1024 && weights >= kProjCacheBytes;
    if (p->rows <= 32) plan->placed = false;
    else if (large) plan->placed = true;
    else if (p->rows <= 64) plan->placed = plan->k_per_split >= 512 && weights >= l2s && list >= cus && list <= 2 * cus;
    else
      plan->placed = (row_tiles > 1 && (int64_t)p->n * plan->k_per_split * 2 >= l2s) ||
                     (blocks < 8 && (plan->k_per_split >= 512 || (slices >= 32 && 4 * list >= 3 * cus)));
    plan->rotated = large && plan->placed;
  }
  plan->direct = ks == 1 && (!sum_groups || p->groups == 1);
  plan->part_bytes = plan->direct ? 0 : (size_t)p->groups * ks * p->rows * p->n * sizeof(float);
  return GLA_OK;
}

// Never less than for fewer rows (a plan depends on the number of blocks of 32 rows only, and its partials grow with the
// rows), so that a program may size its workspace once, for its largest batch.
inline size_t proj_workspace(const gla_proj_params* p, int sum_groups, int cus) {
  ProjPlan plan;
  if (proj_plan(p, sum_groups, cus, 0, &plan) != GLA_OK) return 0;
  size_t need = std::max<size_t>(plan.part_bytes, 256);
  if (!sum_groups && p->k < 1024) return need;  // (too short to be cut)
  gla_proj_params fewer = *p;
  for (fewer.rows = 32; fewer.rows < p->rows; fewer.rows += 32)
    if (proj_plan(&fewer, sum_groups, cus, 0, &plan) == GLA_OK) need = std::max(need, plan.part_bytes);
  return need;
}

}  // namespace gla
