// Host side of the tuned decode-attention path: shape check and plan, workspace
// size, and the choice of the launch function (tuned_launch.hpp).
#pragma once

#include <algorithm>

#include "../../include/gla_decode.h"
#include "tuned_main_kernel.hpp"

namespace gla {

// ---- host side ---------------------------------------------------------------

struct TunedPlan {
  int dv, dn;      // state dims (value / score)
  int ng, wpg, ks; // groups per workgroup, row slabs per group, waves per row slab
  int tok, stages; // tile tokens and pipeline depth of the chosen instantiation
  int rows;        // 32 * ng * wpg
  int mb;          // row blocks per (sequence, group)
  int units;       // batch * (h_c / ng) * mb
  int num_chunks;  // chunks of the tile list; the main-kernel grid is num_chunks * mb
  int chunk_tiles; // fixed tiles per chunk, 0: derived on the device
  size_t slot_floats;
  int wide_tiles;  // > 0: the eight-wave kernel is launched too and runs, instead, on lists of that many tiles or more
  int wide_chunks; // its chunks, of twice the tokens per tile
  bool stream;     // fetch the cache with the streaming hint
  int64_t list_bound; // tiles of the list at most
};

inline int device_cu_count() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cus = n;
    else
      cus = 256;  // MI355X
  }
  return cus;
}

inline bool aligned16(const void* ptr) { return ((uintptr_t)ptr & 15u) == 0; }

constexpr int kMinChunkTiles = 4;

// What a chunk's step into another unit costs, in tiles (cut_list): on the four-wave kernel 8 to 11 us, a tile being 1.3 to
// 1.45.  us per call with 0 / 3 / 6 / 9 / 12: absorbed query, decode of 24 ragged sequences and output projection 132.2 /
// 121.5 / 114.9 / 113.2 / 112.6; GLA-2 16 ragged sequences 39.2 / 33.3 / 30.7 / 30.4 / 30.3, 100 60.2 / 50.0 / 47.0 / 44.8 /
// 45.8, two query positions 37 sequences 116.0 / 107.9 / 99.8 / 97.0 / 97.2; MLA shape 15 x 1024 and 1 x 65536 73.5 / 71.4 /
// 67.4 / 67.3 / 66.7, 100 x 50 to 600 65.5 / 52.1 / 50.9 / 48.7 / 47.0; GTA-4 d_h 128 (a smaller result to store) 128 long
// sequences 417.5 / 414.3 / 414.2 / 415.7 / 415.6, 10 of 500 to 6000 27.1 / 23.1 / 22.9 / 22.7 / 22.5.
// Eight-wave kernel, tiles of 64 tokens, MLA shape 128 ragged sequences, 0 / 2 / 4 / 7 / 10: 374.7 / 368.2 / 360.2 / 356.9 / 358.0.
// Second MFMA kernel 0 / 2 / 4 / 8 / 12: GTA-4 d_h 64 48 sequences 36.3 / 34.4 / 34.4 / 34.7 / 35.4, d_h 96 30 sequences
// 25.7 / 23.4 / 22.3 / 22.6 / 22.6, GQA-4 12 sequences 22.7 / 20.6 / 20.7 / 20.4 / 20.6.
constexpr int kSetupTiles = 8, kSetupTiles128 = 6, kSetupTilesWide = 6, kSetupTilesFlex = 4;
// (none where positions could leave 32 bits)
inline int setup_tiles(int n, int64_t list_bound) { return list_bound <= 0x3fffffff / (n + 1) ? n : 0; }

// Batches of up to this many sequences may be cut into chunks of fewer tiles while the grid is small (tuned_plan,
// flex_plan).  Larger ones have their parallelism already, and a cut that falls badly costs them more than the rest
// gains.  us per call without and with the short chunks, equal lengths: GLA-2 8 x 100 tokens 21.9 -> 17.0, 8 x 600 28.8 ->
// 28.3, 24 x 256 23.0 -> 31.0; MLA shape 8 x 100 22.4 -> 19.9, 8 x 600 33.2 -> 33.3, 12 x 256 23.2 -> 31.1; GTA-4 d_h 128 8 x 256
// 15.5 -> 14.3, 24 x 256 16.9 -> 20.8; GTA-4 d_h 64 8 x 600 18.1 -> 13.9, 32 x 600 18.7 -> 16.4; GQA-4 8 x 256 16.1 -> 12.2.
// 70 random batches of five to eight ragged sequences of up to 2000 tokens, all shapes: 20 % less on average, the worst 3.5 % more.
constexpr int kShortChunkBatch = 8;

// From how many tiles of 32 tokens on (of the whole list) does the eight-wave kernel take a batch?  0: never, it is not
// launched.  It wins where the matrix pipe sets the pace and chunks are long; it starts a chunk and a sequence more slowly
// (twice the tokens per tile, queries loaded by twice the waves).  What counts is therefore the real number of tiles per
// chunk t and of sequences' parts per chunk, 1 + u, which only the device knows: both kernels are launched, both count,
// and the one that is not meant leaves (0.1 to 1 us per call).  Measured when the line was drawn, four waves -> eight waves, us per
// call, tiles of 64 tokens (t, u):
//   512 dims, 128 rows, pages of 64: (63, 1) 206 -> 185, (75, 2.3) 269 -> 259, (32, 1) 118 -> 108, (31, 0.1) 116 -> 115,
//     (16, 0) 65 -> 63, (16, 0.1) 73 -> 76, (64, 4) 243 -> 245, (16, 4) 104 -> 120, (32, 8) 207 -> 225, (4, 0) 35 -> 39
//   ... pages of 1: (16, 0.5) 91 -> 71, (16, 1) 79 -> 66, (8, 0.5) 53 -> 51, (4, 1) 35 -> 35, (16, 8) 190 -> 187
//   256 dims, 256 rows, pages of 64: (128, 0.5) 339 -> 316, (125, 0.3) 329 -> 310, (126, 2) 348 -> 334, (128, 0.1) 337 -> 316,
//     (63, 1) 176 -> 171, (63, 0.5) 178 -> 184, (31, 0.3) 103 -> 110, (64, 2) 185 -> 186, (117, 4.7) 369 -> 381
//   ... pages of 1: (32, 1) 108 -> 96, (32, 2) 123 -> 114, (31, 0.3) 116 -> 112, (16, 0.3) 75 -> 78, (16, 8) 178 -> 183
// With 128 rows and 256 dims (no second row block to share the tiles with) it loses, 117 -> 123.
// That was before the four-wave kernel's tiles came in runs, and with sequences of equal length.  Now, pages of 64: 512 dims (16, 0)
// 75 -> 81, (40, 0) 155 -> 156, (64, 0) 217 -> 207, (24, 0.5) 91 -> 101, (38, 0.5) 135 -> 155, (60, 0.5) 208 -> 199, (32, 1) 120 -> 118,
// (54, 2.3) 212 -> 234, (136, 2.3) 452 -> 456, (216, 2.3) 684 -> 669; ragged (62, 0.5) 213 -> 223, (99, 0.5) 320 -> 313, (49, 1) 181 ->
// 196, (121, 1) 392 -> 392; 256 dims (80, 0) 214 -> 216, (201, 0) 489 -> 479, (82, 0.1) 213 -> 227, (206, 0.1) 504 -> 489, (90, 0.5) 232
// -> 234, (225, 0.5) 543 -> 529, (160, 1) 391 -> 387; ragged (165, 1) 416 -> 433, (372, 0.1) 889 -> 871.  The line below is right for
// long chunks but about half as high as it should be: batches up to twice above it lose up to 15 % (512 dims) and 7 % (256 dims).
inline int wide_tiles_of(const gla_decode_params* p, const TunedPlan& plan) {
  if (!eight_wave_shape(p->d_v, plan.ng, plan.wpg, plan.ks) || (p->d_v == 256 && plan.mb == 1)) return 0;
  const bool small_pages = p->page_size < 16;
  // tiles wanted per chunk, and more per unit of the list
  const int64_t a = p->d_v == 512 ? (small_pages ? 8 : 32) : (small_pages ? 36 : 160);
  const int64_t b = p->d_v == 512 ? (small_pages ? 8 : 32) : (small_pages ? 12 : 40);
  const int64_t units = (int64_t)p->batch * p->num_groups;
  int64_t need;
  if (plan.chunk_tiles > 0) {  // (chunks of a given length, as many as the list has: need = a need / length + b units)
    if (plan.chunk_tiles <= a) return 0;
    need = (b * units * plan.chunk_tiles + plan.chunk_tiles - a - 1) / (plan.chunk_tiles - a);
  } else {
    need = a * plan.num_chunks + b * units;
  }
  // What the list can hold at most, by the page table's row length and, where its size is given, by the pool (pages shared
  // by several sequences may hold more: such a batch stays with the four-wave kernel).
  int64_t most = units * (((int64_t)p->max_pages_per_seq * p->page_size + kTok - 1) / kTok);
  if (p->num_pages > 0) most = std::min(most, p->num_groups * ((p->num_pages * p->page_size + kTok - 1) / kTok + p->batch));
  return need <= most ? (int)std::max<int64_t>(need, 1) : 0;
}

// lean: the plan a call gets whose workspace is too small for the one it would get otherwise (see run() in
// gla_decode.hip): no chunks of fewer than kMinChunkTiles tiles, no eight-wave kernel.
inline bool tuned_plan(const gla_decode_params* p, int is_gta, bool lean, TunedPlan* plan) {
  const int ps = p->page_size;
  if (ps < 1 || ps > 64 || (ps & (ps - 1))) return false;  // 64, 32, ..., 1 tokens
  if (p->d_rope != 64 && p->d_rope != 48 && p->d_rope != 32) return false;  // (fewer than 64: padded inside the kernel)
  const bool lane = ps < 16;  // addresses per row and lane
  if (!(p->softmax_scale > 0.f)) return false;  // row maxima are taken on the raw dot products
  if (!((!is_gta && (p->d_v == 256 || p->d_v == 512)) || (is_gta && p->d_v == 128))) return false;
  // layout the kernels assume: token rows contiguous, everything 16-byte aligned
  if (p->state_stride[2] != p->d_v || p->rope_stride[1] != p->d_rope) return false;
  if (p->state_stride[0] % 8 || p->state_stride[1] % 8 || p->rope_stride[0] % 8) return false;
  if (p->state_stride[0] < 0 || p->state_stride[1] < 0 || p->rope_stride[0] < 0 ||
      p->state_stride[0] >= (1ll << 30) || p->state_stride[1] >= (1ll << 30) || p->rope_stride[0] >= (1ll << 30))
    return false;  // page / group strides are handled as 32-bit byte counts
  if (p->num_pages >= (1ll << 31)) return false;
  for (int i = 0; i < 3; ++i)
    if (p->q_nope_stride[i] % 8 || p->q_rope_stride[i] % 8 || p->out_stride[i] % 4) return false;
  if (p->q_nope && !(aligned16(p->q_nope) && aligned16(p->q_rope) && aligned16(p->state_cache) &&
                     aligned16(p->rope_cache) && aligned16(p->out)))
    return false;
  const int rows_group = (p->num_q_heads / p->num_groups) * p->q_len;
  // waves per group from the rows of a group, then as many groups per workgroup
  // as four waves allow (they share one RoPE-key tile)
  // A latent of 512 dims needs two waves per row slab: 32 rows x 512 fp32
  // output accumulators alone would fill a wave's accumulation registers.
  const int ks = p->d_v > 256 ? 2 : 1;
  const int wpg = rows_group <= 32 ? 1 : ((rows_group <= 64 || ks == 2) ? 2 : 4);
  int ng = 4 / (wpg * ks);
  while (ng > 1 && (p->num_groups % ng || 4 * (ng * 32 * p->d_v * 2 + 32 * 128) > 160 * 1024)) ng >>= 1;
  plan->dv = p->d_v;
  plan->dn = p->d_nope;
  plan->ng = ng;
  plan->wpg = wpg;
  plan->ks = ks;
  plan->rows = 32 * ng * wpg;
  plan->mb = (rows_group + 32 * wpg - 1) / (32 * wpg);
  plan->units = p->batch * (p->num_groups / ng) * plan->mb;
  // (small pages: page-id windows in LDS where tiles and mailboxes leave room for them, else in registers)
  const bool lds_windows = lane && tuned_windows_fit(p->d_v, ng, wpg, ks);
  const int tok = kTok, stages = tuned_stages(p->d_v, ng, wpg, ks, lds_windows);
  // co-resident workgroups per CU: one wave per SIMD, 160 KiB of LDS
  const int smem = stages * (ng * tok * p->d_v * 2 + tok * 128) + (ks > 1 ? ng * wpg * ks * 4096 : 0) +
                   (lds_windows ? ng * wpg * ks * 2 * kPageWindow * 4 : 0);
  if (smem > 160 * 1024) return false;
  const int per_cu = std::max(1, std::min((160 * 1024) / smem, 4 / (ng * wpg * ks)));
  plan->tok = tok;
  plan->stages = stages;
  // the tile list holds each (sequence, group block) once; every chunk of it is
  // worked on by mb workgroups (one per row block), so the grid is num_chunks * mb
  const int64_t max_tiles = ((int64_t)p->max_pages_per_seq * p->page_size + tok - 1) / tok;
  const int64_t bound = (int64_t)(plan->units / plan->mb) * max_tiles;
  if (bound * plan->mb > 0x3fffffff) return false;
  if (p->num_splits > 0) {
    plan->chunk_tiles = (int)((max_tiles + p->num_splits - 1) / p->num_splits);
    plan->num_chunks = (int)std::max<int64_t>(1, (bound + plan->chunk_tiles - 1) / plan->chunk_tiles);
  } else {
    plan->chunk_tiles = 0;
    // one chunk per resident workgroup, but no chunk shorter than kMinChunkTiles
    // (by the upper bound on the list length): a partial costs as much memory
    // traffic as three or four tiles, and every extra chunk is one more to merge
    const int64_t resident = std::max<int64_t>(1, (int64_t)device_cu_count() * per_cu / plan->mb);
    int64_t by_length = std::max<int64_t>(1, bound / kMinChunkTiles);
    // While the grid is small the chip is idle and a tile more in the serial chain of a chunk costs more than a
    // partial: chunks of two tiles up to a quarter of the compute units, of one up to an eighth.  Measured, us per
    // call: 16 heads x 256 tokens 17.8 -> 14.6, batch 1 x 100 tokens 21.5 -> 16.4, x 512 20.4 -> 17.8, x 2048
    // 21.9 -> 20.4; further (one tile up to a quarter) loses again, 22.8 at 2048; with the grid full (batch 64 x 300)
    // two tiles take 36.6 against 34.2 with four.
    if (!lean && p->batch <= kShortChunkBatch) by_length = std::max({by_length, std::min(bound / 2, resident / 4), std::min(bound, resident / 8)});
    plan->num_chunks = (int)std::max<int64_t>(1, std::min<int64_t>(by_length, resident));
  }
  plan->slot_floats = (size_t)plan->rows * p->d_v + (size_t)32 * ng * wpg * ks;
  plan->wide_tiles = lean ? 0 : wide_tiles_of(p, *plan);
  plan->wide_chunks = plan->num_chunks;
  if (plan->wide_tiles > 0 && plan->chunk_tiles > 0) {
    const int64_t ct = (plan->chunk_tiles + 1) / 2, max64 = (max_tiles + 1) / 2;
    plan->wide_chunks = (int)(((int64_t)(plan->units / plan->mb) * max64 + ct - 1) / ct);
  }
  plan->list_bound = bound;
  // upper bound of the batch's cache bytes (the lengths are known on the device only) against the chip's
  // last-level cache
  plan->stream = bound * tok * 2 * ((int64_t)ng * p->d_v + p->d_rope) > kLastLevelCacheBytes;
  return true;
}

inline bool tuned_supported(const gla_decode_params* p, int is_gta) {
  TunedPlan plan;
  return tuned_plan(p, is_gta, false, &plan);
}

// Workspace: two partial slots per chunk, then per unit the chunk range holding it.
inline size_t tuned_slots_bytes(const TunedPlan& plan) {
  return (((size_t)std::max(plan.num_chunks, plan.wide_chunks) * plan.mb * 2 * plan.slot_floats * sizeof(float)) + 255) & ~(size_t)255;
}

inline size_t tuned_workspace(const gla_decode_params* p, int is_gta, bool lean) {
  TunedPlan plan;
  if (!tuned_plan(p, is_gta, lean, &plan)) return 0;
  return tuned_slots_bytes(plan) + (size_t)plan.units * 2 * sizeof(int32_t);
}

// Main and merge kernel of a plan, per state shape (tuned_256.hip, tuned_512.hip, tuned_128.hip), and the eight-wave
// main kernel that shares its merge (wide.hip).
int tuned_launch_256(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev);
int tuned_launch_512(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev);
int tuned_launch_128(const TunedPlan& plan, const DevParams& d, hipStream_t st, hipEvent_t* ev);
int wide_launch(const TunedPlan& plan, const DevParams& d, hipStream_t st);

inline int tuned_launch(const gla_decode_params* p, int is_gta, bool lean, DevParams& d, hipStream_t st,
                        hipEvent_t* ev) {
  TunedPlan plan;
  if (!tuned_plan(p, is_gta, lean, &plan)) return GLA_ERR_UNSUPPORTED_SHAPE;
  d.ws_out = (float*)p->workspace;
  d.ws_lse = (float*)((char*)p->workspace + tuned_slots_bytes(plan));  // per-unit chunk ranges (int32 pairs)
  d.num_chunks = plan.num_chunks;
  d.chunk_tiles = plan.chunk_tiles;
  {
    const int g_q = p->num_q_heads / p->num_groups;
    int lg = 0;
    while ((1 << lg) < p->page_size) ++lg;
    d.mb = plan.mb;
    d.upb = p->num_groups / plan.ng;
    d.lg_page = lg;
    d.xcd_map = (plan.num_chunks * plan.mb) % (8 * plan.mb) == 0 ? 1 : 0;
    d.tiles_full = (int)(((int64_t)p->max_pages_per_seq * p->page_size + plan.tok - 1) / plan.tok);
    const int64_t total_full = (int64_t)p->batch * d.upb * d.tiles_full;
    d.chunk_guess = plan.chunk_tiles > 0 ? plan.chunk_tiles
                                         : (int)((total_full + plan.num_chunks - 1) / plan.num_chunks);
    d.fd_mb = make_fastdiv((uint32_t)plan.mb);
    d.fd_chunks = make_fastdiv((uint32_t)plan.num_chunks);
    d.fd_gq = make_fastdiv((uint32_t)g_q);
    d.fd_tiles_full = make_fastdiv((uint32_t)d.tiles_full);
    d.fd_units_full = make_fastdiv((uint32_t)(d.upb * d.tiles_full));
    d.fd_upb_mb = make_fastdiv((uint32_t)(d.upb * plan.mb));
  }
  d.wide_tiles = plan.wide_tiles;
  d.setup_tiles = setup_tiles(plan.dv == 128 ? kSetupTiles128 : kSetupTiles, plan.list_bound);
  if (plan.dv == 256 && plan.dn == 256) return tuned_launch_256(plan, d, st, ev);
  if (plan.dv == 128 && plan.dn == 64) return tuned_launch_128(plan, d, st, ev);
  if (plan.dv == 512 && plan.dn == 512) return tuned_launch_512(plan, d, st, ev);
  return GLA_ERR_UNSUPPORTED_SHAPE;
}

}  // namespace gla
