// Host side of the decode-attention library: argument checks, kernel choice,
// workspace sizing and launches.  The exported functions and their contracts
// are declared in include/gla_decode.h.
#include "../../include/gla_decode.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "common.hpp"
#include "flex_kernels.hpp"
#include "generic_kernels.hpp"
#include "generic_mfma_kernel.hpp"
#include "proj_kernels.hpp"
#include "proj_plan.hpp"
#include "tuned_kernels.hpp"

namespace gla {
namespace {

constexpr int kVersion = 105;  // 1.05: gla_decode_kernel_name

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// `is_gta` arguments: 0 = GLA / MLA shape, 1 = GTA, kModeGqa = grouped-query baseline with its own key cache.
constexpr int kModeGqa = 2;
// The key cache of a gqa_decode call in flight (host-side hand-over from the entry point to the launch code).
struct KeyCache {
  const void* ptr;
  int64_t stride[3];
};

int check_shape(const gla_decode_params* p, int is_gta) {
  if (!p) return GLA_ERR_INVALID_ARG;
  if (p->batch < 0 || p->q_len < 1 || p->q_len > 4) return GLA_ERR_INVALID_ARG;
  if (p->num_q_heads < 1 || p->num_groups < 1 || p->num_q_heads % p->num_groups != 0)
    return GLA_ERR_INVALID_ARG;
  if (p->d_v < 1 || p->d_nope < 1 || p->d_rope < 0) return GLA_ERR_INVALID_ARG;
  if (is_gta == kModeGqa) {
    if (p->d_rope != 0) return GLA_ERR_INVALID_ARG;  // (rotated dims are part of the cached key)
  } else if (is_gta) {
    if (p->d_v % 2 != 0 || p->d_nope != p->d_v / 2) return GLA_ERR_INVALID_ARG;
  } else {
    if (p->d_nope != p->d_v) return GLA_ERR_INVALID_ARG;
  }
  if (p->page_size < 1 || p->max_pages_per_seq < 1 || p->num_pages < 0) return GLA_ERR_INVALID_ARG;
  if (p->num_splits < 0) return GLA_ERR_INVALID_ARG;
  if (p->out_dtype != GLA_OUT_BF16 && p->out_dtype != GLA_OUT_FP32) return GLA_ERR_INVALID_ARG;
  if (p->impl != GLA_IMPL_AUTO && p->impl != GLA_IMPL_GENERIC && p->impl != GLA_IMPL_TUNED)
    return GLA_ERR_INVALID_ARG;
  if ((int64_t)p->batch * p->q_len * p->num_q_heads > (int64_t)0x7fffffff) return GLA_ERR_INVALID_ARG;
  return GLA_OK;
}

bool generic_supported(const gla_decode_params* p) { return p->d_v <= 1024 && p->d_nope <= 1024 && p->d_rope <= 128; }

// ---- flex kernel (flex_kernels.hpp): which instantiation, how the key tiles are cut into chunks
struct FlexPlan {
  int id;           // index into the instantiation list below, -1: none
  int gpw;          // groups per wave (2: two groups of at most eight rows share a wave's 16 rows)
  int rb;           // blocks of 16 rows per group
  int strands;      // (group block, row block) pairs: each walks the whole tile list
  int chunks;       // chunks of the tile list (one wave per chunk and strand)
  int chunk_tiles;  // > 0: fixed tiles per chunk; 0: ceil(total / chunks), worked out on the device
  bool lane;        // pages of fewer than 32 tokens: the kernel variant that forms one address per row and lane
  int64_t list_bound; // tiles of the list at most
};

int flex_variant(const gla_decode_params* p, int mode) {
  if (mode == kModeGqa) {
    if (p->d_nope == 128 && p->d_v == 128) return 0;
    if (p->d_nope == 64 && p->d_v == 64) return 1;
    return -1;
  }
  if (mode == 1) {  // GTA: tied state d_h, key = its first half + a RoPE key of d_h / 2
    if (p->d_v == 64 && p->d_rope == 32) return 2;
    if (p->d_v == 96 && p->d_rope == 48) return 3;
    return -1;
  }
  if (p->d_v == 128 && p->d_rope == 32) return 4;  // latent heads of 2 x 64 dims
  return -1;
}

bool flex_plan(const gla_decode_params* p, int mode, const KeyCache* kc, bool lean, FlexPlan* plan) {  // (lean: as in tuned_plan)
  plan->id = flex_variant(p, mode);
  if (plan->id < 0) return false;
  const int ps = p->page_size;
  if (ps < 1 || (ps & (ps - 1))) return false;
  plan->lane = ps < 32;  // (else a tile of 32 tokens lies inside one page)
  if (!(p->softmax_scale > 0.f)) return false;
  // layout the kernel assumes: contiguous rows, 16-byte aligned rows and bases
  if (p->state_stride[2] != p->d_v || p->state_stride[0] % 8 || p->state_stride[1] % 8) return false;
  if (p->d_rope > 0 && (p->rope_stride[1] != p->d_rope || p->rope_stride[0] % 8)) return false;
  for (int i = 0; i < 3; ++i)
    if (p->q_nope_stride[i] % 4 || (p->d_rope > 0 && p->q_rope_stride[i] % 4) || p->out_stride[i] % 4) return false;
  if (p->q_nope && (((uintptr_t)p->q_nope | (uintptr_t)p->q_rope) & 7u)) return false;
  if (p->q_nope && (((uintptr_t)p->state_cache | (uintptr_t)p->rope_cache | (uintptr_t)p->out) & 15u)) return false;
  if (mode == kModeGqa && kc && kc->ptr) {
    if (kc->stride[2] != p->d_nope || kc->stride[0] % 8 || kc->stride[1] % 8 || ((uintptr_t)kc->ptr & 15u)) return false;
  }
  const int rows_group = (p->num_q_heads / p->num_groups) * p->q_len;
  plan->rb = (rows_group + 15) / 16;
  plan->gpw = (plan->id == 2 && rows_group <= 8 && p->num_groups % 2 == 0) ? 2 : 1;
  plan->strands = (p->num_groups / plan->gpw) * plan->rb;
  // the tile list holds every sequence once; its length is known on the device only, here its upper bound
  const int64_t max_tiles = std::max<int64_t>(1, ((int64_t)p->max_pages_per_seq * ps + 31) / 32);
  const int64_t bound = (int64_t)p->batch * max_tiles;
  int64_t chunks;
  if (p->num_splits > 0) {
    plan->chunk_tiles = (int)((max_tiles + p->num_splits - 1) / p->num_splits);
    chunks = (bound + plan->chunk_tiles - 1) / plan->chunk_tiles;
  } else {
    // one wave per SIMD, chunks of at least four tiles (by the upper bound): a wave's start (lengths, page ids, queries,
    // first tile) costs several tiles' worth of time.  us per call with eight / five / four / three / two: GTA-4 d_h 64
    // 100 x 50 to 600 tokens 17.1 / 16.1 / 15.6 / 15.6 / 15.6, 10 sequences 14.5 / 14.0 / 13.9 / 14.6 / 14.6, d_h 96 3 x 3000 14.3 /
    // 14.3 / 14.3 / 13.7 / 13.4, GQA-4 6 sequences 15.0 / 15.0 / 14.5 / 15.1 / 15.1.  (Long sequences: FlexTraits::kPieces.)
    // (lean: eight, what a workspace was sized for before)
    plan->chunk_tiles = 0;
    const int64_t waves = device_cu_count();
    int64_t by_length = lean ? bound / 8 : bound / 4;
    // ... but while most of the chip is idle a shorter serial chain pays: chunks of two tiles up to half a wave per compute
    // unit.  us per call: GTA-4 d_h 64, batch 1 x 200 12.9 -> 11.0; GQA-4 batch 2 x 300 18.1 -> 11.9.
    if (!lean && p->batch <= kShortChunkBatch) by_length = std::max(by_length, std::min(bound / 2, waves / 2 / plan->strands));
    chunks = std::min<int64_t>((4 * waves + plan->strands - 1) / plan->strands, by_length);
  }
  chunks = std::max<int64_t>(1, chunks);
  if (chunks * plan->strands > (int64_t)0x3fffffff || bound + chunks > (int64_t)0x7fffffff) return false;
  plan->chunks = (int)chunks;
  plan->list_bound = bound;
  return true;
}

// Workspace: two partial slots of 16 rows per wave, then per (sequence, strand) the chunks holding its pieces.
size_t flex_slots(const FlexPlan& plan) { return (size_t)plan.chunks * plan.strands * 2 * 16; }
size_t flex_workspace(const gla_decode_params* p, const FlexPlan& plan) {
  return align_up(flex_slots(plan) * p->d_v * sizeof(float), 256) + align_up(flex_slots(plan) * sizeof(float), 256) +
         align_up((size_t)p->batch * plan.strands * 2 * sizeof(int32_t), 256);
}

// Workgroups of the generic MFMA kernel per range of tokens, about (64 rows each).
int64_t generic_units(const gla_decode_params* p) {
  return std::max<int64_t>(1, (int64_t)p->batch * p->num_groups * (((int64_t)p->num_q_heads / p->num_groups * p->q_len + 63) / 64));
}

// The generic MFMA kernel's shape for a call.
struct GenericPlan {
  int dvb, wr;      // dims and 16-row slabs per workgroup of the instantiation
  int ws;           // waves per slab
  bool half;        // half as many as fit: two workgroups and more per compute unit then
  int tile, meet;   // LDS bytes of a ring stage, and where the waves of a slab meet
  int per_cu;       // workgroups that a compute unit holds with two stages each (one or two)
};
GenericPlan generic_plan(const gla_decode_params* p, bool sepk) {
  GenericPlan g;
  const int dmax = std::max(p->d_v, p->d_nope), rows_group = p->num_q_heads / p->num_groups * p->q_len, cus = device_cu_count();
  g.dvb = dmax <= 128 ? 128 : dmax <= 256 ? 256 : 512;
  // as many slabs as the rows of a group fill, at most four
  g.wr = rows_group <= 16 ? 1 : rows_group <= 32 ? 2 : 4;
  g.ws = generic_ws(g.dvb, g.wr, sepk);
  // (short sequences that fill the chip as they are have no work for more waves: GTA-4 d_h 128, three positions, 77 x 23 tokens
  // 12.5 -> 7.4 us, GQA-4 87 x 1 to 52 13.7 -> 9.2; 64 x 4000 149 -> 154)
  g.half = g.ws > 1 && generic_units(p) >= cus && (int64_t)p->max_pages_per_seq * p->page_size <= 512;
  if (g.half) g.ws /= 2;
  const int cpr = p->d_v / 8 + (sepk ? p->d_nope : p->d_rope) / 8;
  g.tile = 32 * g.ws * (cpr | 1) * 16;
  g.meet = generic_meet_bytes(g.dvb, g.wr, g.ws);
  g.per_cu = std::max(2 * g.tile, g.meet) <= 80 * 1024 && 2 * g.wr * g.ws <= generic_max_waves(g.dvb) ? 2 : 1;
  return g;
}

// Ranges of fewer than 256 tokens (64 at least) that a sequence may fall into: as many as keep the grid within the compute
// units; where that would be less than four (a second range then gains little, and merging costs short sequences in a wide
// table more), or beyond 4096 tokens (longer: ranges of 256 are many already), within two thirds of them.  us per call with two
// thirds / all: GLA-2 9 x 2500 tokens 29.6 / 26.7, MLA shape 4 of 722 to 1922 36.4 / 33.7; 120 units of 29 tokens in a table for 128
// 9.9 / 19.1.  With a quarter / half / three quarters / all / twice as many: MLA shape 4 of 200 to 2500 59.0 / 39.8 / 36.2 / 33.1 /
// 33.1, GLA-2 2 x up to 5000 at two positions 28.4 / 23.4 / 23.2 / 21.2 / 21.2, 9 x up to 4500 31.2 up to all and 46.5 with twice
// as many.
int64_t small_ranges(int64_t units, bool longer) {
  const int64_t cus = device_cu_count();
  return cus / units >= 4 && !longer ? cus / units : cus * 2 / 3 / units;
}

// Ranges of the generic route.  The scalar kernel has one wave per row and range: about 4096 of them.
int scalar_splits(const gla_decode_params* p) {
  const int64_t rows = std::max<int64_t>(1, (int64_t)p->batch * p->q_len * p->num_q_heads);
  int64_t s = p->num_splits > 0 ? p->num_splits : (4096 + rows - 1) / rows;
  s = std::min<int64_t>(s, p->max_pages_per_seq);
  return (int)std::max<int64_t>(std::min<int64_t>(s, 65535), 1);
}

// The MFMA variant works on 64 rows at once: ranges for two workgroups per compute unit, no more than the longest
// sequence the table can hold is cut into (range_tokens), within 64 ranges (one per lane of the merge; beyond them it
// goes through the ranges one by one) and 64 MB of partials.  16 heads, one sequence of 30000 tokens: 93 us in 64
// ranges, 340 in the 235 that the scalar kernel's rule makes of it.
int mfma_splits(const gla_decode_params* p) {
  if (p->num_splits > 0) return scalar_splits(p);
  const int64_t rows = std::max<int64_t>(1, (int64_t)p->batch * p->q_len * p->num_q_heads);
  const int64_t units = generic_units(p), tokens = (int64_t)p->max_pages_per_seq * p->page_size;
  int64_t want = (2 * (int64_t)device_cu_count() + units - 1) / units;
  want = std::min(want, std::max((tokens + 255) / 256, std::min((tokens + 63) / 64, small_ranges(units, false))));
  // (not within one tile, and with many rows not for a second range of 64 tokens, which costs more in the merge: GLA-2 42 x 4
  // to 59 tokens in a table for 128 20.3 us, 11.7 in one; MLA shape with 16 heads, 75 x 8 to 80, 32 us, 37 in one)
  if (tokens <= 32 * generic_plan(p, false).ws || (tokens <= 128 && rows > 2048)) want = 1;
  want = std::min<int64_t>(want, (64ll << 20) / std::max<int64_t>(1, rows * (p->d_v + 1) * 4));
  return (int)std::max<int64_t>(std::min<int64_t>(want, 64), 1);
}

// Internal choice: GLA_IMPL_TUNED (the tuned kernel), kImplFlex (the second MFMA kernel, reported to
// callers as GLA_IMPL_TUNED: "an MFMA kernel"), GLA_IMPL_GENERIC, or an error.
constexpr int kImplFlex = 3;
int select_kernel(const gla_decode_params* p, int is_gta, const KeyCache* kc) {
  int rc = check_shape(p, is_gta);
  if (rc != GLA_OK) return rc;
  const bool tuned_ok = is_gta != kModeGqa && tuned_supported(p, is_gta);
  FlexPlan fp;
  const bool flex_ok = !tuned_ok && flex_plan(p, is_gta, kc, false, &fp);
  if (p->impl != GLA_IMPL_GENERIC) {
    if (tuned_ok) return GLA_IMPL_TUNED;
    if (flex_ok) return kImplFlex;
    if (p->impl == GLA_IMPL_TUNED) return GLA_ERR_UNSUPPORTED_SHAPE;
  }
  return generic_supported(p) ? GLA_IMPL_GENERIC : GLA_ERR_UNSUPPORTED_SHAPE;
}
int select_impl(const gla_decode_params* p, int is_gta) {
  const int k = select_kernel(p, is_gta, nullptr);
  return k == kImplFlex ? GLA_IMPL_TUNED : k;
}

// Does the MFMA variant of the generic kernel take this call?  Every 16-byte piece it loads or stores must be
// aligned: dims in steps of eight (value: sixteen), strides likewise, aligned bases.  (It computes what the scalar
// kernel computes, to the same precision: no size at which the scalar one is the better choice.)
bool generic_mfma_dims(const gla_decode_params* p) {
  if (p->d_v % 16 || p->d_nope % 8 || p->d_rope % 8 || std::max(p->d_v, p->d_nope) > 512) return false;
  return (int64_t)p->max_pages_per_seq * p->page_size <= (1ll << 30);  // (token indices and divisions in 32 bits)
}
bool generic_mfma_ok(const gla_decode_params* p, const KeyCache* kc) {
  if (!generic_mfma_dims(p)) return false;
  for (int i = 0; i < 3; ++i) {
    if (p->q_nope_stride[i] % 8 || p->state_stride[i] % 8 || p->out_stride[i] % 4) return false;
    if (p->d_rope > 0 && (p->q_rope_stride[i] % 8 || (i < 2 && p->rope_stride[i] % 8))) return false;
    if (kc && kc->stride[i] % 8) return false;
  }
  uintptr_t bases = (uintptr_t)p->q_nope | (uintptr_t)p->state_cache | (uintptr_t)p->out;
  if (p->d_rope > 0) bases |= (uintptr_t)p->q_rope | (uintptr_t)p->rope_cache;
  if (kc) bases |= (uintptr_t)kc->ptr;
  return (bases & 15u) == 0;
}

size_t generic_bytes(const gla_decode_params* p, int splits) {
  if (splits == 1) return 0;
  const size_t rows = (size_t)p->batch * p->q_len * p->num_q_heads;
  return align_up((size_t)splits * rows * p->d_v * sizeof(float), 256) + align_up((size_t)splits * rows * sizeof(float), 256);
}

// (lean: what the scalar kernel's ranges need; else enough for either kernel, as strides and pointers may not be known yet)
size_t generic_workspace(const gla_decode_params* p, bool lean) {
  const size_t scalar = generic_bytes(p, scalar_splits(p));
  return lean || !generic_mfma_dims(p) ? scalar : std::max(scalar, generic_bytes(p, mfma_splits(p)));
}

int check_pointers(const gla_decode_params* p) {
  if (p->batch == 0) return GLA_OK;
  if (!p->q_nope || !p->state_cache || !p->page_table || !p->seq_lens || !p->out || !p->lse)
    return GLA_ERR_INVALID_ARG;
  if (p->d_rope > 0 && (!p->q_rope || !p->rope_cache)) return GLA_ERR_INVALID_ARG;
  return GLA_OK;
}

template <int DN, int DR, int DV, bool SEPK, int GPW>
int launch_flex_kernels(bool lane, dim3 grid, dim3 rows, hipStream_t st, hipEvent_t* ev, const DevParams& d) {
  if (ev) (void)hipEventRecord(ev[0], st);
  if (lane) hipLaunchKernelGGL((flex_main_kernel<DN, DR, DV, SEPK, GPW, true>), grid, dim3(256), 0, st, d);
  else hipLaunchKernelGGL((flex_main_kernel<DN, DR, DV, SEPK, GPW, false>), grid, dim3(256), 0, st, d);
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  if (ev) (void)hipEventRecord(ev[1], st);
  // (always: it also fills the rows of empty sequences, which no chunk holds)
  hipLaunchKernelGGL((flex_combine_kernel<DV, GPW>), rows, dim3(64), 0, st, d);
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  if (ev) (void)hipEventRecord(ev[2], st);
  return GLA_OK;
}

int launch_flex(const gla_decode_params* p, const FlexPlan& plan, DevParams& d, hipStream_t st, hipEvent_t* ev) {
  d.num_chunks = plan.chunks;
  d.chunk_tiles = plan.chunk_tiles;
  d.flex_rb = plan.rb;
  d.setup_tiles = setup_tiles(kSetupTilesFlex, plan.list_bound);
  d.fd_chunks = make_fastdiv((uint32_t)plan.chunks);
  d.fd_strands = make_fastdiv((uint32_t)plan.strands);
  d.fd_group_blocks = make_fastdiv((uint32_t)(p->num_groups / plan.gpw));
  d.fd_heads = make_fastdiv((uint32_t)p->num_q_heads);
  d.fd_q_len = make_fastdiv((uint32_t)p->q_len);
  d.fd_gq = make_fastdiv((uint32_t)(p->num_q_heads / p->num_groups));
  int lg = 0;
  while ((1 << lg) < p->page_size) ++lg;
  d.lg_page = lg;
  const size_t rows = (size_t)p->batch * p->q_len * p->num_q_heads;
  {
    char* w = (char*)p->workspace;
    d.ws_out = (float*)w;
    w += align_up(flex_slots(plan) * p->d_v * sizeof(float), 256);
    d.ws_lse = (float*)w;
    w += align_up(flex_slots(plan) * sizeof(float), 256);
    d.flex_rng = (int32_t*)w;
  }
  const int64_t waves = (int64_t)plan.chunks * plan.strands;
  const dim3 grid((unsigned)((waves + 3) / 4)), merge((unsigned)rows);
  switch (plan.id) {
    case 0: return launch_flex_kernels<128, 0, 128, true, 1>(plan.lane, grid, merge, st, ev, d);
    case 1: return launch_flex_kernels<64, 0, 64, true, 1>(plan.lane, grid, merge, st, ev, d);
    case 2:
      return plan.gpw == 2 ? launch_flex_kernels<32, 32, 64, false, 2>(plan.lane, grid, merge, st, ev, d)
                           : launch_flex_kernels<32, 32, 64, false, 1>(plan.lane, grid, merge, st, ev, d);
    case 3: return launch_flex_kernels<48, 48, 96, false, 1>(plan.lane, grid, merge, st, ev, d);
    case 4: return launch_flex_kernels<128, 32, 128, false, 1>(plan.lane, grid, merge, st, ev, d);
    default: return GLA_ERR_UNSUPPORTED_SHAPE;
  }
}

void fill_dev(const gla_decode_params* p, DevParams* d) {
  std::memset(d, 0, sizeof(*d));
  d->q_nope = (const uint16_t*)p->q_nope;
  d->q_rope = (const uint16_t*)p->q_rope;
  d->state = (const uint16_t*)p->state_cache;
  d->rope = (const uint16_t*)p->rope_cache;
  d->page_table = p->page_table;
  d->seq_lens = p->seq_lens;
  d->out = p->out;
  d->lse = p->lse;
  for (int i = 0; i < 3; ++i) {
    d->qn_s[i] = p->q_nope_stride[i];
    d->qr_s[i] = p->q_rope_stride[i];
    d->st_s[i] = p->state_stride[i];
    d->out_s[i] = p->out_stride[i];
  }
  d->rp_s[0] = p->rope_stride[0];
  d->rp_s[1] = p->rope_stride[1];
  d->B = p->batch;
  d->T = p->q_len;
  d->h_q = p->num_q_heads;
  d->h_c = p->num_groups;
  d->g_q = p->num_q_heads / p->num_groups;
  d->d_v = p->d_v;
  d->d_n = p->d_nope;
  d->d_r = p->d_rope;
  d->P = p->page_size;
  d->max_pages = p->max_pages_per_seq;
  d->causal = p->causal ? 1 : 0;
  d->out_fp32 = p->out_dtype == GLA_OUT_FP32;
  d->scale = p->softmax_scale;
  d->stream_min_bytes = kLastLevelCacheBytes;
}

template <int DVB, int WR, bool SEPK>
void launch_generic_mfma_waves(const GenericPlan& g, dim3 grid, size_t lds, hipStream_t st, const DevParams& d) {
  constexpr int WS = generic_ws(DVB, WR, SEPK), HALF = WS > 1 ? WS / 2 : 1;
  if (g.half) hipLaunchKernelGGL((generic_mfma_kernel<DVB, WR, HALF, SEPK>), grid, dim3(64 * WR * HALF), lds, st, d);
  else hipLaunchKernelGGL((generic_mfma_kernel<DVB, WR, WS, SEPK>), grid, dim3(64 * WR * WS), lds, st, d);
}

template <bool SEPK>
void launch_generic_mfma(const gla_decode_params* p, DevParams& d, hipStream_t st) {
  const GenericPlan g = generic_plan(p, SEPK);
  const int64_t tokens = (int64_t)p->max_pages_per_seq * p->page_size;
  if (p->num_splits > 0) d.split_tokens = (int32_t)(((tokens + d.splits - 1) / d.splits + 31) / 32 * 32);
  d.small_ranges = (int32_t)small_ranges(generic_units(p), false);
  d.small_ranges_longer = (int32_t)small_ranges(generic_units(p), true);
  // One round instead of two (range_tokens): with one workgroup per compute unit, two ranges at least, and less than a tenth
  // more of the chip busy in two (GQA-4 with 256 dims, 18 x 1353 to 2545 tokens, 72 units: seven ranges 100 us, three 128; 53 x
  // up to 1061, 212 units: three 117, one 153).
  const int64_t units = generic_units(p), cus = device_cu_count(), one = cus / units, two = 2 * cus / units;
  d.resident = (int32_t)cus;
  d.one_round = g.per_cu == 1 && one >= 2 && 10 * two <= 11 * 2 * one ? (int32_t)one : 1 << 20;
  d.fd_page = make_fastdiv((uint32_t)p->page_size);
  d.fd_cpr = make_fastdiv((uint32_t)(p->d_v / 8 + (SEPK ? p->d_nope : p->d_rope) / 8) | 1u);
  const int rows_group = p->num_q_heads / p->num_groups * p->q_len;
  const dim3 grid((unsigned)((int64_t)p->batch * p->num_groups * ((rows_group + 16 * g.wr - 1) / (16 * g.wr))), (unsigned)d.splits);
  // Ring: as deep as the LDS allows, four stages at most; but where the grid fills the chip and two workgroups fit into a
  // compute unit, as deep as leaves room for both (MLA shape with 16 heads, one wave per workgroup, 16 x 8000 tokens 178 ->
  // 106 us, GTA-4 d_h 64 64 x 4000 105 -> 63).  Half the waves: two stages.
  const bool full = (int64_t)grid.x * grid.y > device_cu_count();
  d.ring_stages = g.half ? 2 : std::min(4, (full && g.per_cu == 2 ? 80 : 160) * 1024 / g.tile);
  const size_t lds = (size_t)std::max(d.ring_stages * g.tile, g.meet);
  switch (g.dvb * 10 + g.wr) {
    case 1281: launch_generic_mfma_waves<128, 1, SEPK>(g, grid, lds, st, d); break;
    case 1282: launch_generic_mfma_waves<128, 2, SEPK>(g, grid, lds, st, d); break;
    case 1284: launch_generic_mfma_waves<128, 4, SEPK>(g, grid, lds, st, d); break;
    case 2561: launch_generic_mfma_waves<256, 1, SEPK>(g, grid, lds, st, d); break;
    case 2562: launch_generic_mfma_waves<256, 2, SEPK>(g, grid, lds, st, d); break;
    case 2564: launch_generic_mfma_waves<256, 4, SEPK>(g, grid, lds, st, d); break;
    case 5121: launch_generic_mfma_waves<512, 1, SEPK>(g, grid, lds, st, d); break;
    case 5122: launch_generic_mfma_waves<512, 2, SEPK>(g, grid, lds, st, d); break;
    default: launch_generic_mfma_waves<512, 4, SEPK>(g, grid, lds, st, d); break;
  }
}

int launch_generic(const gla_decode_params* p, const KeyCache* kc, bool lean, DevParams& d, hipStream_t st, hipEvent_t* ev) {
  const bool mfma = generic_mfma_ok(p, kc);
  const int s = mfma && !lean ? mfma_splits(p) : scalar_splits(p);
  d.splits = s;
  d.pages_per_split = (p->max_pages_per_seq + s - 1) / s;
  const size_t rows = (size_t)p->batch * p->q_len * p->num_q_heads;
  if (s > 1) {
    d.ws_out = (float*)p->workspace;
    d.ws_lse = (float*)((char*)p->workspace + align_up((size_t)s * rows * p->d_v * sizeof(float), 256));
  }
  dim3 grid((unsigned)rows, (unsigned)s), block(64);
  const int nv = (std::max(p->d_v, p->d_nope) + 63) / 64;
  if (ev) (void)hipEventRecord(ev[0], st);
  if (mfma && kc) launch_generic_mfma<true>(p, d, st);
  else if (mfma) launch_generic_mfma<false>(p, d, st);
  else if (nv <= 2) hipLaunchKernelGGL(generic_main_kernel<2>, grid, block, 0, st, d);
  else if (nv <= 4) hipLaunchKernelGGL(generic_main_kernel<4>, grid, block, 0, st, d);
  else if (nv <= 8) hipLaunchKernelGGL(generic_main_kernel<8>, grid, block, 0, st, d);
  else hipLaunchKernelGGL(generic_main_kernel<16>, grid, block, 0, st, d);
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  if (ev) (void)hipEventRecord(ev[1], st);
  if (s > 1) {
    hipLaunchKernelGGL(generic_combine_kernel, dim3((unsigned)rows), block, 0, st, d);
    if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  }
  if (ev) (void)hipEventRecord(ev[2], st);
  return GLA_OK;
}

size_t workspace_need(const gla_decode_params* p, int is_gta, int kernel, const KeyCache* kc, bool lean) {
  if (kernel == GLA_IMPL_TUNED) return tuned_workspace(p, is_gta, lean);
  if (kernel == kImplFlex) {
    FlexPlan fp;
    return flex_plan(p, is_gta, kc, lean, &fp) ? flex_workspace(p, fp) : 0;
  }
  return generic_workspace(p, lean);
}

// What gla_decode_workspace_size() reports: never less than for a smaller batch on the MFMA kernels, so that a program
// may size its workspace once, for its largest batch.  (Batches of up to kShortChunkBatch may be cut into more chunks
// than larger ones; among themselves, and beyond it, the need grows with the batch.)
size_t workspace_reported(const gla_decode_params* p, int is_gta, int kernel) {
  size_t need = workspace_need(p, is_gta, kernel, nullptr, false);
  if (p->batch > kShortChunkBatch && kernel != GLA_IMPL_GENERIC) {
    gla_decode_params small = *p;
    small.batch = kShortChunkBatch;
    need = std::max(need, workspace_need(&small, is_gta, kernel, nullptr, false));
  }
  return need;
}

int run(const gla_decode_params* p, int is_gta, hipEvent_t* ev, const KeyCache* kc = nullptr) {
  const int impl = select_kernel(p, is_gta, kc);
  if (impl < 0) return impl;
  int rc = check_pointers(p);
  if (rc != GLA_OK) return rc;
  if (is_gta == kModeGqa && p->batch > 0 && (!kc || !kc->ptr)) return GLA_ERR_INVALID_ARG;
  if (p->batch == 0) return GLA_OK;
  // A workspace that is too small for the plan of this call may do for the lean one: the call then runs on that (more
  // slowly, and with the roundings of its chunks) and is not refused.
  size_t need = workspace_need(p, is_gta, impl, kc, false);
  const bool lean = need > p->workspace_bytes;
  if (lean) need = workspace_need(p, is_gta, impl, kc, true);
  if (need > 0 && (!p->workspace || p->workspace_bytes < need)) return GLA_ERR_WORKSPACE_TOO_SMALL;
  if (need > 0 && ((uintptr_t)p->workspace & 255u)) return GLA_ERR_INVALID_ARG;
  DevParams d;
  fill_dev(p, &d);
  if (is_gta == kModeGqa) {
    d.kstate = (const uint16_t*)kc->ptr;
    for (int i = 0; i < 3; ++i) d.k_s[i] = kc->stride[i];
  }
  hipStream_t st = (hipStream_t)p->stream;
  if (impl == GLA_IMPL_TUNED) return tuned_launch(p, is_gta, lean, d, st, ev);
  if (impl == kImplFlex) {
    FlexPlan fp;
    if (!flex_plan(p, is_gta, kc, lean, &fp)) return GLA_ERR_UNSUPPORTED_SHAPE;
    return launch_flex(p, fp, d, st, ev);
  }
  return launch_generic(p, kc, lean, d, st, ev);
}

// Name of the kernel that does a call's main work; tiles32: sum over the sequences of ceil(length / 32).
const char* kernel_name(const gla_decode_params* p, int is_gta, int64_t tiles32) {
  const int impl = select_kernel(p, is_gta, nullptr);
  if (impl < 0) return "";
  if (impl == kImplFlex) return "second MFMA kernel";
  if (impl == GLA_IMPL_GENERIC) return generic_mfma_ok(p, nullptr) ? "generic MFMA kernel" : "scalar kernel";
  TunedPlan plan;
  tuned_plan(p, is_gta, false, &plan);
  return plan.wide_tiles > 0 && tiles32 * (p->num_groups / plan.ng) >= plan.wide_tiles ? "eight-wave kernel" : "four-wave kernel";
}

// ---- fixed scratch buffer of the allocation-free entry point -------------------
// One array per GPU the library runs on, in that GPU's memory for the lifetime
// of the process.  In host code the array's name is only a handle: the device
// address is asked for once per device (with that device current) and every
// later use goes through the address kept here.
constexpr size_t kScratchBytes = (size_t)GLA_DECODE_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
static void* scratch_addr[kMaxDevices];  // device address of `scratch` per device, null until asked for
static std::mutex scratch_mutex;

int scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GLA_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_addr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return GLA_ERR_LAUNCH;
    }
    scratch_addr[dev] = ptr;
  }
  *out = scratch_addr[dev];
  return GLA_OK;
}

int run_noalloc(const gla_decode_params* p, int is_gta) {
  const int impl = select_impl(p, is_gta);
  if (impl < 0) return impl;
  const int kernel = select_kernel(p, is_gta, nullptr);
  if (std::min(workspace_need(p, is_gta, kernel, nullptr, false), workspace_need(p, is_gta, kernel, nullptr, true)) > kScratchBytes) return GLA_ERR_WORKSPACE_TOO_SMALL;  // beyond the fixed buffer: use gla_decode / gta_decode
  gla_decode_params q = *p;
  void* ptr = nullptr;
  if (p->batch > 0) {
    const int rc = scratch_of_current_device(&ptr);
    if (rc != GLA_OK) return rc;
  }
  q.workspace = ptr;
  q.workspace_bytes = kScratchBytes;
  // (nothing in the buffer has to start at zero: every word a call reads back
  // was written by that call's own kernels first)
  return run(&q, is_gta, nullptr);
}

// ---- projections around the attention ------------------------------------------
template <int MT>
void launch_proj_long(bool stream, dim3 grid, hipStream_t st, const ProjParams& d) {
  if (stream) hipLaunchKernelGGL((proj_kernel<MT, 2, true>), grid, dim3(256), 0, st, d);
  else hipLaunchKernelGGL((proj_kernel<MT, 2, false>), grid, dim3(256), 0, st, d);
}

int run_proj(const gla_proj_params* p, int sum_groups) {
  ProjPlan plan;
  int rc = proj_plan(p, sum_groups, device_cu_count(), 0, &plan);
  for (int small = 1; small <= 2 && rc == GLA_OK && plan.part_bytes > p->workspace_bytes; ++small)
    rc = proj_plan(p, sum_groups, device_cu_count(), small, &plan);
  if (rc != GLA_OK) return rc;
  if (p->rows == 0) return GLA_OK;
  if (!p->a || !p->w || !p->c) return GLA_ERR_INVALID_ARG;
  if (((uintptr_t)p->a | (uintptr_t)p->w | (uintptr_t)p->c) & 15u) return GLA_ERR_UNSUPPORTED_SHAPE;
  if (plan.part_bytes > 0 && (!p->workspace || p->workspace_bytes < plan.part_bytes)) return GLA_ERR_WORKSPACE_TOO_SMALL;
  if (plan.part_bytes > 0 && ((uintptr_t)p->workspace & 255u)) return GLA_ERR_INVALID_ARG;
  ProjParams d;
  d.a = (const uint16_t*)p->a;
  d.w = (const uint16_t*)p->w;
  d.c = p->c;
  d.part = (float*)p->workspace;
  d.a_row = p->a_row_stride;
  d.a_group = p->a_group_stride;
  d.c_row = p->c_row_stride;
  d.c_group = p->c_group_stride;
  d.M = p->rows;
  d.N = p->n;
  d.K = p->k;
  d.ksplit = plan.ksplit;
  d.k_per_split = plan.k_per_split;
  d.sum_groups = sum_groups ? 1 : 0;
  d.c_fp32 = p->c_dtype == GLA_OUT_FP32;
  d.direct = plan.direct ? 1 : 0;
  hipStream_t st = (hipStream_t)p->stream;
  const int wg_n = 128 * plan.nt;
  const unsigned blocks = (unsigned)((p->n + wg_n - 1) / wg_n), tiles = (unsigned)((p->rows + 32 * plan.mt - 1) / (32 * plan.mt));
  const unsigned slices = (unsigned)(p->groups * plan.ksplit);
  if (tiles > 65535u || slices > 65535u) return GLA_ERR_UNSUPPORTED_SHAPE;
  // (One dimension of a launch holds fewer than 2^24 workgroups of 256 threads.  The list is shorter: at most 2^31 results, at
  // least some 33 rows x 32 features each, make 2^21 workgroups per range, and proj_plan cuts the sums of no more than 1000 rounds
  // of workgroups, into 64 ranges at most.)
  const dim3 grid = plan.placed ? dim3(blocks * tiles * slices) : dim3(blocks, tiles, slices);
  d.total = plan.placed ? grid.x : 0;
  d.tiles = tiles;
  d.blocks = blocks;
  d.by_tiles = proj_reciprocal(tiles);
  d.by_blocks = proj_reciprocal(blocks);
  d.by_ksplit = proj_reciprocal((uint32_t)plan.ksplit);
  d.rotated = plan.rotated ? 1 : 0;
  if (plan.nt == 2) {
    if (plan.mt == 1) launch_proj_long<1>(plan.stream, grid, st, d);
    else if (plan.mt == 2) launch_proj_long<2>(plan.stream, grid, st, d);
    else launch_proj_long<4>(plan.stream, grid, st, d);
  } else {
    if (plan.mt == 1) hipLaunchKernelGGL((proj_kernel<1, 1, false>), grid, dim3(256), 0, st, d);
    else hipLaunchKernelGGL((proj_kernel<2, 1, false>), grid, dim3(256), 0, st, d);
  }
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  if (!plan.direct) {
    const int64_t outs = (int64_t)p->rows * (sum_groups ? 1 : p->groups) * (p->n / 4);
    ProjReduceParams q;
    q.part = d.part;
    q.c = d.c;
    q.c_row = d.c_row;
    q.c_group = sum_groups ? 0 : d.c_group;
    q.M = d.M;
    q.N = d.N;
    q.outs = sum_groups ? 1u : (uint32_t)p->groups;
    q.slices = sum_groups ? p->groups * plan.ksplit : plan.ksplit;
    q.c_fp32 = d.c_fp32;
    q.by_n4 = make_fastdiv((uint32_t)p->n / 4);
    q.by_outs = make_fastdiv(q.outs);
    hipLaunchKernelGGL(proj_reduce_kernel, dim3((unsigned)((outs + 255) / 256)), dim3(256), 0, st, q);
    if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  }
  return GLA_OK;
}

__global__ void zero_int_kernel(int* x) { *x = 0; }

// Device contents the decode kernels trust: one thread per (sequence, table
// entry).  Counts lengths outside [0, max_pages * page_size] and held table
// entries outside [0, num_pages) into *bad (a vector-memory atomic).
__global__ void check_contents_kernel(const int32_t* seq_lens, const int32_t* page_table, int B, int max_pages,
                                      int page_size, int64_t num_pages, int* bad) {
  // (the batch is folded into grid.x: grid.y would cap it at 65535 sequences)
  const int bpr = (max_pages + (int)blockDim.x - 1) / (int)blockDim.x;  // blocks per table row
  const int b = (int)(blockIdx.x / (unsigned)bpr);
  const int j = (int)(blockIdx.x % (unsigned)bpr) * (int)blockDim.x + (int)threadIdx.x;
  if (b >= B) return;
  const int L = seq_lens[b];
  const int64_t cap = (int64_t)max_pages * page_size;
  if (L < 0 || L > cap) {
    if (j == 0) atomicAdd(bad, 1);
    return;
  }
  const int held = (L + page_size - 1) / page_size;
  if (j < held) {
    const int32_t pg = page_table[(int64_t)b * max_pages + j];
    if (pg < 0 || (int64_t)pg >= num_pages) atomicAdd(bad, 1);
  }
}

int check_contents(const gla_decode_params* p, int is_gta, int* n_bad) {
  const int impl = select_impl(p, is_gta);
  if (impl < 0) return impl;
  int rc = check_pointers(p);
  if (rc != GLA_OK) return rc;
  if (!n_bad || p->num_pages <= 0) return GLA_ERR_INVALID_ARG;
  *n_bad = 0;
  if (p->batch == 0) return GLA_OK;
  if (!p->workspace || p->workspace_bytes < 256) return GLA_ERR_WORKSPACE_TOO_SMALL;
  hipStream_t st = (hipStream_t)p->stream;
  int* counter = (int*)p->workspace;
  hipLaunchKernelGGL(zero_int_kernel, dim3(1), dim3(1), 0, st, counter);
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  const int threads = 256;
  const int64_t blocks = (int64_t)((p->max_pages_per_seq + threads - 1) / threads) * p->batch;
  if (blocks > 0x7fffffff) return GLA_ERR_INVALID_ARG;
  const dim3 grid((unsigned)blocks);
  hipLaunchKernelGGL(check_contents_kernel, grid, dim3(threads), 0, st, p->seq_lens, p->page_table, p->batch,
                     p->max_pages_per_seq, p->page_size, p->num_pages, counter);
  if (hipGetLastError() != hipSuccess) return GLA_ERR_LAUNCH;
  if (hipMemcpyAsync(n_bad, counter, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return GLA_ERR_LAUNCH;
  return GLA_OK;
}

}  // namespace
}  // namespace gla

extern "C" {

int gla_decode_check_contents(const gla_decode_params* p, int is_gta, int* n_bad) {
  return gla::check_contents(p, is_gta, n_bad);
}

int gla_decode(const gla_decode_params* p) { return gla::run(p, 0, nullptr); }

int gta_decode(const gla_decode_params* p) { return gla::run(p, 1, nullptr); }

int gla_decode_noalloc(const gla_decode_params* p, int is_gta) { return gla::run_noalloc(p, is_gta); }

size_t gla_decode_workspace_size(const gla_decode_params* p, int is_gta) {
  const int impl = gla::select_kernel(p, is_gta, nullptr);
  if (impl < 0) return 0;
  // A little more than nothing, so callers can always pass a real buffer.
  return std::max<size_t>(gla::workspace_reported(p, is_gta, impl), 256);
}

int gqa_decode(const gla_decode_params* p, const void* key_cache, const int64_t* key_stride) {
  if (!key_stride) return GLA_ERR_INVALID_ARG;
  const gla::KeyCache kc = {key_cache, {key_stride[0], key_stride[1], key_stride[2]}};
  return gla::run(p, gla::kModeGqa, nullptr, &kc);
}

int gla_absorb_query(const gla_proj_params* p) { return gla::run_proj(p, 0); }

int gla_output_proj(const gla_proj_params* p) { return gla::run_proj(p, 1); }

size_t gla_proj_workspace_size(const gla_proj_params* p, int sum_groups) {
  return gla::proj_workspace(p, sum_groups, gla::device_cu_count());
}

int gla_decode_select_impl(const gla_decode_params* p, int is_gta) {
  return gla::select_impl(p, is_gta);
}

const char* gla_decode_kernel_name(const gla_decode_params* p, int is_gta, int64_t tiles32) {
  return gla::kernel_name(p, is_gta, tiles32);
}

int gla_decode_profile(const gla_decode_params* p, int is_gta, int iters, float* main_us,
                       float* combine_us) {
  if (!p || !main_us || !combine_us || iters < 1 || iters > 256) return GLA_ERR_INVALID_ARG;
  hipEvent_t ev[3 * 256];
  int made = 0;
  int rc = GLA_OK;
  for (; made < 3 * iters; ++made)
    if (hipEventCreate(&ev[made]) != hipSuccess) { rc = GLA_ERR_LAUNCH; break; }
  for (int i = 0; rc == GLA_OK && i < iters; ++i) rc = gla::run(p, is_gta, &ev[3 * i]);
  if (hipStreamSynchronize((hipStream_t)p->stream) != hipSuccess && rc == GLA_OK) rc = GLA_ERR_LAUNCH;
  if (rc == GLA_OK && p->batch > 0) {
    double a = 0, b = 0;
    for (int i = 0; i < iters; ++i) {
      float t0 = 0, t1 = 0;
      if (hipEventElapsedTime(&t0, ev[3 * i], ev[3 * i + 1]) != hipSuccess ||
          hipEventElapsedTime(&t1, ev[3 * i + 1], ev[3 * i + 2]) != hipSuccess) {
        rc = GLA_ERR_LAUNCH;
        break;
      }
      a += t0;
      b += t1;
    }
    *main_us = (float)(a * 1000.0 / iters);
    *combine_us = (float)(b * 1000.0 / iters);
  } else {
    *main_us = *combine_us = 0.f;
  }
  for (int i = 0; i < made; ++i) (void)hipEventDestroy(ev[i]);
  return rc;
}

const char* gla_status_string(int status) {
  switch (status) {
    case GLA_OK: return "ok";
    case GLA_ERR_INVALID_ARG: return "invalid argument";
    case GLA_ERR_UNSUPPORTED_SHAPE: return "no kernel for this shape with the requested implementation";
    case GLA_ERR_WORKSPACE_TOO_SMALL: return "workspace missing or too small (allocation-free entry point: the problem needs more than its fixed buffer)";
    case GLA_ERR_LAUNCH: return "HIP launch or event call failed";
    default: return "unknown status";
  }
}

int gla_decode_version(void) { return gla::kVersion; }

}  // extern "C"
