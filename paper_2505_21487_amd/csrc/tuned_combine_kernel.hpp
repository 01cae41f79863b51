// Merge kernel of the tuned decode-attention path: combines the partial
// results the main kernel leaves for units that span several chunks.
#pragma once

#include "tuned_device.hpp"

namespace gla {

// Merge of the partial results of units that span several chunks, and zero fill
// of units without any key:  lse = ln sum_s exp(lse_s),
// out = sum_s exp(lse_s - lse) out_s.  The main kernel leaves, per unit, the
// range of chunks that hold it, and stores partial outputs in the register
// order of its waves, one contiguous 1 KiB block per wave, 32-dim block and
// quarter.
//
// Bound by the latency of a list's loads and by what one compute unit can pull (some 50 bytes per ns), then by the
// 33 MB of partials that a full grid leaves.  So the work of a unit is spread by the length of its list.  A panel is
// four 32-dim blocks of one wave of the main kernel, 16 blocks of 1 KiB per chunk.  A short list has one workgroup of
// four waves per panel, each wave taking four blocks over the whole list.  A longer one has up to 16 workgroups per
// panel ("sets"), each taking its share of the blocks, down to a block for one wave, two or all four, with
// four chunks in flight per wave (eight where four waves have one block: 4 to 32 per workgroup; 64 in the one of sixteen
// waves).  Every unit has 1 << merge_sets_lg sets (more than one in a small grid of long lists).  How many
// more only its list tells, so the workgroups beyond these belong to windows of merge_span chunks: the k-th window that
// lies inside a unit's list is its k-th further set, and the windows that are not needed leave.  Their number is that of the
// chunks over merge_span, however long or short the lists turn out.
// us per call, against four waves (or, by the mean length, one or sixteen) for every 32-dim block of every unit: GLA-2 15 x
// 1024 and 1 x 65536 tokens 56.8 -> 41.2, MLA shape 66.1 -> 53.6, GTA-4 10 sequences of up to 6000 20.7 -> 19.1, 1 x 100000
// 39.1 -> 35.1, GLA-2 1 x 131072 55.4 -> 53.6, 3 x 1000 19.1 -> 17.8, 64 x 8192 122.0 -> 120.6.
//
// Grid: (units * sets * panels, then windows * row blocks * panels), in rows where that is more than a grid's width.
template <int DV, int NG, int WPG, int KS, int TOK, int NW>
__global__ __launch_bounds__(64 * NW) void tuned_combine_kernel(DevParams p) {
  constexpr int NWAVES = NG * WPG * KS;
  constexpr int NDB = DV / KS / 32;  // 32-dim blocks per wave of the main kernel
  constexpr int kRows = 32 * NG * WPG;
  constexpr size_t kSlotFloats = (size_t)kRows * DV + 32 * NWAVES;
  constexpr int PANELS = NWAVES * NDB / 4;
  constexpr int kMaxSets = 16;
  static_assert(NDB % 4 == 0 && (PANELS & (PANELS - 1)) == 0, "panels of a unit");
  static_assert(NW == 4 || NW == 16, "waves per workgroup");
  __shared__ float red_m[NW][64], red_z[NW][64];
  __shared__ f32x4_t red_a[16][64];
  fetch_params();
  const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6);
  const int col = lane & 31, hi = lane >> 5;
  const int MB = p.mb;
  const int UPB = p.upb * MB;
  const unsigned block = blockIdx.y * gridDim.x + blockIdx.x, panel = block % PANELS, item = block / PANELS;
  const unsigned base_items = ((unsigned)p.B * (unsigned)UPB) << p.merge_sets_lg;

  int unit = (int)(item >> p.merge_sets_lg), set = (int)(item & ((1u << p.merge_sets_lg) - 1));  // unit: (sequence, group block, row block)
  int2 span = {0, 0};
  if (item >= base_items) {  // a window: whose?
    const unsigned n = item - base_items, win = fast_div(n, p.fd_mb);
    if (win >= (unsigned)p.merge_windows) return;  // (the grid's last row)
    const int mb = (int)(n - win * (unsigned)MB);
    const int w0 = (int)win * p.merge_span, w1 = w0 + p.merge_span - 1;
    const int n_units = p.B * p.upb;  // (row blocks apart: they share their chunks)
    unit = -1;
    for (int base = 0; base < n_units && unit < 0; base += 256) {
      int2 sp[4];
      int len[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = min(base + 64 * u + lane, n_units - 1);
        sp[u] = ((const int2*)p.ws_lse)[(int64_t)i * MB + mb];
        len[u] = p.seq_lens[(int)fast_div((unsigned)i * (unsigned)MB, p.fd_upb_mb)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        // (the range of a unit without tiles is garbage)
        const unsigned long long hit = __ballot(base + 64 * u + lane < n_units && len[u] > 0 && sp[u].x <= w0 && sp[u].y >= w1);
        if (hit && unit < 0) {
          const int src = __ffsll((long long)hit) - 1;
          unit = (base + 64 * u + src) * MB + mb;
          span.x = __builtin_amdgcn_readlane(sp[u].x, src);
          span.y = __builtin_amdgcn_readlane(sp[u].y, src);
        }
      }
    }
    if (unit < 0) return;  // (several units share these chunks)
    set = (int)win - (span.x + p.merge_span - 1) / p.merge_span + (1 << p.merge_sets_lg);
  }
  const int b = (int)fast_div((unsigned)unit, p.fd_upb_mb);
  const int ub = unit - b * UPB;
  const int gb = (int)fast_div((unsigned)ub, p.fd_mb), mb = ub - gb * MB;
  bool empty = false;
  if (item < base_items) {
    const int L = p.seq_lens[b];
    span = ((const int2*)p.ws_lse)[unit];  // garbage for units without tiles: not used then
    empty = tiles_of<TOK>(L) == 0;
    if (!empty && span.x == span.y) return;  // written directly by the main kernel
  }
  int sets = 1 << p.merge_sets_lg;
  if (!empty && p.merge_windows > 0) {
    const int inside = (span.y + 1) / p.merge_span - (span.x + p.merge_span - 1) / p.merge_span;
    while (sets < kMaxSets && 2 * sets <= inside + (1 << p.merge_sets_lg)) sets *= 2;
  }
  if (set >= sets) return;

  const int w = (int)panel * 4 / NDB, db0 = (int)panel * 4 % NDB;  // wave of the main kernel, its first 32-dim block
  const int wpos = w % (WPG * KS), kx = wpos % KS;
  const int rows_group = p.g_q * p.T;
  const int g = gb * NG + w / (WPG * KS);
  const int R = (mb * WPG + wpos / KS) * 32 + col;
  const bool valid = R < rows_group;  // (what pads a slab has no partials)
  if (__ballot(valid) == 0) return;   // (the same in every wave)
  const int Rc = valid ? R : 0;
  const int t = (int)fast_div((unsigned)Rc, p.fd_gq);
  const int h = g * p.g_q + (Rc - t * p.g_q);
  // Chunk span.x holds the unit's first tile (partial slot 1); every later
  // chunk sees a unit that began before it (slot 0).
  const int k_first = empty ? 0 : span.x, k_last = empty ? -1 : span.y;
  const float* const lse0 = p.ws_out + (size_t)kRows * DV + w * 32 + col;  // this row's entry among a slot's log-sum-exps
  const int64_t ob = b * p.out_s[0] + t * p.out_s[1] + h * p.out_s[2] + kx * (DV / KS);
  float* const lse_out = p.lse + ((int64_t)b * p.T + t) * p.h_q + h;
  const bool writes_lse = hi == 0 && kx == 0 && db0 == 0;

  // NQ consecutive blocks from block c0 (of the panel's 16) by kw waves, wave `share` of them taking every kw-th chunk:
  // one pass around a running reference, U chunks requested together.
  auto run = [&](auto nqc, auto uc, int c0, int share, int kw) {
    constexpr int NQ = decltype(nqc)::value, U = decltype(uc)::value;
    constexpr float kLog2e = 1.4426950408889634f;
    const float* const frag0 = p.ws_out + (size_t)((w * NDB + db0) * 4 + c0) * 256 + lane * 4;
    float m = -INFINITY, z = 0.f;
    f32x4_t acc[NQ];
#pragma unroll
    for (int c = 0; c < NQ; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // (the difference first: it is small where the weight counts, and so is then the error of the exponent)
    auto weight = [&](float ls, float ref) { return __builtin_amdgcn_exp2f((ls - ref) * kLog2e); };
    // everything so far to a reference that is not below it
    auto rebase = [&](float m_new) {
      const float keep = m == -INFINITY ? 0.f : weight(m, m_new);
      z *= keep;
#pragma unroll
      for (int c = 0; c < NQ; ++c) acc[c] *= keep;
      m = m_new;
    };
    if (valid) {
      for (int k = k_first + share; k <= k_last; k += U * kw) {
        float ls[U];
        f32x4_t v[U][NQ];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int ku = k + u * kw;
          ls[u] = -INFINITY;
          if (ku <= k_last) {
            const size_t so = (((size_t)ku * MB + mb) * 2 + (ku == k_first)) * kSlotFloats;
            ls[u] = lse0[so];
#pragma unroll
            for (int c = 0; c < NQ; ++c) v[u][c] = *(const f32x4_t*)(frag0 + so + c * 256);
          } else {
#pragma unroll
            for (int c = 0; c < NQ; ++c) v[u][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          }
        }
        float m_new = m;
#pragma unroll
        for (int u = 0; u < U; ++u) m_new = fmaxf(m_new, ls[u]);
        if (m_new == -INFINITY) continue;
        if (m_new != m) rebase(m_new);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // a slot marked "no key" may hold anything: its values are dropped, not multiplied by zero
          const bool live = ls[u] != -INFINITY;
          const float wgt = weight(ls[u], m);
          z += wgt;
#pragma unroll
          for (int c = 0; c < NQ; ++c) acc[c] += wgt * (live ? v[u][c] : f32x4_t{0.f, 0.f, 0.f, 0.f});
        }
      }
    }
    if (kw > 1) {  // the waves that share the blocks meet in the first of them
      if (share > 0) {
        red_m[wave][lane] = m;
        red_z[wave][lane] = z;
#pragma unroll
        for (int c = 0; c < NQ; ++c) red_a[wave * NQ + c][lane] = acc[c];
      }
      __syncthreads();
      if (share > 0) return;
      float m_new = m;
#pragma unroll
      for (int j = 1; j < NW; ++j)
        if (j < kw) m_new = fmaxf(m_new, red_m[wave + j][lane]);
      if (m_new != -INFINITY) {
        if (m_new != m) rebase(m_new);
#pragma unroll
        for (int j = 1; j < NW; ++j) {
          if (j >= kw) continue;
          const float wgt = weight(red_m[wave + j][lane], m);  // (no key: 0, as are the sums)
          z += wgt * red_z[wave + j][lane];
#pragma unroll
          for (int c = 0; c < NQ; ++c) acc[c] += wgt * red_a[(wave + j) * NQ + c][lane];
        }
      }
    }
    const float inv = z > 0.f ? 1.0f / z : 0.f;
#pragma unroll
    for (int c = 0; c < NQ; ++c) acc[c] *= inv;
    if (valid && writes_lse && c0 == 0) *lse_out = m == -INFINITY ? -INFINITY : m + logf(z);
    const int dim0 = (db0 + (c0 >> 2)) * 32 + (c0 & 3) * 8;  // first of the 8 * NQ dims that the two half-waves hold
    if (p.out_fp32) {
      if (valid) {
#pragma unroll
        for (int c = 0; c < NQ; ++c) *(f32x4_t*)((float*)p.out + ob + dim0 + 8 * c + 4 * hi) = acc[c];
      }
    } else if constexpr (NQ == 1) {
      if (valid) *(u32x2_t*)((uint16_t*)p.out + ob + dim0 + 4 * hi) = u32x2_t{cvt_pk_bf16(acc[0][0], acc[0][1]), cvt_pk_bf16(acc[0][2], acc[0][3])};
    } else {
#pragma unroll
      for (int c = 0; c < NQ; c += 2) {
        const u32x4_t v = join_halves_bf16(acc[c], acc[c + 1]);
        if (valid) store_b128_align8((uint16_t*)p.out + ob + dim0 + 8 * c + 8 * hi, v);
      }
    }
  };
  using std::integral_constant;
  constexpr integral_constant<int, 1> one{};
  constexpr integral_constant<int, 2> two{};
  constexpr integral_constant<int, 4> four{};
  constexpr integral_constant<int, 8> eight{};
  if constexpr (NW == 16) {  // (16 sets)
    run(one, four, set, wave, 16);
  } else {
    if (sets <= 4) run(four, four, 4 * (set * (4 / sets) + (wave & ~(sets - 1)) / sets), wave & (sets - 1), sets);
    else if (sets == 8) run(two, four, 2 * set, wave, 4);
    else run(one, eight, set, wave, 4);
  }
}

}  // namespace gla
