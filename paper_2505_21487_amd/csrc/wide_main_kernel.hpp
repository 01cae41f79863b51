// Split-KV main kernel with eight waves per workgroup, for units with so many
// query rows that the matrix pipe and not HBM sets the pace (GLA with two or
// more query positions, the 512-dim latent): two waves per SIMD, so that one
// wave's softmax, LDS latency and load issue run under the other's MFMAs.
//
// What makes two waves per SIMD possible is that no wave holds a whole row
// slab's output.  The two halves of a tile's work are split differently:
//   scores   a wave computes the scores of HALF the tile's tokens (32 of 64) for
//            its query rows, over all contraction dims: the softmax of those
//            scores is complete in the wave and done once;
//   values   a wave accumulates 128 of the output dims for ALL tokens of the
//            tile and all 32 rows of a slab (64 accumulation registers).
// In between the bf16 weights go through LDS in MFMA operand order (4 KB per
// slab and tile).  Four waves form a group that owns its rows (two slabs of 32
// with 256 dims, one with 512); the two groups of a workgroup share the tiles.
//
// Weights are relative to a per-row reference that is moved only when a row
// maximum exceeds it by more than 2^8.  References are whole numbers (log2
// domain), so that the two waves holding the two token halves of a row need
// not agree on it before they form their weights: a wave that moves its
// reference raises a flag, and behind the barrier the value phase rescales
// accumulators and weights by exact powers of two.  The row sums (of the fp32
// weights for the log-sum-exp, of the rounded weights for the normalisation)
// stay in the wave that formed the weights and meet at the end of a segment.
//
// Schedule.  256 dims (three ring stages): the groups run half a tile apart, one in its score half-step (matrix and
// vector pipe) while the other is in its value half-step (matrix pipe, tile loads).  512 dims (two stages of 72 KB):
// both groups in the same half-step.
//
// What bounds it: latency chains inside a half-step more than any one pipe.  Measured per tile of 64 tokens and 128
// rows (256 dims): 4900 cycles, of which the matrix pipe is busy for 2300, LDS for 1650, the vector pipe for about
// 2000 in the two waves of a SIMD; without the tile loads 3900, without the value MFMAs 3800.  The four-wave kernel
// takes 5000 cycles for the same work with one address per 64-token page, and more with small pages, whose address
// work here hides under the other wave.  Times: see wide_tiles_of() in tuned_host.hpp.
//
// Rare paths (a moved reference, heavy weights, tails) are written so that nothing in them costs the tile loop
// registers or waits: LDS accesses as assembly, indices worked out on the spot.  A first version whose rare path
// spilled two registers spent 20 000 cycles in it each time, waiting for every tile load in flight.
#pragma once

#include "tuned_main_kernel.hpp"

namespace gla {

template <int DV_, bool PP_>
struct WideTraits {
  static constexpr int DV = DV_;
  static constexpr bool PP = PP_;               // the two groups half a tile apart (see the kernel)
  static constexpr int TT = 64;                 // tokens per tile
  static constexpr int NST = DV == 256 ? 3 : 2; // ring stages
  static constexpr int E = DV / 128;            // waves a slab's output dims are spread over
  static constexpr int NSG = 4 / E;             // 32-row slabs per group of four waves
  static constexpr int NSL = 2 * NSG;           // slabs per workgroup
  static constexpr int kRows = 32 * NSL;
  static constexpr int ROWB = DV * 2;
  static constexpr int kStateBytes = TT * ROWB, kRopeBytes = TT * 128;
  static constexpr int kStageBytes = kStateBytes + kRopeBytes;
  static constexpr int kSlabP = TT * 64;        // bytes of a slab's weights of one tile
  static constexpr bool kLoRegion = PP;         // rounding residuals have an LDS region of their own
  static constexpr int OFF_P = NST * kStageBytes;
  static constexpr int OFF_LO = OFF_P + NSL * kSlabP;
  static constexpr int OFF_MREF = OFF_LO + (kLoRegion ? NSL * kSlabP : 0);  // [slab][token half][row]: references
  static constexpr int OFF_FLAG = OFF_MREF + NSL * 64 * 4;                  // one word per wave
  static constexpr int OFF_WIN = OFF_FLAG + 64;                             // page ids: two windows of 64 per wave
  static constexpr int kSmem = OFF_WIN + 8 * 2 * 256;
  // partials as the four-wave kernel leaves them: the same block order, a log-sum-exp for every second wave
  static constexpr size_t kSlotFloats = (size_t)kRows * DV + 32 * 4;
  static_assert(DV == 256 || DV == 512, "state dims");
  static_assert(!PP || NST == 3, "half a tile apart a tile is in use for three half-steps: two stages are too few");
  static_assert(kSmem <= 160 * 1024, "LDS capacity");
};

// 16-byte-chunk swizzle of the state rows: as swz16, but with the two upper token bits mixed so that the score
// reads are conflict-free here too.  A 16-byte LDS read serves its lanes in groups {0-3, 12-15, 20-23, 24-27}, ...:
// with 16-row operands such a group holds tokens 0-3, 12-15 at one chunk and tokens 4-11 at the next, so the
// keys of either set must be closed under a change of the lowest bit (with swz16 every read took twice as long).
__host__ __device__ constexpr int swzw(int t) { return ((t & 3) << 2) | ((((t >> 2) ^ (t >> 3)) & 1) << 1) | ((t >> 2) & 1); }

__device__ __forceinline__ void lds_write_b64(unsigned addr, u32x2_t v) {
  asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
// LDS accesses of the rare paths, as assembly too: in front of an LDS access of its own the compiler waits for
// every tile load in flight.
__device__ __forceinline__ float lds_read_f32_sync(unsigned addr) {
  float v;
  asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr) : "memory");
  return v;
}
__device__ __forceinline__ void lds_write_f32(unsigned addr, float v) {
  asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
// A copy the compiler cannot see through: what is derived from it is worked out where it is used (rare paths,
// the ends of a segment) and not kept in registers, or spilled, across the tile loop.
__device__ __forceinline__ int here(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ void lds_write_b32(unsigned addr, uint32_t v) {
  asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory");
}

__device__ __forceinline__ void lds_wait_b32(uint32_t& x) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(x)); }
// sum + a.lo + a.hi for a pair of bf16 (exact products with one, fp32 sums)
__device__ __forceinline__ float add_pk_bf16(float sum, uint32_t a) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, 0x3f803f80u), sum, false);
}
__device__ __forceinline__ float max3_f32(float a, float b, float c) {
  float r;  // (fmaxf() first canonicalises operands that come out of an MFMA)
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
template <int OFF>
__device__ __forceinline__ void lds_read_b32(uint32_t& dst, unsigned addr) {
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}

// PM 0: pages of 8 tokens or more (the eight token rows a wave fetches lie in one page),
// PM 1: pages of 4, 2 or 1 tokens (one address per lane and row).
template <int DV, bool PP, int PM, bool STREAM>
__global__ __launch_bounds__(512) void wide_main_kernel(DevParams p) {
  using TT = WideTraits<DV, PP>;
  constexpr int TOK = TT::TT, NST = TT::NST, NSG = TT::NSG, NSL = TT::NSL, ROWB = TT::ROWB;
  constexpr int NRB = NSG;              // 16-row blocks of a wave's scores
  constexpr int NTB = TOK / 32;         // 16-token blocks of a wave's scores (half the tile)
  constexpr int NKN = DV / 32, NK = NKN + 2;  // contraction steps: state, + RoPE
  constexpr int NSTEP = TOK / 16;       // contraction steps of the value product
  constexpr int SLW = 8 * ROWB / 1024;  // state loads per wave and tile (eight token rows)
  constexpr int LPW = SLW + 1;          // ... plus one of RoPE keys
  __shared__ __attribute__((aligned(1024))) unsigned char smem[TT::kSmem];
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int grp = wave >> 2, g4 = wave & 3;
  const int r16 = lane & 15, q = lane >> 4;      // score layout: row r16 (+ 16 per block), tokens 4q .. 4q + 3
  const int hi = lane >> 5;                      // value layout: row lane % 32
  const int th = g4 & 1;                         // token half of this wave's scores
  const int sslab = grp * NSG + (NSG == 2 ? g4 >> 1 : 0), srow0 = NSG == 2 ? 0 : 16 * (g4 >> 1);
  const int pslab = grp * NSG + (NSG == 2 ? g4 >> 1 : 0), pe = NSG == 2 ? (g4 & 1) : g4;  // value side: slab, 128-dim part

  const int rows_group = p.g_q * p.T;
  const int MB = p.mb, UPB = p.upb, n_chunks = p.num_chunks;
  int chunk_id, mb_wg;  // (placement on the XCDs: see tuned_main_kernel)
  if (p.xcd_map) {
    const int xcd = (int)blockIdx.x & 7, n = (int)blockIdx.x >> 3;
    const int qd = (int)fast_div((unsigned)n, p.fd_mb);
    mb_wg = n - qd * MB;
    chunk_id = xcd * (n_chunks >> 3) + qd;
  } else {
    chunk_id = (int)fast_div(blockIdx.x, p.fd_mb);
    mb_wg = (int)blockIdx.x - chunk_id * MB;
  }

  // ---- this workgroup's chunk of the flat tile list
  const int L_first = lane < p.B ? load_i32_sync(p.seq_lens + lane) : 0;
  if (p.wide_tiles > 0 &&  // (counted as the four-wave kernel counts them: one of the two runs)
      total_tiles<kTok>(p, UPB, lane, wave_incl_scan(tiles_of<kTok>(L_first) * UPB)) < p.wide_tiles)
    return;
  const ListCut cut = cut_list<TOK, 0>(p, UPB, lane, L_first, MB);
  if (cut.tiles <= 0) return;
  const ChunkSpan span0 = locate_chunk<TOK>(p, UPB, cut, chunk_id, lane, L_first);
  const int n_tiles = span0.n_tiles;
  if (n_tiles <= 0) return;
  TileCursor cur = span0.cur;
  int unit_at = span0.at;  // list position of the unit's first tile

  auto next_unit = [&](TileCursor& c) {
    c.j = 0;
    if (++c.ub < UPB) return;
    c.ub = 0;
    do {
      ++c.b;
      c.L = c.b >= p.B ? 0 : c.b < 64 ? __builtin_amdgcn_readlane(L_first, c.b) : uniform(load_i32_sync(p.seq_lens + c.b));
      c.tiles_b = tiles_of<TOK>(c.L);
    } while (c.b < p.B && c.tiles_b == 0);
  };

  // ---- page ids: every wave keeps the ids of its own eight token rows for the next tiles in LDS, in two
  //      windows (the one in use and the one after it, requested when the first is entered; a window never
  //      crosses a unit).  PM 0: one id per tile, 64 tiles per window; PM 1: one per token, 8 tiles.
  constexpr int W = PM == 0 ? 64 : 8;
  const int lgP = p.lg_page;
  const unsigned pmask = (1u << lgP) - 1;
  unsigned char* const win_w = smem + TT::OFF_WIN + wave * 512;
  const unsigned win_addr = lds_base + TT::OFF_WIN + wave * 512;
  auto req_window = [&](int slot, const TileCursor& c) {
    const int tok = PM == 0 ? (c.j + lane) * TOK + 8 * wave : (c.j + (lane >> 3)) * TOK + 8 * wave + (lane & 7);
    const int e = min(tok >> lgP, (c.L - 1) >> lgP);  // (past the end: the last page the sequence holds)
    const int32_t* src = p.page_table + (int64_t)c.b * p.max_pages + e;
    __builtin_amdgcn_global_load_lds((global_cvoid_t*)src, (lds_void_t*)(win_w + slot * 256), 4, 0, 0);
  };
  TileCursor pre = cur, nw = cur;  // tile to fetch next; start of the next window
  int pre_left = n_tiles;          // tiles of the chunk not yet requested
  int win_sel = 0, win_j0 = pre.j, win_left = min(W, pre.tiles_b - pre.j);
  int round = 0, win_round = 0;    // tile steps done; the step in which the next window was requested
  auto step_window = [&]() {       // move nw past the window in use, request the window there
    nw.j = pre.j + win_left;
    if (nw.j >= nw.tiles_b) next_unit(nw);
    if (pre_left > win_left) req_window(win_sel ^ 1, nw);
    win_round = round;
  };
  // PM 0: the window in use is held in a register, one tile per lane, so that a tile's page id is a lane read
  int win_ids = 0;
  auto open_window = [&]() {
    if constexpr (PM == 0) {
      uint32_t id;
      lds_read_b32<0>(id, win_addr + (unsigned)(win_sel * 256 + here(lane) * 4));
      lds_wait_b32(id);
      win_ids = (int)id;
    }
  };
  req_window(0, pre);
  wait_vmcnt<0>();
  open_window();
  step_window();

  // ---- tile loads: this wave moves token rows 8 * wave .. + 7 of the state and of the RoPE tile, 16 bytes per
  //      lane; the LDS side is linear in the lane, each lane fetches the chunk whose swizzled home is its slot
  constexpr int RPL = 1024 / ROWB, CPR = ROWB / 16;
  const int s_rl = lane / CPR, s_pc = lane % CPR;
  const unsigned s_lane = (unsigned)(s_rl * ROWB + ((s_pc & ~15) << 4) + (((s_pc & 15) ^ swzw(s_rl) ^ swzw(8 * wave)) << 4));
  const int r_rl = lane >> 3, r_pc = lane & 7;
  const unsigned rrb = (unsigned)p.d_r * 2u, cpg = (unsigned)p.d_r >> 3;
  unsigned r_voff;  // (RoPE keys of fewer than 64 dims: missing chunks are fetched as duplicates, see tuned_main_kernel)
  {
    const unsigned ch = (unsigned)(r_pc ^ (r_rl >> 1) ^ ((wave & 1) << 2));
    r_voff = (PM == 0 ? (unsigned)r_rl * rrb : 0u) + ((ch >= cpg ? ch - cpg : ch) << 4);
  }
  const uint32_t st_page_bytes = (uint32_t)p.st_s[0] * 2u, st_group_bytes = (uint32_t)p.st_s[1] * 2u;
  const uint32_t rp_page_bytes = (uint32_t)p.rp_s[0] * 2u;
  const unsigned char* const state_b = (const unsigned char*)p.state;
  const unsigned char* const rope_b = (const unsigned char*)p.rope;
  constexpr int kAux = STREAM ? 2 : 0;  // (streaming hint: see tuned_main_kernel)
  int st_load = 0;                      // stage the next tile goes to
  // The next tile is prepared (page id, addresses) and its loads requested: in one burst where the other group
  // has MFMAs to run meanwhile (PP), else one by one between the MFMAs of the scores, since all waves would hold
  // still together in front of the memory pipe.
  const unsigned char *ld_s = nullptr, *ld_r = nullptr;
  unsigned char *ld_ds = nullptr, *ld_dr = nullptr;
  unsigned ld_widx = 0;
  // Once the whole chunk has been requested the last tile's addresses are kept: the loads then fetch lines that
  // are still in L2 into a stage nobody reads, and the tile loop has no branches around them.
  uint64_t ld_goff = 0;
  auto prepare_tile = [&]() {
    ld_ds = smem + st_load * TT::kStageBytes + wave * (8 * ROWB);
    ld_dr = smem + st_load * TT::kStageBytes + TT::kStateBytes + wave * 1024;
    st_load = st_load == NST - 1 ? 0 : st_load + 1;
    if (__builtin_expect(pre_left <= 0, 0)) return;
    if (__builtin_expect(win_left == 0, 0)) {
      if (win_round == round) wait_vmcnt<0>();  // (else covered by the wait that ended the last step)
      win_sel ^= 1;
      pre = nw;
      win_j0 = pre.j;
      win_left = min(W, pre.tiles_b - pre.j);
      open_window();
      step_window();
    }
    if constexpr (PM != 0) ld_widx = win_addr + (unsigned)(win_sel * 256 + (pre.j - win_j0) * 32);
    ld_goff = (uint64_t)pre.ub * st_group_bytes;
    if constexpr (PM == 0) {
      const uint32_t page = (uint32_t)__builtin_amdgcn_readlane(win_ids, pre.j - win_j0);
      const unsigned tip = ((unsigned)pre.j * TOK + 8u * (unsigned)wave) & pmask;  // first token row inside its page
      ld_s = state_b + ((uint64_t)page * st_page_bytes + ld_goff + (uint64_t)tip * ROWB);
      ld_r = rope_b + ((uint64_t)page * rp_page_bytes + (uint64_t)tip * rrb);
    }
    ++pre.j;
    --win_left;
    --pre_left;
  };
  auto load_piece = [&](auto ic) {  // load i of LPW, the RoPE keys last
    constexpr int i = decltype(ic)::value;
    if constexpr (i < SLW) {
      const unsigned off = s_lane ^ ((unsigned)swzw(i * RPL) << 4);
      if constexpr (PM == 0) {
        __builtin_amdgcn_global_load_lds((global_cvoid_t*)(ld_s + (i / 4) * 4096 + off), (lds_void_t*)(ld_ds + (i / 4) * 4096), 16,
                                         (i % 4) * 1024, kAux);
      } else {
        uint32_t id;
        lds_read_b32<i * RPL * 4>(id, ld_widx + (unsigned)s_rl * 4u);
        lds_wait_b32(id);
        const unsigned row = (unsigned)(i * RPL + s_rl);
        const unsigned char* src = state_b + ((uint64_t)id * st_page_bytes + ld_goff + ((row & pmask) * ROWB + (off & (ROWB - 1))));
        __builtin_amdgcn_global_load_lds((global_cvoid_t*)src, (lds_void_t*)(ld_ds + i * 1024), 16, 0, kAux);
      }
    } else {
      if constexpr (PM == 0) {
        __builtin_amdgcn_global_load_lds((global_cvoid_t*)(ld_r + r_voff), (lds_void_t*)ld_dr, 16, 0, 0);
      } else {
        uint32_t id;
        lds_read_b32<0>(id, ld_widx + (unsigned)r_rl * 4u);
        lds_wait_b32(id);
        const unsigned char* src = rope_b + ((uint64_t)id * rp_page_bytes + ((unsigned)r_rl & pmask) * rrb + r_voff);
        __builtin_amdgcn_global_load_lds((global_cvoid_t*)src, (lds_void_t*)ld_dr, 16, 0, 0);
      }
    }
  };
  auto issue_tile = [&]() {
    prepare_tile();
    static_for<0, LPW>(load_piece);
  };
  issue_tile();

  // ---- LDS addresses of this lane's operand reads, stage 0
  const unsigned k_addr = lds_base + (unsigned)((th * (TOK / 2) + r16) * ROWB + ((q ^ swzw(r16)) << 4));  // step s of a 256-byte run: ^ (s << 6)
  const unsigned r_addr = lds_base + (unsigned)(TT::kStateBytes + (th * (TOK / 2) + r16) * 128 + ((q ^ swz8(r16)) << 4));  // second step: ^ 64
  const int i16 = lane & 15, tr_r = i16 >> 2, tr_q = i16 & 3, dh = (lane >> 4) & 1;
  const unsigned v_addr = lds_base + (unsigned)((4 * hi + tr_r) * ROWB + pe * 256 +
                                                (((tr_r << 2) | ((2 * dh + (tr_q >> 1)) ^ (3 * hi))) << 4) + (tr_q & 1) * 8);
  const unsigned p_rd = lds_base + (unsigned)(TT::OFF_P + pslab * TT::kSlabP + lane * 16);
  const unsigned p_wr = lds_base + (unsigned)(TT::OFF_P + sslab * TT::kSlabP + th * (NTB * 1024) +
                                              ((q & 1) * 32 + srow0 + r16) * 16 + (q >> 1) * 8);
  constexpr unsigned kLoDelta = TT::OFF_LO - TT::OFF_P;
  const unsigned flag_mine = lds_base + (unsigned)(TT::OFF_FLAG + wave * 4);
  const unsigned flag_grp = lds_base + (unsigned)(TT::OFF_FLAG + grp * 16);
  const unsigned flag_all = lds_base + (unsigned)TT::OFF_FLAG;
  // reference of entry e = [slab][token half][row]
  auto mref_at = [&](int e) { return lds_base + (unsigned)(TT::OFF_MREF + e * 4); };
  const int srow_u = sslab * 64 + th * 32 + srow0;  // this wave's first entry

  const float sc2 = p.scale * 1.4426950408889634f;
  constexpr float kRebase = 8.f, kLogHeavyShare = -2.f, kNone = -1e30f;

  int k = 0, st_cur = 0;
  while (k < n_tiles) {
    const int seg_n = min(n_tiles - k, cur.tiles_b - cur.j), seg_j0 = cur.j, seg_L = cur.L;
    // ---- query fragments (B operand of the score MFMAs): rows of this wave's score blocks
    u32x4_t qf[NK][NRB];
    int n_vis[NRB];
    const int ln = here(lane), r16 = ln & 15, q = ln >> 4;
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      const int R = (mb_wg * NSL + sslab) * 32 + srow0 + 16 * rb + r16;
      const bool ok = R < rows_group;
      const int Rc = ok ? R : rows_group - 1;
      const int t = (int)fast_div((unsigned)Rc, p.fd_gq);
      const int h = cur.ub * p.g_q + (Rc - t * p.g_q);
      const uint16_t* qn = p.q_nope + cur.b * p.qn_s[0] + t * p.qn_s[1] + h * p.qn_s[2] + 8 * q;
      const uint16_t* qr = p.q_rope + cur.b * p.qr_s[0] + t * p.qr_s[1] + h * p.qr_s[2];
#pragma unroll
      for (int ks = 0; ks < NKN; ++ks) qf[ks][rb] = *(const u32x4_t*)(qn + 32 * ks);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int d = 32 * ks + 8 * q;
        qf[NKN + ks][rb] = d < p.d_r ? *(const u32x4_t*)(qr + d) : u32x4_t{0, 0, 0, 0};
      }
      // visible keys; padding rows are left unmasked (never stored)
      n_vis[rb] = ok ? (p.causal ? cur.L - p.T + 1 + t : cur.L) : 0x7fffffff;
    }
    const int n_vis_min = __builtin_amdgcn_readlane(n_vis[0], 0);
    f32x16_t o[4];
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[d][i] = 0.f;
    float m_o = kNone, m_ref[NRB], l_run[NRB], r_run[NRB], lim[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      m_ref[rb] = kNone;
      l_run[rb] = r_run[rb] = 0.f;
      lim[rb] = -INFINITY;
    }
    uint32_t flag = 0;
    bool flag_set = true;    // the flag in LDS is not zero, or not known to be
    // (the other tiles of the ring behind the first queries: the first step waits for one tile only)
    const bool first = k == 0;
    if (first) {
#pragma unroll
      for (int s = 0; s < NST - 2; ++s) issue_tile();
    }
    // (a use of the queries that cannot move into the loop, where the compiler would wait for every tile load)
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) pin_arch(qf[ks][rb]);
    if (q == 0) {
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        lds_write_f32(mref_at(srow_u + r16 + 16 * rb), kNone);
      }
    }
    // (later segments: the tile had landed at the end of the step before)
    if (first) wait_vmcnt<LPW * (NST - 2)>();
    lds_barrier();  // the first tile is in LDS, and nobody reads the row sums of the segment before any more
    if (PP && grp == 1) lds_barrier();

    for (int i = 0; i < seg_n; ++i) {
      const int tok0 = (seg_j0 + i) * TOK;
      const unsigned st_off = (unsigned)(st_cur * TT::kStageBytes);
      // ================= scores and weights
      if constexpr (!PP) prepare_tile();
      if constexpr (PP) __builtin_amdgcn_s_setprio(1);  // (the longer of the two half-steps)
      // value rows at or past the end of the sequence may hold anything: zero them (0 x NaN must not leak)
      if (__builtin_expect((PP ? grp == 0 : true) && tok0 + TOK > seg_L, 0)) {
        constexpr int kThr = PP ? 256 : 512;
        const u32x4_t z = {0, 0, 0, 0};
        for (int off = (seg_L - tok0) * ROWB + (tid & (kThr - 1)) * 16; off < TT::kStateBytes; off += kThr * 16)
          lds_write_b128<0>(lds_base + st_off + (unsigned)off, z);
      }
      f32x4_t s[NTB][NRB];
      {
        constexpr int D = PP ? 3 : 4;  // steps of operand reads in flight
        u32x4_t kf[D][NTB];
        const unsigned ka = k_addr + st_off, ra = r_addr + st_off;
        auto rd = [&](auto kc) {
          constexpr int ks = decltype(kc)::value;
          static_for<0, NTB>([&](auto tc) {
            constexpr int tb = decltype(tc)::value;
            if constexpr (ks < NKN) lds_read_b128<tb * 16 * ROWB + (ks >> 2) * 256>(kf[ks % D][tb], ka ^ (unsigned)((ks & 3) << 6));
            else lds_read_b128<tb * 16 * 128>(kf[ks % D][tb], ra ^ (unsigned)((ks - NKN) << 6));
          });
        };
        static_for<0, D>(rd);
        static_for<0, NK>([&](auto kc) {
          constexpr int ks = decltype(kc)::value;
          constexpr int ahead = (NK - 1 - ks < D - 1 ? NK - 1 - ks : D - 1) * NTB;
          static_for<0, NTB>([&](auto tc) { pin_arch(kf[ks % D][decltype(tc)::value]); });
          lds_wait<ahead>(kf[ks % D][0]);
          static_for<0, NTB>([&](auto tc) { pin_arch(kf[ks % D][decltype(tc)::value]); });
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb)
              s[tb][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8_t, kf[ks % D][tb]), __builtin_bit_cast(bf16x8_t, qf[ks][rb]),
                  ks == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : s[tb][rb], 0, 0, 0);
          if constexpr (ks + D < NK) rd(std::integral_constant<int, ks + D>{});
          if constexpr (!PP) static_for<(ks * LPW) / NK, ((ks + 1) * LPW) / NK>(load_piece);
          __builtin_amdgcn_sched_barrier(0);
        });
      }
      // The scores are read by assembly below (max3_f32): the compiler does not count an MFMA's wait states in front
      // of a read that it does not see as an instruction.
      asm volatile("s_nop 15" : "+v"(s[0][0]));
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) pin_arch(s[tb][rb]);
      if (__builtin_expect(tok0 + TOK > n_vis_min, 0)) {  // mask by select (last tiles only)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              s[tb][rb][e] = tok0 + th * (TOK / 2) + 16 * tb + 4 * q + e < n_vis[rb] ? s[tb][rb][e] : -INFINITY;
      }
      // One test per tile, on the row maxima: has a row left its reference (by more than 2^8), or does a weight
      // hold more than a quarter of its row's running sum?  lim, in the same units as the scaled scores, is the
      // smaller of the two limits.  The running sum is that of the tiles before and of this wave's token half alone:
      // never too large, so the test errs on the safe side (and depends on nothing another wave does meanwhile).
      float mx[NRB];
      bool odd = false;
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        const float m = max3_f32(max3_f32(s[0][rb][0], s[0][rb][1], s[0][rb][2]), s[0][rb][3], s[1][rb][0]);
        mx[rb] = max3_f32(max3_f32(s[1][rb][1], s[1][rb][2], s[1][rb][3]), m, m) * sc2;
        static_assert(NTB == 2, "two token blocks");
        odd = odd || mx[rb] > lim[rb];
      }
      bool heavy = false;
      if (__builtin_expect(__ballot(odd) != 0, 0)) {
        flag = 0;
        odd = false;
        const int l2 = here(lane), e0 = srow_u + (l2 & 15);
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
          float m = mx[rb];
          m = fmaxf(m, __shfl_xor(m, 16, 64));
          m = fmaxf(m, __shfl_xor(m, 32, 64));
          const float m_new = m > m_ref[rb] + kRebase ? ceilf(m) : m_ref[rb];
          odd = odd || m_new != m_ref[rb];
          const float alpha = __builtin_amdgcn_exp2f(m_ref[rb] - m_new);
          l_run[rb] *= alpha;
          r_run[rb] *= alpha;
          m_ref[rb] = m_new;
          float l = l_run[rb];
          l += __shfl_xor(l, 16, 64);
          l += __shfl_xor(l, 32, 64);
          if (l2 < 16) lds_write_f32(mref_at(e0 + 16 * rb), m_new);
          // (no key yet: log2 0 = -inf, every weight is heavy)
          const float thr = __builtin_amdgcn_logf(l) + kLogHeavyShare;
          heavy = heavy || m > m_new + thr;
          lim[rb] = m_new + fminf(thr, kRebase);
        }
        if (__ballot(odd) != 0) flag = 1;
        heavy = __ballot(heavy) != 0;
        if (heavy) flag |= 2;
        flag_set = true;
      }
      uint32_t pk[NTB][NRB][2], lo[NTB][NRB][2];
      float pw[NTB][NRB][4];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        float ls = 0.f, rs = 0.f;
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            pw[tb][rb][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[tb][rb][e], sc2, -m_ref[rb]));
            ls += pw[tb][rb][e];
          }
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            pk[tb][rb][e] = cvt_pk_bf16(pw[tb][rb][2 * e], pw[tb][rb][2 * e + 1]);
            rs = add_pk_bf16(rs, pk[tb][rb][e]);
          }
        }
        l_run[rb] += ls;
        r_run[rb] += rs;
        pin_arch(l_run[rb]);  // (here, not behind the barrier)
      }
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
          lds_write_b64(p_wr + (unsigned)(tb * 1024 + rb * 256), u32x2_t{pk[tb][rb][0], pk[tb][rb][1]});
      // Heavy weights in this tile: it gets a second value pass with the rounding residuals of this wave's
      // weights (why, and at what cost: see tuned_main_kernel).
      if (__builtin_expect(heavy, 0)) {
        {
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                const uint32_t h2 = pk[tb][rb][e];
                lo[tb][rb][e] = cvt_pk_bf16(pw[tb][rb][2 * e] - __builtin_bit_cast(float, h2 << 16),
                                            pw[tb][rb][2 * e + 1] - __builtin_bit_cast(float, h2 & 0xffff0000u));
                r_run[rb] = add_pk_bf16(r_run[rb], lo[tb][rb][e]);
              }
          if constexpr (TT::kLoRegion) {
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
              for (int rb = 0; rb < NRB; ++rb)
                lds_write_b64(p_wr + kLoDelta + (unsigned)(tb * 1024 + rb * 256), u32x2_t{lo[tb][rb][0], lo[tb][rb][1]});
          }
        }
      }
      if constexpr (!TT::kLoRegion) {
        if (!heavy) {
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) lo[tb][rb][0] = lo[tb][rb][1] = 0;
        }
      }
      if (__builtin_expect(flag_set, 0)) {  // (most tiles leave the zero of the tiles before)
        lds_write_b32(flag_mine, flag);
        flag_set = flag != 0;
        flag = 0;
      }
      if constexpr (PP) __builtin_amdgcn_s_setprio(0);
      auto wait_tile = [&]() {  // the next tile has landed (what group 0 has requested in this step may be in flight)
        if constexpr (PP) {
          if (grp == 0) wait_vmcnt<LPW>();  // (the other group requests tiles behind this point of its step)
          else wait_vmcnt<0>();
        } else {
          wait_vmcnt<LPW * (NST - 2)>();
        }
        ++round;
      };
      if (PP && grp == 1) wait_tile();
      lds_barrier();

      // ================= values
      if constexpr (PP) issue_tile();  // (under the other group's score MFMAs; between the value MFMAs it cost 3 % more)
      {
        u32x4_t fl, fl2 = {0, 0, 0, 0}, pf[NSTEP];
        lds_read_b128<0>(fl, TT::kLoRegion ? flag_grp : flag_all);
        if constexpr (!TT::kLoRegion) lds_read_b128<16>(fl2, flag_all);
        static_for<0, NSTEP>([&](auto sc) { lds_read_b128<decltype(sc)::value * 1024>(pf[decltype(sc)::value], p_rd); });
        const unsigned va = v_addr + st_off;
        constexpr int NV = NSTEP * 4, D = 3;
        u32x2_t vl[D], vh[D];
        auto rd = [&](auto ic) {
          constexpr int i2 = decltype(ic)::value, st = i2 / 4, db = i2 % 4;
          lds_read_tr16_b64<st * 16 * ROWB>(vl[i2 % D], va ^ (unsigned)(db << 6));
          lds_read_tr16_b64<st * 16 * ROWB + 8 * ROWB>(vh[i2 % D], va ^ (unsigned)((db << 6) | 32));
        };
        static_for<0, NSTEP>([&](auto sc) { pin_arch(pf[decltype(sc)::value]); });
        // the first value operands travel with flags and weights; all of them have arrived before the branch on the
        // flags (no register may be in flight across code in which the compiler could move it)
        static_for<0, D>(rd);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fl), "+v"(fl2));
        static_for<0, NSTEP>([&](auto sc) { pin_arch(pf[decltype(sc)::value]); });
        static_for<0, D>([&](auto ic) {
          pin_arch(vl[decltype(ic)::value]);
          pin_arch(vh[decltype(ic)::value]);
        });
        const int mine = grp == 0 || TT::kLoRegion ? 0 : 1;
        const uint32_t f_grp = (uint32_t)uniform((int)(mine ? (fl2[0] | fl2[1] | fl2[2] | fl2[3]) : (fl[0] | fl[1] | fl[2] | fl[3])));
        const uint32_t f_all = TT::kLoRegion ? f_grp : (uint32_t)uniform((int)(fl[0] | fl[1] | fl[2] | fl[3] | fl2[0] | fl2[1] | fl2[2] | fl2[3]));
        float sc_w[2] = {1.f, 1.f};  // what the weights of the two token halves are multiplied with
        auto scale_weights = [&](u32x4_t& w, float f) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            w[e] = cvt_pk_bf16(__builtin_bit_cast(float, w[e] << 16) * f, __builtin_bit_cast(float, w[e] & 0xffff0000u) * f);
        };
        if (__builtin_expect((f_grp & 1) != 0, 0)) {
          // a reference has moved: everything to the largest one (exact powers of two)
          const int l2 = here(lane);
          const float a0 = lds_read_f32_sync(mref_at(pslab * 64 + (l2 & 31))), a1 = lds_read_f32_sync(mref_at(pslab * 64 + 32 + (l2 & 31)));
          const float m_new = fmaxf(m_o, fmaxf(a0, a1));
          const float alpha = __builtin_amdgcn_exp2f(m_o - m_new);
          sc_w[0] = __builtin_amdgcn_exp2f(a0 - m_new);
          sc_w[1] = __builtin_amdgcn_exp2f(a1 - m_new);
          m_o = m_new;
#pragma unroll
          for (int d = 0; d < 4; ++d) {
#pragma unroll
            for (int e = 0; e < 16; ++e) o[d][e] *= alpha;
            pin_arch(o[d]);
          }
          static_for<0, NSTEP>([&](auto sc) { scale_weights(pf[decltype(sc)::value], sc_w[decltype(sc)::value * 2 / NSTEP]); pin_arch(pf[decltype(sc)::value]); });
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb) {  // the score side of this wave
            const int row = sslab * 64 + srow0 + 16 * rb + (l2 & 15);
            const float mn = fmaxf(lds_read_f32_sync(mref_at(row)), lds_read_f32_sync(mref_at(row + 32)));
            const float f = __builtin_amdgcn_exp2f(m_ref[rb] - mn);
            if (m_ref[rb] != mn) lim[rb] = -INFINITY;  // (worked out again, and the reference posted, at the next tile)
            l_run[rb] *= f;
            r_run[rb] *= f;
            m_ref[rb] = mn;
          }
        }
        auto value_mfmas = [&]() {
          static_for<0, NV>([&](auto ic) {
            constexpr int i2 = decltype(ic)::value, st = i2 / 4, db = i2 % 4;
            constexpr int ahead = (NV - 1 - i2 < D - 1 ? NV - 1 - i2 : D - 1) * 2;
            pin_arch(vl[i2 % D]);
            lds_wait2<ahead>(vl[i2 % D], vh[i2 % D]);
            const u32x4_t a4 = {vl[i2 % D][0], vl[i2 % D][1], vh[i2 % D][0], vh[i2 % D][1]};
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a4), __builtin_bit_cast(bf16x8_t, pf[st]), o[db], 0, 0, 0);
            if constexpr (i2 + D < NV) rd(std::integral_constant<int, i2 + D>{});
                        __builtin_amdgcn_sched_barrier(0);
          });
        };
        value_mfmas();
        if (__builtin_expect((f_all & 2) != 0, 0)) {
          if constexpr (!TT::kLoRegion) {
            // (all waves are in this phase: the residuals take the place of the weights)
            lds_barrier();
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
              for (int rb = 0; rb < NRB; ++rb)
                lds_write_b64(p_wr + (unsigned)(tb * 1024 + rb * 256), u32x2_t{lo[tb][rb][0], lo[tb][rb][1]});
            lds_barrier();
          }
          static_for<0, NSTEP>([&](auto sc) {
            constexpr int st = decltype(sc)::value;
            lds_read_b128<st * 1024>(pf[st], p_rd + (TT::kLoRegion ? kLoDelta : 0u));
            lds_wait<0>(pf[st]);
            if constexpr (TT::kLoRegion) {
              // (a wave without heavy weights has not written its residuals; a slab's token half is one wave's)
              const uint32_t f_src = (g4 >> 1) == 0 ? fl[st * 2 / NSTEP] : fl[2 + st * 2 / NSTEP];
              if ((uniform((int)f_src) & 2) == 0) pf[st] = u32x4_t{0, 0, 0, 0};
            }
            scale_weights(pf[st], sc_w[st * 2 / NSTEP]);
          });
          static_for<0, D>(rd);
          value_mfmas();
        }
      }
      st_cur = st_cur == NST - 1 ? 0 : st_cur + 1;
      if (!PP || grp == 0) wait_tile();
      else ++round;
      lds_barrier();
    }
    if (PP && grp == 0) lds_barrier();
    k += seg_n;

    // ================= end of segment: row sums meet in LDS, then the unit's result or its partial
    float* const sum_lds = (float*)(smem + TT::OFF_P);  // [slab][token half][row] pairs
    const int le = here(lane), col = le & 31, hi = le >> 5;
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      float l = l_run[rb], r = r_run[rb];
      l += __shfl_xor(l, 16, 64);
      l += __shfl_xor(l, 32, 64);
      r += __shfl_xor(r, 16, 64);
      r += __shfl_xor(r, 32, 64);
      if (le < 16) *(float2*)(sum_lds + 2 * (srow_u + le + 16 * rb)) = make_float2(l, r);
    }
    lds_barrier();
    {
      const float2 s0 = *(const float2*)(sum_lds + 2 * (pslab * 64 + col)), s1 = *(const float2*)(sum_lds + 2 * (pslab * 64 + 32 + col));
      const float l_tot = s0.x + s1.x, r_tot = s0.y + s1.y;
      const float inv = r_tot > 0.f ? 1.0f / r_tot : 0.f;
      const float lse = l_tot > 0.f ? (m_o + log2f(l_tot)) * 0.6931471805599453f : -INFINITY;
      const int R = (mb_wg * NSL + pslab) * 32 + col;
      const bool row_valid = R < rows_group;
      const int Rc = row_valid ? R : rows_group - 1;
      const int t = (int)fast_div((unsigned)Rc, p.fd_gq);
      const int h = cur.ub * p.g_q + (Rc - t * p.g_q);
      const int64_t ob = cur.b * p.out_s[0] + t * p.out_s[1] + h * p.out_s[2];
      const bool complete = seg_j0 == 0 && seg_n == cur.tiles_b;
      // partial: slot 1 if the unit's first tile is in this chunk, slot 0 if it began earlier
      float* slot = p.ws_out + (((size_t)chunk_id * MB + mb_wg) * 2 + (seg_j0 == 0 ? 1 : 0)) * TT::kSlotFloats;
      if (seg_j0 == 0 && tid == 0) {  // tells the merge kernel which chunks hold this unit
        int2 span;
        span.x = chunk_id;
        span.y = (int)((unsigned)(unit_at + cur.tiles_b - 1) / (unsigned)cut.chunk);
        ((int2*)p.ws_lse)[(cur.b * UPB + cur.ub) * MB + mb_wg] = span;
      }
      if (hi == 0 && (pe & 1) == 0) {
        if (!complete) slot[(size_t)TT::kRows * DV + (wave >> 1) * 32 + col] = lse;
        else if (row_valid && pe == 0) p.lse[((int64_t)cur.b * p.T + t) * p.h_q + h] = lse;
      }
      // (one loop per kind of result, as in the four-wave kernel)
      auto quarter = [&](int d, int q4) { return f32x4_t{o[d][4 * q4] * inv, o[d][4 * q4 + 1] * inv, o[d][4 * q4 + 2] * inv, o[d][4 * q4 + 3] * inv}; };
      if (!complete) {
        float* const dst = slot + (size_t)(wave * 16) * 256 + le * 4;
        if (row_valid) {
#pragma unroll
          for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) *(f32x4_t*)(dst + (d * 4 + q4) * 256) = quarter(d, q4);
        }
      } else if (p.out_fp32) {
        float* const dst = (float*)p.out + ob + pe * 128 + 4 * hi;
        if (row_valid) {
#pragma unroll
          for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) *(f32x4_t*)(dst + 32 * d + 8 * q4) = quarter(d, q4);
        }
      } else {
        uint16_t* const dst = (uint16_t*)p.out + ob + pe * 128 + 8 * hi;
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
          for (int q8 = 0; q8 < 2; ++q8) {
            const u32x4_t v = join_halves_bf16(quarter(d, 2 * q8), quarter(d, 2 * q8 + 1));
            if (row_valid) store_b128_align8(dst + 32 * d + 16 * q8, v);
          }
      }
    }
    unit_at += cur.tiles_b + cut.setup;
    next_unit(cur);
  }
  wait_vmcnt<0>();  // (tiles fetched again past the end of the chunk: let them land before the wave leaves)
}

}  // namespace gla
