// Generic decode-attention kernel on bf16 MFMA: any page size, any strides and any dims in steps of eight (sixteen
// for the value), as long as rows of cache, query and output are 16-byte aligned; what is not aligned stays with the
// scalar kernel (generic_kernels.hpp).  Same operation, same partials, same merge, and the same precision: products
// of bf16 are exact in fp32, and each fp32 softmax weight enters the value product as a sum of three bf16 (24
// significant bits, three MFMAs), never rounded to 16 bits.
//
// One workgroup takes one (sequence, group, block of 16 * WR query rows, range of tokens).  WS waves share a slab of 16
// rows: of each tile of 32 * WS tokens every one takes 32, with a softmax of its own, and they meet in LDS at the end
// (transposed form, S^T = K . Q^T and O^T += V^T . P^T, on 16x16x32 MFMAs; row statistics in the four lanes of a
// row).  Tiles lie in a ring of two to four stages, filled by direct-to-LDS loads.  A cache row lies in LDS as its 16-byte
// chunks [value | RoPE key] or [value | key], in rows of an odd number of chunks, so that reads of one column
// spread over the banks and an operand's address is the lane's own plus a constant.  The ids of 64 or 128 consecutive pages sit in the lanes of one or two registers.
//
// Bound by latency and vector work (address arithmetic with run-time dims, the three-way split).  Two latent heads of
// 256 dims, 128 heads, 9 sequences of up to 4500 tokens at 128 tokens per page: 38.0 us per call with one wave per slab and
// two stages, 30.8 with two and three, 29.1 with rows of an odd number of chunks besides (rotated by the row number
// before: five instructions more per operand read); 1923 with the scalar kernel, whose waves each read the whole cache
// for one row.  At two query positions, 2 sequences 32.8 -> 22.7 -> 21.2; one latent head of 512 dims, 4 sequences 56.3 ->
// 39.1 -> 37.6; four tied states of 128, 20 short sequences 35.9 -> 19.1 -> 18.2.
#pragma once

#include "common.hpp"
#include "generic_kernels.hpp"
#include "tuned_device.hpp"

namespace gla {

// Tokens per range, for every sequence the same: the caller's, else the batch's longest sequence in ranges of at least
// 256 tokens (a partial costs as much as a few tiles: 18 units of up to 4500 tokens take 39 us in 17 ranges, 46 in 28),
// of at least 64 while the grid is small (2 units of 256 tokens: 19 us in four ranges, 49 in one).  In no more ranges than
// run side by side, if they would fill a second round less than the first (one_round, launch_generic_mfma) and the sequences
// are so much alike that they would run in two: GLA-2 32 x 3000 tokens 70 -> 65 us, MLA shape 16 x 4000 125 -> 104.  By the lengths
// and not by the page table's row length, which is all the host knows: in a table for the longest context every sequence
// would lie in its first range (nine sequences of up to 4500 tokens, table for 72000: 213 us, 41 this way).
// (len: the length of sequence `lane`, loaded ahead; per_seq: workgroups per sequence and range)
__device__ __forceinline__ int range_tokens(const DevParams& p, int lane, int len, int per_seq) {
  if (p.split_tokens > 0) return p.split_tokens;
  int longest = len;
  for (int i = lane + 64; i < p.B; i += 64) longest = max(longest, p.seq_lens[i]);
  longest = wave_max(max(longest, 1));
  int n = max(1, min(p.splits, max((longest + 255) >> 8, min((longest + 63) >> 6, longest <= 4096 ? p.small_ranges : p.small_ranges_longer))));
  if (n > p.one_round) {
    const float inv = (float)n / (float)longest;
    float held = ceilf((float)max(len, 0) * inv);  // ranges that hold tokens
    for (int i = lane + 64; i < p.B; i += 64) held += ceilf((float)max(p.seq_lens[i], 0) * inv);
    if (wave_sum(held) * (float)per_seq > (float)p.resident) n = p.one_round;
  }
  return ((longest + n - 1) / n + 31) & ~31;
}

// At most N of this wave's loads still in flight, N known at run time only (the next lower count that has an instruction
// here: waiting for more than needed is always right).
__device__ __forceinline__ void wait_vmcnt_at_most(int n) {
  if (n >= 24) wait_vmcnt<24>();
  else if (n >= 16) wait_vmcnt<16>();
  else if (n >= 12) wait_vmcnt<12>();
  else if (n >= 10) wait_vmcnt<10>();
  else if (n >= 8) wait_vmcnt<8>();
  else if (n >= 6) wait_vmcnt<6>();
  else if (n >= 5) wait_vmcnt<5>();
  else if (n >= 4) wait_vmcnt<4>();
  else if (n >= 3) wait_vmcnt<3>();
  else if (n >= 2) wait_vmcnt<2>();
  else if (n >= 1) wait_vmcnt<1>();
  else wait_vmcnt<0>();
}

// Waves that share a 16-row slab (each takes every WS-th 32 tokens of a tile), at most: as many as registers allow (512
// dims: a wave needs more than 256) and two ring stages leave room for.  Rows of up to dvb dims, RoPE keys of up to 128.
constexpr int generic_chunks(int dvb, bool sepk) { return (sepk ? 2 * dvb / 8 : (dvb + 128) / 8) | 1; }  // 16-byte chunks per row in LDS
constexpr int generic_max_waves(int dvb) { return dvb > 256 ? 4 : 8; }
constexpr int generic_ws(int dvb, int wr, bool sepk) {
  const int block = 32 * generic_chunks(dvb, sepk) * 16;  // 32 tokens
  return wr * 4 <= generic_max_waves(dvb) && block * 8 <= 160 * 1024 ? 4 : wr * 2 <= generic_max_waves(dvb) && block * 4 <= 160 * 1024 ? 2 : 1;
}
// LDS where the waves of a slab meet
constexpr int generic_meet_bytes(int dvb, int wr, int ws) { return wr * (ws - 1) * 64 * (dvb + 8); }

template <int DVB, int WR, int WS, bool SEPK>
__global__ __launch_bounds__(64 * WR * WS) void generic_mfma_kernel(DevParams p) {
  static_assert(2 * WS * 32 * generic_chunks(DVB, SEPK) * 16 <= 160 * 1024 && generic_meet_bytes(DVB, WR, WS) <= 160 * 1024, "LDS capacity");
  constexpr int NW = WR * WS, STEP = 32 * WS;
  constexpr int NDB = DVB / 16, NKN = DVB / 32, NKR = SEPK ? 0 : 4;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];  // (ring, then where the waves of a slab meet)
  const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6);
  const int r16 = lane & 15, q = lane >> 4;

  const int rows_group = p.g_q * p.T;
  const int blocks = (rows_group + 16 * WR - 1) / (16 * WR);
  const int unit = (int)blockIdx.x / blocks, rb = (int)blockIdx.x - unit * blocks;
  const int b = unit / p.h_c, g = unit - b * p.h_c;
  const int split = blockIdx.y;
  const int slab = wave % WR, ws = wave / WR;  // this wave's rows, and its share of a tile's tokens
  const int R = (rb * WR + slab) * 16 + r16;
  const bool row_valid = R < rows_group;
  const int Rc = row_valid ? R : rows_group - 1;
  const int t = Rc / p.g_q, h = g * p.g_q + (Rc - t * p.g_q);
  const int row = (b * p.T + t) * p.h_q + h;

  const int L = p.seq_lens[b], len_lane = lane < p.B ? p.seq_lens[lane] : 0;
  const int n_vis = p.causal ? L - p.T + 1 + t : L;  // visible keys of this lane's row

  // ---- chunks of a cache row in LDS: value first, then RoPE key or key
  const int cv = p.d_v >> 3, ck = p.d_n >> 3, cr = p.d_r >> 3;
  const int cpr = cv + (SEPK ? ck : cr);
  // (an odd number of chunks per row: the rows at one chunk spread over the banks, and every operand address is the lane's
  // own plus a constant)
  const int pitch = (cpr | 1) * 16;
  const int tile_bytes = STEP * pitch;
  const int nst = p.ring_stages;  // (two at least)

  // ---- queries (B operand): dims beyond the real ones are zero, whatever the key operand holds there
  u32x4_t qn[NKN], qr[NKR > 0 ? NKR : 1];
  {
    const uint16_t* src = p.q_nope + b * p.qn_s[0] + t * p.qn_s[1] + h * p.qn_s[2];
#pragma unroll
    for (int ks = 0; ks < NKN; ++ks) qn[ks] = 4 * ks + q < ck ? *(const u32x4_t*)(src + (4 * ks + q) * 8) : u32x4_t{0, 0, 0, 0};
    if constexpr (!SEPK) {
      const uint16_t* srcr = p.q_rope + b * p.qr_s[0] + t * p.qr_s[1] + h * p.qr_s[2];
#pragma unroll
      for (int ks = 0; ks < NKR; ++ks) qr[ks] = 4 * ks + q < cr ? *(const u32x4_t*)(srcr + (4 * ks + q) * 8) : u32x4_t{0, 0, 0, 0};
    }
  }
  // ---- this range (behind the loads of the queries, which need no lengths)
  const int span = p.splits == 1 ? 1 << 30 : range_tokens(p, lane, len_lane, p.h_c * blocks);
  const int j_begin = (int)min((int64_t)split * span, (int64_t)max(L, 0));
  const int j_end = (int)min((int64_t)j_begin + span, (int64_t)max(L, 0));
  if (p.splits > 1 && j_begin >= j_end) {  // nothing here: the merge needs no values
    if (q == 0 && row_valid) p.ws_lse[(int64_t)split * p.B * p.T * p.h_q + row] = -INFINITY;
    return;
  }

  f32x4_t o[NDB];
#pragma unroll
  for (int d = 0; d < NDB; ++d) o[d] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const float sc2 = p.scale * 1.4426950408889634f;

  // ---- tile loads.  The ids of 64 consecutive pages (128 where a tile can span as many) sit in the lanes of a register
  //      and are fetched again when a tile leaves them (rows past the end of the sequence repeat its last token: valid
  //      memory, masked and zeroed below).  The load is complete where it stands: it waits for the tiles in flight, which
  //      costs pages of one token the depth of the ring.
  constexpr int NWIN = STEP > 64 ? 2 : 1;
  int win0 = 0, win1 = 0, win_page = -0x40000000;
  //      Of the last tile of a range only the 32-token blocks are fetched that hold tokens of it.
  auto tile_rows = [&](int tok0) { return min(STEP, (j_end - tok0 + 31) & ~31); };
  auto loads_of = [&](int rows) { return uniform((((rows * (cpr | 1) + 63) >> 6) - wave + NW - 1) / NW); };  // this wave's load instructions
  const int n_mine = loads_of(STEP);
  auto load_tile = [&](int tok0, int stage) {
    const int rows = tile_rows(tok0), n_slots = rows * (cpr | 1), n_inst = (n_slots + 63) >> 6;
    const int first_page = (int)fast_div((unsigned)tok0, p.fd_page), last_page = (int)fast_div((unsigned)min(tok0 + rows - 1, L - 1), p.fd_page);
    if (uniform(last_page) >= uniform(win_page) + 64 * NWIN) {
      win_page = first_page;
      const int held = (int)fast_div((unsigned)(L - 1), p.fd_page);
      const int32_t* row = p.page_table + (int64_t)b * p.max_pages;
      win0 = load_i32_sync(row + min(first_page + lane, held));
      if constexpr (NWIN == 2) win1 = load_i32_sync(row + min(first_page + 64 + lane, held));
    }
    for (int i = wave; i < n_inst; i += NW) {
      const int n = i * 64 + lane;
      const int row_i = min((int)fast_div((unsigned)n, p.fd_cpr), STEP - 1);
      const int chunk = min(n - row_i * (cpr | 1), cpr - 1);  // (what pads a row repeats its last chunk)
      const int tok = min(tok0 + row_i, L - 1);
      const int pg = (int)fast_div((unsigned)tok, p.fd_page);
      const int64_t tip = tok - pg * p.P;
      int id = __builtin_amdgcn_ds_bpermute((pg - win_page) << 2, win0);
      if constexpr (NWIN == 2) {
        const int id1 = __builtin_amdgcn_ds_bpermute((pg - win_page) << 2, win1);  // (lane index modulo 64)
        id = pg - win_page >= 64 ? id1 : id;
      }
      const int64_t page = id;
      const uint16_t* src;
      if (chunk < cv) src = p.state + page * p.st_s[0] + g * p.st_s[1] + tip * p.st_s[2] + chunk * 8;
      else if constexpr (SEPK) src = p.kstate + page * p.k_s[0] + g * p.k_s[1] + tip * p.k_s[2] + (chunk - cv) * 8;
      else src = p.rope + page * p.rp_s[0] + tip * p.rp_s[1] + (chunk - cv) * 8;
      if (n < n_slots) __builtin_amdgcn_global_load_lds((global_cvoid_t*)src, (lds_void_t*)(smem + stage * tile_bytes + i * 1024), 16, 0, 0);
    }
  };

  const int row0 = 32 * ws;  // first row of this wave's share of a tile
  const int tr_r = r16 >> 2, tr_c = r16 & 3;
  // operand addresses of this lane in stage 0: key row r16, chunk q of the key (its RoPE part after the value); value row
  // 4 q + tr_r, half a chunk (transposing reads); 16 rows further on the second token block
  const unsigned k_at = lds_base + (unsigned)((row0 + r16) * pitch + ((SEPK ? cv : 0) + q) * 16), r_at = lds_base + (unsigned)((row0 + r16) * pitch + (cv + q) * 16);
  const unsigned v_at = lds_base + (unsigned)((row0 + 4 * q + tr_r) * pitch + tr_c * 8);
  const unsigned block2 = (unsigned)(16 * pitch);

  if (j_begin < j_end) {
    const int n_tiles = (j_end - j_begin + STEP - 1) / STEP;
    for (int t = 0; t < min(nst - 1, n_tiles); ++t) load_tile(j_begin + t * STEP, t);
    const int n_last = loads_of(tile_rows(j_begin + (n_tiles - 1) * STEP));
    int stage = 0;
    for (int tile = 0; tile < n_tiles; ++tile) {
      const int j = j_begin + tile * STEP;
      const int behind = n_tiles - 1 - tile;
      wait_vmcnt_at_most(behind > nst - 2 ? n_mine * (nst - 2) : behind > 0 ? n_mine * (behind - 1) + n_last : 0);  // this wave's part of the tile ...
      lds_barrier();  // ... and everybody's; nobody reads the stage of the tile before any more
      const unsigned off = (unsigned)(stage * tile_bytes);
      const int stage_load = stage == 0 ? nst - 1 : stage - 1;
      stage = stage == nst - 1 ? 0 : stage + 1;
      if (tile + nst - 1 < n_tiles) load_tile(j + (nst - 1) * STEP, stage_load);
      if (j + STEP > L) {  // rows past the end may hold anything: 0 x NaN must not leak (uniform over the workgroup)
        for (int z = (L - j) * pitch + (int)threadIdx.x * 16; z < tile_rows(j) * pitch; z += 64 * NW * 16)
          lds_write_b128<0>(lds_base + off + (unsigned)z, u32x4_t{0, 0, 0, 0});
        lds_barrier();
      }
      if (j + row0 >= j_end) continue;  // (the last tile of a range may end before this wave's share)
      // ---- scores of 2 x 16 tokens: S^T[token 16 tb + 4 q + e][row r16]
      f32x4_t s[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
      // (four steps at a time, their eight reads in flight together; where the key ends inside them, the lanes beyond its
      // dims read its last chunk again, against zeros of the query)
      auto score_steps = [&](auto nc, const auto& qf, unsigned at, int chunks) {
        static_for<0, decltype(nc)::value / 4>([&](auto gc) {
          constexpr int k4 = 4 * decltype(gc)::value;
          auto four = [&](auto back) {  // back(ks): how far this lane's chunk of step ks lies beyond the last one, in bytes
            u32x4_t kf[4][2];
            static_for<0, 4>([&](auto kc) {
              constexpr int ks = decltype(kc)::value;
              lds_read_b128<(k4 + ks) * 64>(kf[ks][0], at - back(kc));
              lds_read_b128<(k4 + ks) * 64>(kf[ks][1], at + block2 - back(kc));
            });
            static_for<0, 4>([&](auto kc) {
              constexpr int ks = decltype(kc)::value;
              pin_arch(kf[ks][0]);
              lds_wait<2 * (3 - ks)>(kf[ks][1]);
              pin_arch(kf[ks][0]);
              static_for<0, 2>([&](auto tc) {
                constexpr int tb = decltype(tc)::value;
                s[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kf[ks][tb]), __builtin_bit_cast(bf16x8_t, qf[k4 + ks]), s[tb], 0, 0, 0);
              });
            });
          };
          const int n = chunks - 4 * k4;  // chunks from these steps on
          if (n >= 16) four([&](auto) { return 0u; });
          else if (n > 0) four([&](auto kc) { return (unsigned)(16 * max(0, 4 * decltype(kc)::value + q + 1 - n)); });
        });
      };
      score_steps(std::integral_constant<int, NKN>{}, qn, k_at + off, ck);
      if constexpr (!SEPK) score_steps(std::integral_constant<int, NKR>{}, qr, r_at + off, cr);
      // ---- online softmax (base 2), masked by select
      float mx = -INFINITY;
      bool visible[8];
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int tok = j + row0 + 16 * tb + 4 * q + e;
          visible[4 * tb + e] = tok < n_vis && tok < j_end;
          mx = fmaxf(mx, visible[4 * tb + e] ? s[tb][e] * sc2 : -INFINITY);
        }
      mx = half_swap_max(row_swap_max(mx));
      const float m_new = fmaxf(m, mx);
      if (__ballot(m_new != m) != 0) {
        const float alpha = m_new != m ? __builtin_amdgcn_exp2f(m - m_new) : 1.f;  // (m = -inf on the first key: 0)
        l *= alpha;
#pragma unroll
        for (int d = 0; d < NDB; ++d) o[d] *= alpha;
        m = m_new;
      }
      const float ref = m == -INFINITY ? 0.f : m;
      uint32_t w[3][4];  // the weights as sums of three bf16, in B operand order
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        // (one rounding between the score and the exponential)
        float a0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e2 >> 1][2 * (e2 & 1)], sc2, -ref));
        float a1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e2 >> 1][2 * (e2 & 1) + 1], sc2, -ref));
        a0 = visible[2 * e2] ? a0 : 0.f;
        a1 = visible[2 * e2 + 1] ? a1 : 0.f;
        l += a0 + a1;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          w[i][e2] = cvt_pk_bf16(a0, a1);
          a0 -= __builtin_bit_cast(float, w[i][e2] << 16);
          a1 -= __builtin_bit_cast(float, w[i][e2] & 0xffff0000u);
        }
      }
      // ---- values
      static_for<0, NDB / 4>([&](auto gc) {
        constexpr int d4 = 4 * decltype(gc)::value;
        auto four = [&](auto back) {
          u32x2_t v0[4], v1[4];
          const unsigned at = v_at + off;
          static_for<0, 4>([&](auto dc) {
            constexpr int d = decltype(dc)::value;
            lds_read_tr16_b64<(d4 + d) * 32>(v0[d], at - back(dc));
            lds_read_tr16_b64<(d4 + d) * 32>(v1[d], at + block2 - back(dc));
          });
          static_for<0, 4>([&](auto dc) {
            constexpr int d = decltype(dc)::value;
            lds_wait2<2 * (3 - d)>(v0[d], v1[d]);
            const u32x4_t a4 = {v0[d][0], v0[d][1], v1[d][0], v1[d][1]};
#pragma unroll
            for (int i = 0; i < 3; ++i) {
              const u32x4_t b4 = {w[i][0], w[i][1], w[i][2], w[i][3]};
              o[d4 + d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a4), __builtin_bit_cast(bf16x8_t, b4), o[d4 + d], 0, 0, 0);
            }
          });
        };
        const int n = (cv >> 1) - d4;  // 16-dim blocks from these on (blocks past the value's dims repeat the last one: accumulated, never stored)
        if (n >= 4) four([&](auto) { return 0u; });
        else if (n > 0) four([&](auto dc) { return (unsigned)(32 * max(0, decltype(dc)::value + 1 - n)); });
      });
    }
  }

  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if constexpr (WS > 1) {  // the waves of a slab meet in the first of them (an empty share has m = -inf and sums of zero)
    float* const mine = (float*)smem + ((ws - 1) * WR + slab) * 64 * (4 * NDB + 2);
    lds_barrier();  // (the ring is free)
    if (ws > 0) {
      *(float2*)(mine + 64 * 4 * NDB + 2 * lane) = make_float2(m, l);
#pragma unroll
      for (int d = 0; d < NDB; ++d) *(f32x4_t*)(mine + d * 256 + lane * 4) = o[d];
    }
    lds_barrier();
    if (ws > 0) return;
#pragma unroll
    for (int s2 = 1; s2 < WS; ++s2) {
      const float* const other = (const float*)smem + ((s2 - 1) * WR + slab) * 64 * (4 * NDB + 2);
      const float2 ml = *(const float2*)(other + 64 * 4 * NDB + 2 * lane);
      const float m_new = fmaxf(m, ml.x);
      const float a = m_new != m ? __builtin_amdgcn_exp2f(m - m_new) : 1.f, c = ml.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml.x - m_new);
      l = l * a + ml.y * c;
#pragma unroll
      for (int d = 0; d < NDB; ++d) o[d] = o[d] * a + *(const f32x4_t*)(other + d * 256 + lane * 4) * c;
      m = m_new;
    }
  }
  const bool empty = j_begin >= min(j_end, n_vis);  // no visible key in this range
  const float inv = empty ? 0.f : 1.f / l;
  const float lse = empty ? -INFINITY : (m + log2f(l)) * 0.6931471805599453f;

  if (row_valid) {
    if (p.splits == 1) {
      if (q == 0) p.lse[row] = lse;
      const int64_t ob = b * p.out_s[0] + t * p.out_s[1] + h * p.out_s[2];
#pragma unroll
      for (int d = 0; d < NDB; ++d) {
        const int dim = 16 * d + 4 * q;
        if (16 * d >= p.d_v) continue;
        const f32x4_t v = o[d] * inv;
        if (p.out_fp32) {
          *(f32x4_t*)((float*)p.out + ob + dim) = v;
        } else {
          u32x2_t pk;
          pk[0] = cvt_pk_bf16(v[0], v[1]);
          pk[1] = cvt_pk_bf16(v[2], v[3]);
          *(u32x2_t*)((uint16_t*)p.out + ob + dim) = pk;
        }
      }
    } else {
      const int64_t rows = (int64_t)p.B * p.T * p.h_q;
      if (q == 0) p.ws_lse[(int64_t)split * rows + row] = lse;
      float* dst = p.ws_out + ((int64_t)split * rows + row) * p.d_v;
#pragma unroll
      for (int d = 0; d < NDB; ++d)
        if (16 * d < p.d_v) *(f32x4_t*)(dst + 16 * d + 4 * q) = o[d] * inv;
    }
  }

  // Was every number of this row finite?  If not, the scalar loop works the row out again: with NaN or infinities in
  // the cache the products above give too much NaN.  They multiply keys a row does not see (hidden by causality, seen by
  // later rows of the tile) by a weight of zero, and an infinite value by each of the three parts of its weight, zero and
  // negative ones among them.
  f32x4_t probes = {l, 0.f, 0.f, 0.f};  // (blocks past the value's dims repeat the last one's numbers)
#pragma unroll
  for (int d = 0; d < NDB; ++d)
#pragma unroll
    for (int e = 0; e < 4; ++e) probes[e] = __builtin_fmaf(o[d][e], 0.f, probes[e]);
  const float probe = (probes[0] + probes[1]) + (probes[2] + probes[3]);
  const bool odd = empty ? probe != 0.f : !(probe > 0.f && probe < INFINITY);
  uint64_t odd_rows = __ballot(odd && row_valid);
  odd_rows |= odd_rows >> 32;
  odd_rows = (odd_rows | odd_rows >> 16) & 0xffff;
  if (odd_rows) {
    wait_vmcnt<0>();  // (what was stored above is stored)
    // (the arguments once more, through a pointer the compiler cannot see through: what only this loop needs is loaded
    // here and not kept, or spilled, across the kernel)
    auto* kernarg = (__attribute__((address_space(4))) const void*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(kernarg));
    const DevParams& pk = *(const DevParams*)kernarg;
    for (; odd_rows; odd_rows &= odd_rows - 1) {
      const int R1 = (rb * WR + slab) * 16 + __ffsll((unsigned long long)odd_rows) - 1;
      const int t1 = R1 / pk.g_q, h1 = g * pk.g_q + (R1 - t1 * pk.g_q);
      const int j1 = min(j_end, pk.causal ? L - pk.T + 1 + t1 : L);
      float o1[DVB / 64], m1, l1;
      scalar_row(pk, b, t1, h1, lane, j_begin, j1, o1, m1, l1);
      store_scalar_row(pk, b, t1, h1, split, lane, j1 <= j_begin, o1, m1, l1);
    }
  }
}

}  // namespace gla
