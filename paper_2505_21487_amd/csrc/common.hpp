// Shared device-side declarations of the decode-attention library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace gla {

// Division of a 32-bit unsigned number by a divisor fixed on the host, as one
// multiply-high and two shifts:  n / d == (t + ((n - t) >> s1)) >> s2  with
// t = mulhi(n, m), exact for every n < 2^32 (round-up method: m = floor(2^32 *
// (2^l - d) / d) + 1 with l = ceil(log2 d), s1 = min(l, 1), s2 = l - s1).
struct FastDiv {
  uint32_t m, s1, s2;
};
inline FastDiv make_fastdiv(uint32_t d) {
  FastDiv f = {0u, 0u, 0u};
  if (d <= 1) return f;  // t = 0, q = n
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  f.m = (uint32_t)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
  f.s1 = 1;
  f.s2 = l - 1;
  return f;
}
__device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv& f) {
  const uint32_t t = __umulhi(n, f.m);
  return (t + ((n - t) >> f.s1)) >> f.s2;
}

// Cache bytes of a batch from which the MFMA kernels fetch the cache with the streaming hint: the 256 MB
// of the chip's last-level cache (a smaller cache can still be there at the next decode step).
constexpr int64_t kLastLevelCacheBytes = 256ll << 20;

// Kernel-argument block: a flattened copy of the caller's parameter struct.
struct DevParams {
  const uint16_t* q_nope;
  const uint16_t* q_rope;
  const uint16_t* state;
  const uint16_t* rope;
  const uint16_t* kstate;  // keys in a cache of their own (grouped-query baseline); null: key = first d_n dims of the state row
  const int32_t* page_table;
  const int32_t* seq_lens;
  void* out;
  float* lse;
  float* ws_out;   // partial outputs (fp32, normalised by their own row sum)
  float* ws_lse;   // partial log-sum-exp
  int64_t qn_s[3];
  int64_t qr_s[3];
  int64_t st_s[3];
  int64_t rp_s[2];
  int64_t k_s[3];          // strides of kstate (page, head, token)
  int64_t out_s[3];
  int32_t B, T, h_q, h_c, g_q;
  int32_t d_v, d_n, d_r;
  int32_t P, max_pages;
  int32_t causal, out_fp32;
  float scale;
  // generic kernel: uniform split of every sequence's page range
  int32_t splits, pages_per_split;
  // generic MFMA kernel: the split in tokens or, where the caller left it to the library, 0 and the number of ranges
  // allowed while the grid is small, for sequences of up to 4096 tokens and longer ones (range_tokens); divisors (page size,
  // 16-byte chunks of a row in LDS)
  int32_t split_tokens, small_ranges, small_ranges_longer;
  // ... tiles its LDS holds; workgroups that run side by side, ranges that fill one round of them (range_tokens)
  int32_t ring_stages, resident, one_round;
  FastDiv fd_page, fd_cpr;
  int64_t stream_min_bytes; // second MFMA kernel: a batch with more cache bytes than this is fetched with the streaming hint
  int32_t flex_rb;          // flex kernel: blocks of 16 query rows per group
  int32_t* flex_rng;        // flex kernel: per (sequence, strand) the first chunk holding a piece of it (x 2 + its slot) and the last
  // four-wave, eight-wave and second MFMA kernel: flat partition of all key tiles of the batch into chunks
  int32_t num_chunks;       // chunks of the tile list (the main kernel runs one workgroup per chunk and row block)
  int32_t chunk_tiles;      // > 0: fixed tiles per chunk; 0: ceil(total / num_chunks)
  int32_t setup_tiles;      // chunks derived on the device: tiles' worth of time that a chunk's step into another unit costs (cut_list)
  // tuned kernel: constants of the plan, worked out once on the host
  int32_t mb;               // row blocks per group (workgroups per chunk)
  int32_t upb;              // units (group blocks) per sequence
  int32_t lg_page;          // log2(page size)
  int32_t xcd_map;          // 1: grid is a multiple of 8 * mb, chunks are laid out per XCD
  int32_t tiles_full;       // tiles of a sequence that fills its page-table row
  int32_t chunk_guess;      // chunk length if every sequence did
  // Divisors.  Chunks and query heads per group for every kernel with a tile list; the others share their places: one name for the
  // four- and eight-wave kernels, one for the second MFMA kernel (what it divides the number of a wave or of a result row by).
  // Code that both run, cut_list and the rest of tuned_device.hpp, reads neither.  (Places of their own among the generic
  // kernels' fields, two cache lines away, cost the second MFMA kernel 0.2 us: 31.07 -> 31.32.)
  union { FastDiv fd_mb, fd_strands; };
  FastDiv fd_chunks, fd_gq;
  union { FastDiv fd_tiles_full, fd_heads; };
  union { FastDiv fd_units_full, fd_q_len; };
  union { FastDiv fd_upb_mb, fd_group_blocks; };
  int32_t merge_sets_lg, merge_span, merge_windows;  // merge kernel: log2(sets of every unit), chunks per window, windows (tuned_combine_kernel)
  int32_t wide_tiles;       // > 0: the eight-wave kernel runs if the list has that many tiles of 32 tokens, else the four-wave one
};

// The kernel's parameters into the scalar cache, all lines at once.  Left to itself a kernel loads them where it needs them,
// and waits for one line after the other: the four-wave kernel for three before its first memory access and two more before
// its first tile.  us per call without / with (there and in its merge): GLA-2 16 heads 1 x 256 tokens 12.8 / 12.0, 1 x 2048
// 16.4 / 16.1, 1 x 131072 50.7 / 50.2; GTA-4 d_h 128 8 x 2000 16.3 / 15.7.  Nothing in the eight-wave and the second MFMA kernel
// (32.7 / 32.6), and a loss in the generic one (29.3 / 30.1).
__device__ __forceinline__ void fetch_params() {
  static_assert(sizeof(DevParams) > 448 && sizeof(DevParams) <= 512, "eight lines of 64 bytes");
  const auto args = __builtin_amdgcn_kernarg_segment_ptr();
  int t0, t1, t2, t3, t4, t5, t6, t7;
  asm volatile(
      "s_load_dword %0, %8, 0x0\n\ts_load_dword %1, %8, 0x40\n\ts_load_dword %2, %8, 0x80\n\ts_load_dword %3, %8, 0xc0\n\t"
      "s_load_dword %4, %8, 0x100\n\ts_load_dword %5, %8, 0x140\n\ts_load_dword %6, %8, 0x180\n\ts_load_dword %7, %8, 0x1c0\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&s"(t0), "=&s"(t1), "=&s"(t2), "=&s"(t3), "=&s"(t4), "=&s"(t5), "=&s"(t6), "=&s"(t7)
      : "s"(args));
  asm volatile("" ::"s"(t0), "s"(t1), "s"(t2), "s"(t3), "s"(t4), "s"(t5), "s"(t6), "s"(t7));  // (none of them unused; no instruction)
}

// Over the 64 lanes with data-parallel-primitive moves (no LDS round trips): shifts by 1, 2, 4, 8 inside each row of 16
// lanes, then the last lane of row 0 / 2 into row 1 / 3 and lane 31 into the upper half.  A lane that receives nothing
// combines with `none`.
template <class F>
__device__ __forceinline__ float wave_reduce(float v, float none, F f) {
  auto step = [&](auto ctrl, auto rows) {
    v = f(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, none), __builtin_bit_cast(int, v),
                                                                    decltype(ctrl)::value, decltype(rows)::value, 0xf, false)));
  };
  step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});
  step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
  step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
  step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
  step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
  step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_reduce(v, 0.f, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, -__builtin_inff(), [](float a, float b) { return fmaxf(a, b); });
}

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t v) {
  return __builtin_bit_cast(float, ((uint32_t)v) << 16);
}

// Two fp32 values rounded to bf16 (nearest even), `a` in the low half: one
// v_cvt_pk_bf16_f32.  Left to the compiler (not inline asm) so that it sees the
// instruction and provides the wait state a transcendental result needs before
// its first use.
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) { return (uint16_t)cvt_pk_bf16(f, f); }

}  // namespace gla
