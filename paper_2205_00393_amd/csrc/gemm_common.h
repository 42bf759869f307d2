// Device helpers shared by the matrix-core GEMM kernels: bit deposits of the
// output address, per-slice maxima and scales, the block -> tile order and the
// split output layout.
#pragma once

#include "kernels.h"

namespace ltn {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint64_t pdep64(uint64_t x, uint64_t mask) {
  uint64_t r = 0;
  while (mask && x) {
    uint64_t low = mask & (~mask + 1);
    if (x & 1) r |= low;
    x >>= 1;
    mask &= mask - 1;
  }
  return r;
}

// sigma = 2^(-floor(log2 max)), so that max * sigma lies in [1, 2)
__device__ __forceinline__ float scale_of(uint32_t maxbits) {
  int e = (int)((maxbits >> 23) & 0xff);
  if (e == 0 || e == 0xff) return 1.f;
  int se = 254 - e;  // biased exponent of 2^(127 - e)
  if (se < 1) se = 1;
  if (se > 254) se = 254;
  return __uint_as_float((uint32_t)se << 23);
}

// Block -> (slice, row tile, column tile). Hardware dispatch sends block w to
// XCD w % 8, so each XCD first gets a contiguous 1/8 of the logical tiles;
// inside a slice, tiles go in groups of G = 8 row tiles, column-major within a
// group, so the blocks resident at once share both row and column panels in
// their XCD's L2 (operand re-reads ~ A / G_n + B / G_m instead of B per row).
__device__ __forceinline__ void tile_of(int64_t w, int64_t tiles_m, int64_t tiles_n, int nb,
                                        int64_t& b, int64_t& bm, int64_t& bn) {
  const int64_t tiles = tiles_m * tiles_n, total = tiles * nb;
  const int64_t logical = (total % 8 == 0) ? (w % 8) * (total / 8) + w / 8 : w;
  b = logical / tiles;
  const int64_t t = logical % tiles;
  const int64_t G = tiles_m < 8 ? tiles_m : 8;
  const int64_t grp = t / (G * tiles_n), r = t % (G * tiles_n);
  bm = grp * G + r % G;
  bn = r / G;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool BF>
struct SplitType;
template <>
struct SplitType<false> {
  using T = _Float16;
  typedef _Float16 V8 __attribute__((ext_vector_type(8)));
  static constexpr int S = 11;
};
template <>
struct SplitType<true> {
  using T = __bf16;
  typedef __bf16 V8 __attribute__((ext_vector_type(8)));
  static constexpr int S = 0;
};

template <bool BF>
__device__ __forceinline__ uint32_t split_pair(float a, float b, float sigma, uint32_t& lo) {
  using T = typename SplitType<BF>::T;
  constexpr float P = (float)(1 << SplitType<BF>::S);
  float xa = a * sigma, xb = b * sigma;
  T ha = (T)xa, hb = (T)xb;
  T la = (T)((xa - (float)ha) * P), lb = (T)((xb - (float)hb) * P);
  lo = (uint32_t)__builtin_bit_cast(uint16_t, la) | ((uint32_t)__builtin_bit_cast(uint16_t, lb) << 16);
  return (uint32_t)__builtin_bit_cast(uint16_t, ha) | ((uint32_t)__builtin_bit_cast(uint16_t, hb) << 16);
}

// One complex output written in the split layout (groups of 4 consecutive
// complex: 16 bytes of hi words, then 16 bytes of lo words; a word holds
// (re, im)); the same bits as the conversion pass produces with scale sigma.
template <bool BF>
__device__ __forceinline__ void store_split(uint32_t* Cw, uint64_t addr, float re, float im, float sigma) {
  uint32_t lo;
  const uint32_t hi = split_pair<BF>(re, im, sigma, lo);
  uint32_t* g = Cw + (addr >> 2) * 8 + (addr & 3);
  g[0] = hi;
  g[4] = lo;
}

// Scale of an fp16 split output written by its producer: from the bound
// |Re c|, |Im c| <= |c| <= K max|a| max|b| <= 2 K max|Re, Im a| max|Re, Im b|
// (the output's own maximum is not known before it is written). One thread
// stores the bound for the consumer, which derives the same scale from it.
__device__ __forceinline__ float split_out_scale(const GemmDesc& d, int64_t b, int64_t K, bool store) {
  const float bound = 2.f * (float)K * __uint_as_float(d.max_a[b]) * __uint_as_float(d.max_b[b]);
  if (store) d.bound_c[b] = __float_as_uint(bound);
  return scale_of(__float_as_uint(bound));
}

}  // namespace

}  // namespace ltn
