// Complex64 GEMM of one contraction step on the bf16 matrix cores:
//   C[merge(m, n)] = sum_k A[m K + k] B[n K + k]
//
// The FP32 matrix cores run at 1/16 of the bf16 rate, and the FP32 tiles
// reached 82-86 % of it: that rate bounded every large complex64 step. Here
// each real operand is written as three bf16 parts, x = h + m + l, each the
// rounding of what the ones before it leave. 3 x 8 significant bits hold
// FP32's 24, so the sum is x itself, and of the nine products of parts the six
// of weight 2^-18 and more are summed in FP32 (the others are below 2^-26 of
// |x y|, a quarter of an FP32 rounding). The complex product takes three real
// ones (Gauss's method, as on the three-product tiles: the sums Re + Im are
// rounded to FP32 and then split), so a complex multiply-add costs 36 bf16
// flops. Every MFMA adds 16 products per accumulator rounding instead of 2:
// the error against complex128 is 0.84 of the FP32 tiles' at K = 2^10 and
// 2^12 (6.9e-7 against 8.1e-7, 1.39e-6 against 1.62e-6).
//
// In the split fp16 mode the same kernel takes two fp16 parts of the operands
// scaled per slice (11 + 11 bits and a sign, three products): 18 flops per
// complex multiply-add against the 24 of the 2 x 2 real form, and operands read
// as complex64, so nothing is converted before. Only sums of 2^10 and more take
// it: there its error is the split tiles' (5.08e-7 against 5.07e-7 at 2^10,
// 7.11e-7 against 7.15e-7 at 2^11, 1.00e-6 against 1.02e-6 at 2^12); on shorter
// ones the rounded operand sums show (1.24e-7 against 1.05e-7 at 2^4). (13,12,11):
// 1.17 ms against 1.39 on the best split tile, matrix cores 57 % busy at 1.78
// GHz.
//
// What bounds it: power. At (13,12,11) the matrix cores are busy 66 % of the
// cycles and the clock falls to 1.8 GHz; the same step takes 2.00 ms (275
// TFLOP/s of 8 flops per complex multiply-add, 1.24 PFLOP/s executed; a large
// library bf16 product reaches 1.13-1.35 PFLOP/s on the same cards) against
// 3.11 ms on the best FP32 tile. Variants that keep the matrix cores fed
// differently measured no better: a wave-specialised block (four waves that
// convert, four that multiply, two LDS buffers) 2.11 ms, one wave per SIMD
// with conversion and products interleaved 2.3 ms.
//
// Layout: 128 x 128 outputs per block, 2 x 2 waves of 64 x 64; a wave holds
// 3 x 64 accumulators, two blocks share a CU, and one block's loads and
// conversion run under the other's products. Threads take groups of eight
// consecutive k' of one row, as two 16-byte units per row: unit u of a row's
// 128 bytes goes to group u & 1, so that two lanes read 32 consecutive bytes;
// both operands use that order of the sum. Nine LDS planes (3 x parts) of
// 16-byte units; group g of row r is unit 2 r + (g ^ (r >> 3 & 1)), so the 16
// rows of a read pass fall on all 64 banks once (no conflicts counted).
#include "gemm_common.h"

namespace ltn {

namespace {

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

// The last part of a number below 2^-110 falls below bf16's smallest number.
// Circuits have such entries (cos(pi/2) = 6e-17 and its products), so operands
// are scaled up by 2^24, which makes every FP32 number above 2^-126 exact; tiles in
// which something overflows then (operands above 2^104, results above 2^79) are
// computed again at the end, on the FP32 matrix cores. 48 multiplications per wave
// and k-tile: 1-2 % of the time.
constexpr float kUp = 0x1p24f;

// Parts of eight FP32 values times `up`, as the operand words of one MFMA lane.
template <int PARTS>
__device__ __forceinline__ void to_parts(const float (&x)[8], float up, u32x4 (&o)[PARTS]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float a = x[2 * j] * up, b = x[2 * j + 1] * up;
    if constexpr (PARTS == 3) {
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){a, b}, bf16x2));
        o[p][j] = w;
        a -= __uint_as_float(w << 16);
        b -= __uint_as_float(w & 0xffff0000u);
      }
    } else {
      const halfx2 h = __builtin_convertvector((floatx2){a, b}, halfx2);
      o[0][j] = __builtin_bit_cast(uint32_t, h);
      // (float)h exactly subtracted: one mixed-precision instruction each
      const floatx2 r = {__builtin_fmaf((float)h.x, -1.f, a), __builtin_fmaf((float)h.y, -1.f, b)};
      o[1][j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, halfx2));
    }
  }
}

template <int PARTS>
__device__ __forceinline__ floatx16 mfma_part(u32x4 a, u32x4 b, floatx16 c) {
  if constexpr (PARTS == 3)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(SplitType<true>::V8, a),
                                                   __builtin_bit_cast(SplitType<true>::V8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(SplitType<false>::V8, a),
                                                  __builtin_bit_cast(SplitType<false>::V8, b), c, 0, 0, 0);
}

// Two fp16 parts: log2 of the scale that takes the operand's largest |Re|, |Im| to
// [2^13, 2^14), so that Re + Im stays below 2^15. At most 2^127: there fp16's
// smallest number stands for 2^-151, so smaller operands lose nothing.
__device__ __forceinline__ int fp16_up(uint32_t maxbits) {
  const int e = (int)((maxbits >> 23) & 0xff);
  if (e == 0 || e == 0xff) return 0;
  return e < 13 ? 127 : 140 - e;
}

__device__ __forceinline__ float pow2(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }

// SPLITK: block w takes chunk w / (tiles * nb) of the sum for tile w % (tiles *
// nb) and writes its FP32 partial of C to part, as k_cgemm_c64's split-K form.
// INPLACE: rows and sum of either operand at any address bits, either operand
// conjugated (adjoint products on the operands of the forward step). The lanes of
// an operand run along its sum as above where that has the lowest address bit,
// else along its rows, whose elements are then neighbours.
// 256 slices, permutations and the plain tile -> in place: (11 rows, sum 9, 7 columns)
// 1.93 -> 1.29 ms, (9,11,7) 2.05 -> 1.47, (6,10,10) 1.61 -> 0.92, but (10,6,10) 1.05 ->
// 1.16: the caller takes it by what there is to permute.
template <int BM, int BN, int PARTS, bool SPLITK, bool INPLACE>
__global__ __launch_bounds__(256, 2) void k_cgemm_parts(GemmDesc d) {
  constexpr int T = 256, KT = 16, NWM = 2, NWN = 2;
  constexpr int WM = BM / NWM, WN = BN / NWN, TM = WM / 32, TN = WN / 32;
  constexpr int ROWS = BM + BN, GRP = 2 * ROWS, R = (GRP + T - 1) / T;
  static_assert(TM >= 1 && TN >= 1 && GRP % 64 == 0, "tile too small");
  __shared__ u32x4 S[3 * PARTS][GRP];

  const int64_t M = int64_t(1) << d.m, N = int64_t(1) << d.n, K = int64_t(1) << d.k;
  int64_t b, bm, bn, chunk = 0, w = blockIdx.x;
  if constexpr (SPLITK) {
    const int64_t per = (M / BM) * (N / BN) * d.nb;
    chunk = w / per;
    w -= chunk * per;
  }
  tile_of(w, M / BM, N / BN, d.nb, b, bm, bn);
  const int64_t KL = SPLITK ? (int64_t(1) << d.kc_bits) : K;
  const int nt = (int)(KL / KT);
  const float2* A = d.A + b * d.sA + (INPLACE ? (int64_t)pdep64((uint64_t)(bm * BM), d.arow) : bm * BM * K + chunk * KL);
  const float2* B = d.B + b * d.sB + (INPLACE ? (int64_t)pdep64((uint64_t)(bn * BN), d.brow) : bn * BN * K + chunk * KL);
  const int ea = PARTS == 3 ? 0 : fp16_up(d.scale_a[b]), eb = PARTS == 3 ? 0 : fp16_up(d.scale_b[b]);

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tid = threadIdx.x;
  const int wm = wave / NWN, wn = wave % NWN;
  const int h = lane >> 5, i = lane & 31;

  // the groups of a tile may end within a round of the threads, between two waves
  auto has = [&](int r) { return GRP % T == 0 || r < R - 1 || T * r + 64 * wave < GRP; };
  const float4* src[R];
  float up[R];
  int dst[R];
  // INPLACE: round 0 is A's, round 1 B's; the weights of the lowest four sum bits
  // and the tile's offset in the sum
  static_assert(!INPLACE || (2 * BM == T && R == 2 && PARTS == 3), "one round of threads per operand");
  int64_t weight[2][4];
  uint64_t at[2] = {0, 0}, step[2];
  if constexpr (INPLACE) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const uint64_t sum = r ? d.bsum : d.asum;
      step[r] = pdep64(KT, sum);
#pragma unroll
      for (int j = 0; j < 4; ++j) weight[r][j] = (int64_t)pdep64(1ull << j, sum);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int c = tid + T * r;
    int row = c >> 1, g = c & 1;
    if constexpr (INPLACE) {
      constexpr int rows[2] = {BM, BN};
      if (!((r ? d.bsum : d.asum) & 1)) {
        g = (tid / rows[r]) & 1;  // threads past the operand have no group
        row = (tid & (rows[r] - 1)) + (r ? BM : 0);
      }
      src[r] = reinterpret_cast<const float4*>((r ? B + pdep64((uint64_t)(row - BM) & (BN - 1), d.brow)
                                                  : A + pdep64((uint64_t)row, d.arow)) + g * weight[r][1]);
    } else {
      src[r] = reinterpret_cast<const float4*>(row < BM ? A + row * K : B + (row - BM) * K) + g;
    }
    up[r] = PARTS == 3 ? kUp : pow2(row < BM ? ea : eb);
    dst[r] = 2 * row + (g ^ ((row >> 3) & 1));
  }
  // one k-tile of group r, and on to the next tile (`more`: there is one)
  auto load = [&](int r, float4 (&v)[4], bool more) {
    if (!has(r)) return;
    if constexpr (INPLACE) {
      const float2* p = reinterpret_cast<const float2*>(src[r]) + at[r];
      if (weight[r][0] == 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          v[q] = *reinterpret_cast<const float4*>(p + ((q & 1) * weight[r][2] + (q >> 1) * weight[r][3]));
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float2* s = p + ((q & 1) * weight[r][2] + (q >> 1) * weight[r][3]);
          const float2 x = s[0], y = s[weight[r][0]];
          v[q] = make_float4(x.x, x.y, y.x, y.y);
        }
      }
      const uint64_t sum = r ? d.bsum : d.asum;
      if (more) at[r] = ((at[r] | ~sum) + step[r]) & sum;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = src[r][2 * q];
      src[r] += more ? KT / 2 : 0;
    }
  };
  auto stash = [&](int r, const float4 (&v)[4]) {
    if (!has(r)) return;
    float re[8], im[8], su[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      re[2 * q] = v[q].x;
      im[2 * q] = v[q].y;
      re[2 * q + 1] = v[q].z;
      im[2 * q + 1] = v[q].w;
    }
    if constexpr (INPLACE) {
      const float sign = (r ? d.conj_b : d.conj_a) ? -1.f : 1.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) im[q] *= sign;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) su[q] = re[q] + im[q];
    u32x4 o[PARTS];
    to_parts<PARTS>(re, up[r], o);
#pragma unroll
    for (int p = 0; p < PARTS; ++p) S[p][dst[r]] = o[p];
    __builtin_amdgcn_sched_barrier(0);
    to_parts<PARTS>(im, up[r], o);
#pragma unroll
    for (int p = 0; p < PARTS; ++p) S[PARTS + p][dst[r]] = o[p];
    __builtin_amdgcn_sched_barrier(0);
    to_parts<PARTS>(su, up[r], o);
#pragma unroll
    for (int p = 0; p < PARTS; ++p) S[2 * PARTS + p][dst[r]] = o[p];
    __builtin_amdgcn_sched_barrier(0);
  };

  floatx16 acc[3][TM][TN];
  auto clear = [&]() {
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TN; ++y)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[p][x][y][v] = 0.f;
  };
  clear();

  auto unit = [&](int row) { return 2 * row + (h ^ ((row >> 3) & 1)); };
  auto multiply = [&](int pl) {
    u32x4 bv[TN][PARTS];
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int p = 0; p < PARTS; ++p) bv[y][p] = S[pl * PARTS + p][unit(BM + wn * WN + 32 * y + i)];
#pragma unroll
    for (int x = 0; x < TM; ++x) {
      u32x4 av[PARTS];
#pragma unroll
      for (int p = 0; p < PARTS; ++p) av[p] = S[pl * PARTS + p][unit(wm * WM + 32 * x + i)];
      // small products first; the tiles along y alternate
#pragma unroll
      for (int s = PARTS - 1; s >= 0; --s)
#pragma unroll
        for (int pa = 0; pa <= s; ++pa)
#pragma unroll
          for (int y = 0; y < TN; ++y)
            acc[pl][x][y] = mfma_part<PARTS>(av[pa], bv[y][s - pa], acc[pl][x][y]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // A's group is fetched one k-tile ahead, under the products of the last two
  // planes; registers hold no more (256 used, none spilled). B's is in flight
  // while A's is converted. Issuing both at the top of the loop: (15,5,12)
  // 0.31 against 0.28 ms, no difference on long sums.
  float4 v[R][4];
  load(0, v[0], nt > 1);
  for (int t = 0; t < nt; ++t) {
#pragma unroll
    for (int r = 1; r < R; ++r) load(r, v[r], true);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) stash(r, v[r]);
    __syncthreads();
    multiply(0);
    load(0, v[0], t + 2 < nt);
    __builtin_amdgcn_sched_barrier(0);
    multiply(1);
    multiply(2);
  }

  // Re and Im from the three products, in the place of the first and the third;
  // whether any of them is not finite
  auto combine = [&]() {
    float none = 0.f;
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
      for (int y = 0; y < TN; ++y)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float p1 = acc[0][x][y][v], p2 = acc[1][x][y][v];
          acc[0][x][y][v] = p1 - p2;
          acc[2][x][y][v] = acc[2][x][y][v] - p1 - p2;
          if (PARTS == 3) none = fmaf(acc[0][x][y][v], 0.f, fmaf(acc[2][x][y][v], 0.f, none));
        }
    return none != none;
  };
  bool odd = combine();
  float post = 1.f / (kUp * kUp);
  if constexpr (PARTS == 3) {
    // Infinities, NaN, or a number too large for the scaled parts: the block's tile
    // again on the FP32 matrix cores, three products as before. A thread takes a row
    // of a k-tile (stride 17 in LDS: no bank conflicts). Bound by those cores:
    // (13,12,11) with NaN everywhere 5.4 ms, of which 3.3 here, as on the FP32 tiles
    // (3.1); with each lane summing its own outputs 146 ms.
    if (__syncthreads_or(odd)) {
      constexpr int LD = KT + 1, PL = ROWS * LD;
      static_assert(ROWS <= T && 3 * PL * sizeof(float) <= sizeof(S), "a thread per row, three planes");
      float* F = reinterpret_cast<float*>(S);
      const int me = 64 * wave + __lane_id(), col = me - BM;
      const float2* row = me < BM ? A + (INPLACE ? (int64_t)pdep64((uint64_t)me, d.arow) : me * K)
                                   : B + (INPLACE ? (int64_t)pdep64((uint64_t)(col & (BN - 1)), d.brow) : col * K);
      const uint64_t sum = me < BM ? d.asum : d.bsum;
      const float sign = INPLACE && (me < BM ? d.conj_a : d.conj_b) ? -1.f : 1.f;
      uint64_t z = 0;
      clear();
      for (int t = 0; t < nt; ++t) {
        __syncthreads();
        if (me < ROWS) {
#pragma unroll 8
          for (int q = 0; q < KT; ++q) {
            const float2 v = row[z];
            z = INPLACE ? ((z | ~sum) + 1) & sum : z + 1;
            float* f = F + me * LD + q;
            f[0] = v.x;
            f[PL] = v.y * sign;
            f[2 * PL] = v.x + v.y * sign;
          }
        }
        __syncthreads();
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll 2
          for (int q = 0; q < KT; q += 2)
#pragma unroll
            for (int x = 0; x < TM; ++x)
#pragma unroll
              for (int y = 0; y < TN; ++y)
                acc[pl][x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                    F[pl * PL + (wm * WM + 32 * x + i) * LD + q + h],
                    F[pl * PL + (BM + wn * WN + 32 * y + i) * LD + q + h], acc[pl][x][y], 0, 0, 0);
      }
      combine();
      post = 1.f;
    }
  }

  const uint64_t maskA = SPLITK ? ((uint64_t)(M - 1) << d.n) : d.cmask;
  const uint64_t maskB = ~maskA & ((1ull << (d.m + d.n)) - 1);
  const float so =
      !SPLITK && d.split_out == 2 ? split_out_scale(d, b, K, bm == 0 && bn == 0 && threadIdx.x == 0) : 1.f;
  float2* Cc = SPLITK ? d.part + ((b << (d.k - d.kc_bits)) + chunk) * (M * N) : d.C + b * d.sC;
  uint32_t* Cw = reinterpret_cast<uint32_t*>(Cc);
  const int64_t row0 = bm * BM + wm * WM, col0 = bn * BN + wn * WN;
  float vmax = 0.f;
  auto put = [&](uint64_t addr, float re, float im) {
    if (!SPLITK && d.split_out == 1)
      store_split<true>(Cw, addr, re, im, 1.f);
    else if (!SPLITK && d.split_out)
      store_split<false>(Cw, addr, re, im, so);
    else
      Cc[addr] = make_float2(re, im);
  };
  const uint64_t pbase = pdep64((uint64_t)(row0 + 4 * h), maskA);
  uint64_t pq[4], pg[4], pt[TM];
#pragma unroll
  for (int q = 0; q < 4; ++q) pq[q] = pdep64((uint64_t)q, maskA);
#pragma unroll
  for (int g = 0; g < 4; ++g) pg[g] = pdep64((uint64_t)(8 * g), maskA);
#pragma unroll
  for (int x = 0; x < TM; ++x) pt[x] = pdep64((uint64_t)(32 * x), maskA);
  const bool rows4 = (maskA & 3) == 3;
  // the two scales taken back at once: their product reaches 2^254, whose inverse
  // FP32 does not hold
  auto down = [&](float v) { return PARTS == 3 ? v * post : __builtin_ldexpf(v, -(ea + eb)); };
#pragma unroll
  for (int y = 0; y < TN; ++y) {
    const uint64_t pn = pdep64((uint64_t)(col0 + 32 * y + i), maskB);
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float vr[4], vi[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          vr[q] = down(acc[0][x][y][4 * g + q]);
          vi[q] = down(acc[2][x][y][4 * g + q]);
          vmax = fmaxf(vmax, fmaxf(fabsf(vr[q]), fabsf(vi[q])));
        }
        const uint64_t a0 = pbase | pt[x] | pg[g] | pn;
        if (rows4) {
          if (!SPLITK && d.split_out) {
            uint32_t hw[4], lw[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
              hw[q] = d.split_out == 1 ? split_pair<true>(vr[q], vi[q], 1.f, lw[q])
                                       : split_pair<false>(vr[q], vi[q], so, lw[q]);
            uint4* g4 = reinterpret_cast<uint4*>(Cw) + (a0 >> 2) * 2;
            g4[0] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
            g4[1] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
          } else {
            float4* c4 = reinterpret_cast<float4*>(Cc + a0);
            c4[0] = make_float4(vr[0], vi[0], vr[1], vi[1]);
            c4[1] = make_float4(vr[2], vi[2], vr[3], vi[3]);
          }
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) put(a0 | pq[q], vr[q], vi[q]);
        }
      }
  }
  if (!SPLITK && d.scale_c) block_raise_max(d.scale_c + b, vmax, reinterpret_cast<float*>(S));
}

template <int BM, int BN, int PARTS, bool SPLITK, bool INPLACE = false>
void run_parts(const GemmDesc& d, hipStream_t st) {
  const int64_t chunks = SPLITK ? int64_t(1) << (d.k - d.kc_bits) : 1;
  const int64_t blocks = ((int64_t(1) << d.m) / BM) * ((int64_t(1) << d.n) / BN) * d.nb * chunks;
  hipLaunchKernelGGL((k_cgemm_parts<BM, BN, PARTS, SPLITK, INPLACE>), dim3((unsigned)blocks), dim3(256), 0, st, d);
}

struct PartsCfg {
  int bm, bn, parts;
  bool splitk;
  const char* name;
};
const PartsCfg kParts[] = {
    {128, 128, 3, false, "parts_128x128x16"},
    {128, 64, 3, false, "parts_128x64x16"},
    {128, 128, 3, true, "splitk_parts_128x128x16"},
    {128, 64, 3, true, "splitk_parts_128x64x16"},
    // split fp16 mode only
    {128, 128, 2, false, "parts2_128x128x16"},
    {128, 128, 2, true, "splitk_parts2_128x128x16"},
};
constexpr int kNumParts = sizeof(kParts) / sizeof(kParts[0]), kNumParts3 = 4;
constexpr int kParts2MinK = 10;  // shorter sums: less exact than the split tiles

}  // namespace

int parts_config_count(int mode) { return mode == LTN_SPLIT_F16 ? kNumParts : kNumParts3; }

bool parts_config_fits(int cfg, int m, int k, int n, int mode) {
  if (cfg < 0 || cfg >= parts_config_count(mode) || m >= 40 || n >= 40) return false;
  const PartsCfg& t = kParts[cfg];
  const int c = t.splitk ? splitk_chunk_bits(m, k, n) : 0;
  if (t.parts == 2 && k < kParts2MinK) return false;
  return (1ll << m) >= t.bm && (1ll << n) >= t.bn && k - c >= 4 && (!t.splitk || c > 0);
}

bool parts_config_splitk(int cfg) { return cfg >= 0 && cfg < kNumParts && kParts[cfg].splitk; }

const char* parts_config_name(int cfg, int mode) {
  return cfg >= 0 && cfg < parts_config_count(mode) ? kParts[cfg].name : "?";
}

bool parts_config_in_place(int cfg) { return cfg == 0 || cfg == 1; }

// From sums of 2^14 on, the split-K form where it fits: it takes the same time and
// its chunks' sums gather less rounding. 53-qubit slices, (13,17,8), (12,15,9) and
// (14,16,6) of four slices in either form: 34.9, 8.8 and 10.5 ms, errors of the whole
// slice 5.0e-6 split and 7.6e-6 full; split fp16 20.8 and 5.1 ms, 4.1e-6 and 6.8e-6.
// Only while the chunks' partials are few against the sum (16 bytes each way per
// output and chunk: 3 % of the time at the line, 6 % in split fp16).
bool parts_config_yields(int cfg, int m, int k, int n, int mode) {
  const int split = cfg == 0 ? 2 : cfg == 1 ? 3 : cfg == 4 ? 5 : -1;
  return k >= 14 && split >= 0 && parts_config_fits(split, m, k, n, mode) && splitk_chunk_bits(m, k, n) <= k - 12;
}

// complex64: full tiles where two 128 x 128 tiles per CU can share it, or two
// 128 x 64 tiles ((13,10,10), 512 tiles: 0.286 ms; (18,6,6): 0.081 against
// 0.085 on the best FP32 tile); with one per CU, the split-K form on sums from
// 2^11 ((13,11,9): 0.302 against 0.347, (11,12,11): 0.55 against 0.69) and
// full tiles on shorter ones ((11,10,11): 0.163 against 0.177, FP32 0.221) down to
// 2^6 ((12,6,10): 25.7 us, FP32 27.5; (14,5,8) 21.0 and 20.2). Sums of 2^4 take 64
// columns on FP32 ((18,4,6): 65 us on parts, 45 on FP32; (18,5,6) 58 on both).
// Fewer tiles: split-K where its chunks give half a block per CU ((10,10,10):
// 0.065 against 0.076 ms on the best FP32 tile, (13,14,7): 0.55 against 0.90;
// (7,12,7), 16 blocks: 0.053 against 0.029; full tiles, (11,10,10): 0.136
// against 0.124).
// split fp16: the two-part tiles on sums of 2^10 and more ((13,10,10): 0.168
// against 0.207 ms on the best split tile, (13,12,11): 1.30 against 1.53), with
// one tile per CU split-K from 2^12 ((11,12,11): 0.353 against 0.363, (13,11,9):
// 0.210 against 0.198), with fewer from 2^11 ((10,12,10): 0.120 against 0.155,
// (13,15,8): 1.38 against 2.67; at 2^10, (11,10,10): 0.086 against 0.074).
// split bf16, and 64 columns in either split mode: the three-part split-K form
// where a long sum leaves at most one 64 x 64 split tile per CU ((13,14,7) 0.59
// against 1.16 ms, (14,13,6) 0.40 against 0.81; with two per CU, (12,13,9):
// 0.59 against 0.51, and with a shorter sum, (10,12,10): 0.171 against 0.148).
// In place the short sums stay on parts, as FP32 tiles want permuted operands
// (11 rows, sum of 2^4, 7 columns x 256: 176 us, permuted 185).
int parts_config_default(int m, int k, int n, int64_t nb, int mode, bool in_place) {
  if (m < 7 || n < 6 || m + n > 40) return -1;
  const bool wide = n >= 7, f16 = mode == LTN_SPLIT_F16;
  const int64_t outs = (int64_t(1) << (m + n)) * nb, tiles = outs >> (wide ? 14 : 13);
  int full = -1, split = -1;
  if (mode == LTN_C64) {
    full = wide ? 0 : 1;
    split = wide ? 2 : 3;
  } else if (f16 && wide) {
    full = 4;
    split = k >= 11 ? 5 : -1;
  } else if (k >= 13 && outs >> 12 <= 256) {
    split = wide ? 2 : 3;
  }
  const bool yields = !in_place && full >= 0 && parts_config_yields(full, m, k, n, mode);
  if (full >= 0 && !yields && parts_config_fits(full, m, k, n, mode) &&
      (tiles >= 512 ? wide || k >= 5 || in_place
                    : wide && tiles >= 256 && (k >= 6 || in_place) &&
                          (k < (f16 ? 12 : 11) || !parts_config_fits(split, m, k, n, mode))))
    return full;
  if (!parts_config_fits(split, m, k, n, mode) || (tiles << splitk_chunk_bits(m, k, n)) < 128) return -1;
  return tiles < 512 || yields ? split : -1;
}

void launch_cgemm_parts(const GemmDesc& d0, hipStream_t st) {
  GemmDesc d = d0;
  if (parts_config_splitk(d.cfg)) d.kc_bits = d.k - splitk_chunk_bits(d.m, d.k, d.n);
  if (d.asum) {
    if (d.cfg == 0)
      run_parts<128, 128, 3, false, true>(d, st);
    else
      run_parts<128, 64, 3, false, true>(d, st);
    return;
  }
  switch (d.cfg) {
    case 0: run_parts<128, 128, 3, false>(d, st); break;
    case 1: run_parts<128, 64, 3, false>(d, st); break;
    case 2: run_parts<128, 128, 3, true>(d, st); break;
    case 3: run_parts<128, 64, 3, true>(d, st); break;
    case 4: run_parts<128, 128, 2, false>(d, st); break;
    case 5: run_parts<128, 128, 2, true>(d, st); break;
  }
  if (parts_config_splitk(d.cfg)) launch_splitk_reduce(d, st);
}

}  // namespace ltn
