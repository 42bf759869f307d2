// Runs of small contraction steps, one block per slice, or one per slice and group
// of steps that do not depend on those of another.
//
// A step of a few hundred multiply-adds costs a launch (3-5 us, in a graph as
// well) and its operands' way through memory; trees of random circuits begin
// with dozens to hundreds of them. A run is a list of such steps in which a
// step may consume what an earlier one produced: the block keeps everything
// produced and consumed inside the run in LDS, reads the run's inputs (leaves,
// and tensors of earlier launches) into LDS once at its start and writes only
// what later launches need. Steps that do not depend on each other share a
// level; the block meets at one barrier per level, and inside a level each
// small step is one wave's, each larger one the whole block's. The sums are
// those of the generic kernel with the step's TK to the bit (TK partial sums per
// output, added in a fixed order; the fused multiply-adds are spelled out in
// both), so it does not matter to a result whether a step is in a run; how many
// lanes share the TK partial sums goes by the threads there are.
//
// What bounds it: latency (a barrier, descriptor and LDS round trip per level).
// Measured per call, launches of independent steps -> runs: 12-qubit circuit
// (24 steps, one slice) 66 -> 26 us; 20-qubit circuit of 16 slices, complex64, 167 ->
// 77 us (88 with one group); of 256 slices in batches of 96, split fp16, 594 us (669
// with one group).
#include <cstddef>

#include "kernels.h"

namespace ltn {

namespace {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef const f2 __attribute__((address_space(1))) * gptr;  // a pointer read from memory: say that it is global

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int kSide = 64;  // inputs up to this size are read side by side

// Bits of x to the positions of mask, one run of neighbouring mask bits at a
// time: most masks have one to three runs.
__device__ __forceinline__ uint32_t dep(uint32_t x, uint32_t mask) {
  uint32_t r = 0;
  while (mask) {
    const uint32_t low = mask & (0u - mask), top = (mask + low) & ~mask;  // the run, and the bit above it
    const uint32_t run = mask & (top - 1u);
    const int at = __builtin_ctz(mask), len = __builtin_popcount(run);
    r |= (x << at) & run;
    x >>= len;
    mask &= ~run;
  }
  return r;
}

// Offset added by `bits` of x, bit j going to position list[j] (bytes, read eight
// at a time).
__device__ __forceinline__ int64_t scatter(uint64_t x, const int8_t* list, int bits) {
  int64_t r = 0;
  for (int j = 0; j < bits; j += 8) {
    uint64_t w = *reinterpret_cast<const uint64_t*>(list + j);
    for (int i = j; i < bits && i < j + 8; ++i, w >>= 8) r |= (int64_t)((x >> i) & 1) << (w & 63);
  }
  return r;
}

// The values of the sliced axes' bits of id, gathered to the low bits.
__device__ __forceinline__ uint64_t slice_values(uint64_t id, const int8_t* list, int bits) {
  uint64_t r = 0;
  for (int j = 0; j < bits; j += 8) {
    uint64_t w = *reinterpret_cast<const uint64_t*>(list + j);
    for (int i = j; i < bits && i < j + 8; ++i, w >>= 8) r |= ((id >> (w & 63)) & 1) << i;
  }
  return r;
}

extern __shared__ f2 lds[];

// One step for the threads t = 0 .. T - 1 (a wave or the block). Forward:
// out[X(x) | Y(y)] = sum_z P[x Z + z] Q[y Z + z]; adjoint: out[x Y + y] = sum_z
// P[X(x) | Y(z)] conj(Q[z Y + y]), X and Y from the tables. TK partial sums per
// output, W of them by each of TK / W lanes, added in the order of the generic
// kernel's shuffles (its upper lane bits first).
template <int TK, int W, bool ADJ>
__device__ __forceinline__ void small_op(const GenericDesc& d, int b, int t, int T) {
  constexpr int L = TK / W;
  const int lane = t % L, xb = d.xb(), yb = d.yb(), zb = d.zb();
  const int outs = 1 << (xb + yb), zc = 1 << zb;
  const uint16_t* X = reinterpret_cast<const uint16_t*>(lds) + d.nb;
  const uint16_t* Y = X + (1 << xb);
  const f2 *P = lds + d.lp(), *Q = lds + d.lq();
  float top = 0.f;
  for (int o = t / L; o < outs; o += T / L) {
    const int x = o & ((1 << xb) - 1), y = o >> xb;
    const int px = ADJ ? X[x] : x << zb, oa = ADJ ? (x << yb) | y : X[x] | Y[y];
    float re[W], im[W];
#pragma unroll
    for (int j = 0; j < W; ++j) re[j] = im[j] = 0.f;
    // two or more products' operands on their way at a time
    constexpr int U = W > 1 ? W : 2;
    for (int z = lane; z < zc; z += U * L) {
      f2 p[U], q[U];
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const bool in = z + j * L < zc;
        const int w = in ? z + j * L : z;
        p[j] = P[ADJ ? px | Y[w] : px | w];
        q[j] = Q[ADJ ? (w << yb) | y : (y << zb) | w];
        if (!in) p[j] = q[j] = f2{0.f, 0.f};  // both: 0 x inf
        if (ADJ) q[j].y = -q[j].y;
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        re[j % W] += fmaf(p[j].x, q[j].x, -(p[j].y * q[j].y));
        im[j % W] += fmaf(p[j].y, q[j].x, p[j].x * q[j].y);
      }
    }
#pragma unroll
    for (int h = W / 2; h > 0; h >>= 1)
#pragma unroll
      for (int j = 0; j < h; ++j) {
        re[j] += re[j + h];
        im[j] += im[j + h];
      }
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1) {
      re[0] += __shfl_xor(re[0], off, L);
      im[0] += __shfl_xor(im[0], off, L);
    }
    if (lane == 0) {
      const f2 v = f2{re[0], im[0]};
      if (d.lo() >= 0) lds[d.lo() + oa] = v;
      if (d.out) ((f2 __attribute__((address_space(1)))*)(d.out + b * d.sO))[oa] = v;
      top = fmaxf(top, fmaxf(fabsf(v.x), fabsf(v.y)));
    }
  }
  if (d.scale_out) record_max(d.scale_out + b, top);
}

template <bool ADJ>
__global__ __launch_bounds__(kThreads) void k_small_run(const GenericDesc* __restrict__ all, RunGroups groups, int big,
                                                        const float2* __restrict__ leafdata,
                                                        const uint64_t* __restrict__ ids) {
  const uint64_t id = ids[blockIdx.x];
  const GenericDesc* descs = all + groups.off[blockIdx.y];
  const int n = groups.off[blockIdx.y + 1] - groups.off[blockIdx.y];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // inputs (operands with an address in memory) to their places: 16 lanes each,
  // so that the chains descriptor -> leaf descriptor -> data of 32 operands run
  // side by side
  for (int q = tid >> 4; q < 2 * n; q += kThreads / 16) {
    const GenericDesc& d = descs[q >> 1];
    const bool second = q & 1;
    const float2* src = second ? d.Q : d.P;
    if (!src) continue;
    const int size = 1 << ((second ? d.yb() : d.xb()) + d.zb());
    if (size > kSide) continue;
    f2* dst = lds + (second ? d.lq() : d.lp());
    if (second ? d.leafQ() : d.leafP()) {
      const GatherDesc& g = *reinterpret_cast<const GatherDesc*>(src);
      const int64_t base = g.src_off + scatter(slice_values(id, g.sl_bit, g.nsl), g.sl_src_bit, g.nsl);
      for (int e = tid & 15; e < size; e += 16) dst[e] = ((gptr)(leafdata + base))[scatter(e, g.src_bit, g.rank)];
    } else {
      gptr from = (gptr)(src + b * (second ? d.sQ : d.sP));
      for (int e = tid & 15; e < size; e += 16) dst[e] = from[e];
    }
  }
  // larger ones by the block
  for (int i = 0; i < n && big; ++i) {
    const GenericDesc& d = descs[i];
    const int np = d.P ? 1 << (d.xb() + d.zb()) : 0, nq = d.Q ? 1 << (d.yb() + d.zb()) : 0;
    if (np <= kSide && nq <= kSide) continue;
    for (int second = 0; second < 2; ++second) {
      const int size = second ? nq : np;
      const float2* src = second ? d.Q : d.P;
      f2* dst = lds + (second ? d.lq() : d.lp());
      if (size <= kSide) continue;
      if (second ? d.leafQ() : d.leafP()) {
        const GatherDesc& g = *reinterpret_cast<const GatherDesc*>(src);
        const int64_t base = g.src_off + scatter(slice_values(id, g.sl_bit, g.nsl), g.sl_src_bit, g.nsl);
        for (int e = tid; e < size; e += kThreads) dst[e] = ((gptr)(leafdata + base))[scatter(e, g.src_bit, g.rank)];
      } else {
        gptr from = (gptr)(src + b * (second ? d.sQ : d.sP));
#pragma unroll 4
        for (int e = tid; e < size; e += kThreads) dst[e] = from[e];
      }
    }
  }
  // address tables
  for (int i = wave; i < n; i += kWaves) {
    const GenericDesc& d = descs[i];
    const int nx = 1 << d.xb(), ny = 1 << (ADJ ? d.zb() : d.yb());
    uint16_t* X = reinterpret_cast<uint16_t*>(lds) + d.nb;
    for (int e = lane; e < nx + ny; e += 64) {
      const uint32_t mask = (uint32_t)(ADJ ? (e < nx ? d.px : d.pz) : (e < nx ? d.ox : d.oy));
      X[e] = (uint16_t)dep(e < nx ? e : e - nx, mask);
    }
  }
  // A lane holds one word of the descriptor; the next one is on its way during
  // a step (a scalar load at the step's start cost it 0.2 us).
  constexpr int kWords = sizeof(GenericDesc) / 4;
  const uint32_t* words = reinterpret_cast<const uint32_t*>(descs);
  uint32_t next = lane < kWords ? words[lane] : 0u;
  for (int i = 0; i < n; ++i) {
    const uint32_t w = next;
    next = lane < kWords && i + 1 < n ? words[(i + 1) * kWords + lane] : 0u;
    auto word = [&](size_t byte) { return (uint32_t)__builtin_amdgcn_readlane((int)w, (int)(byte / 4)); };
    auto pair = [&](size_t byte) { return word(byte) | (uint64_t)word(byte + 4) << 32; };
    GenericDesc d;
    d.plan = word(offsetof(GenericDesc, plan));
    if (d.level_first()) __syncthreads();
    if (d.wave() >= 0 && d.wave() != wave) continue;
    d.shape = word(offsetof(GenericDesc, shape));
    d.places = word(offsetof(GenericDesc, places));
    d.nb = (int)word(offsetof(GenericDesc, nb));
    d.out = reinterpret_cast<float2*>(pair(offsetof(GenericDesc, out)));
    d.sO = (int64_t)pair(offsetof(GenericDesc, sO));
    d.scale_out = reinterpret_cast<uint32_t*>(pair(offsetof(GenericDesc, scale_out)));
    const int t = d.wave() >= 0 ? lane : tid, T = d.wave() >= 0 ? 64 : kThreads;
    switch (d.sums()) {
      case 0: small_op<1, 1, ADJ>(d, b, t, T); break;
      case 1: small_op<8, 1, ADJ>(d, b, t, T); break;
      case 2: small_op<8, 8, ADJ>(d, b, t, T); break;
      case 3: small_op<64, 1, ADJ>(d, b, t, T); break;
      default: small_op<64, 8, ADJ>(d, b, t, T); break;
    }
  }
}

}  // namespace

int small_run_waves() { return kWaves; }

int small_run_side() { return kSide; }

void launch_small_run(const GenericDesc* d_descs, const RunGroups& groups, bool adjoint, bool big, int lds_elems,
                      const float2* leafdata, const uint64_t* ids, int nb, hipStream_t st) {
  const size_t bytes = (size_t)lds_elems * sizeof(f2);
  const dim3 grid((unsigned)nb, (unsigned)groups.n);
  if (adjoint)
    hipLaunchKernelGGL(k_small_run<true>, grid, dim3(kThreads), bytes, st, d_descs, groups, big, leafdata, ids);
  else
    hipLaunchKernelGGL(k_small_run<false>, grid, dim3(kThreads), bytes, st, d_descs, groups, big, leafdata, ids);
}

}  // namespace ltn
