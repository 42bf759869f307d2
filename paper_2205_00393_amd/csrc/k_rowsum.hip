// Products with few columns read in place: out[X(x) | Y(y)] = sum_z P[X(x) | Z(z)]
// Q[Y(y) | Z(z)] with at most 16 columns y, every bit of x, y and z at any address
// bit, either operand conjugated. These are the adjoint products of steps that
// absorb a small tensor: the sum runs over 2^6 to 2^16 elements of the large
// operand, which lies in the forward step's order, not in the product's.
//
// Bound by HBM (P is read once, about Y / 2 multiply-adds per 8 bytes). A block
// takes a tile of P of 2^xt rows x 2^zt elements that consists of the lowest row
// and sum bits, so of whole runs of addresses: it is read in address order, 16
// bytes a lane, and put into LDS by rows (stride 2^xt + 1 in z: lanes that hold
// neighbouring z write to different banks). A thread has one row, all columns and
// every 2^(8 - xt)-th z of the tile; tiles along z are summed one by one (two
// levels of FP32 sums), the threads of a row are added through LDS at the end.
// The next tile is on its way into registers during the products.
// Measured, 256 slices, against permuting both operands and a narrow or generic
// kernel: sum of 2^8, 2^10 rows, 4 columns 1.03 -> 0.18 ms (537 MB: 3.0 TB/s); sum
// of 2^10, 2^8 rows 0.40 -> 0.16; sum of 2^10, 2^6 rows, 16 columns 0.39 -> 0.16; the
// root's 2^16 rows, sum of 1, 0.23 -> 0.12. With 16 columns LDS reads bound it.
#include <algorithm>

#include "kernels.h"

namespace ltn {

namespace {

__device__ __host__ __forceinline__ uint64_t pdep_r(uint64_t x, uint64_t mask) {
  uint64_t r = 0;
  for (; x; mask &= mask - 1, x >>= 1)
    if (x & 1) r |= mask & (0 - mask);
  return r;
}

__device__ __forceinline__ uint64_t madd_r(uint64_t a, uint64_t d, uint64_t mask) {
  return ((a | ~mask) + d) & mask;
}

constexpr int kTile = 11;              // log2 of a tile's elements
constexpr int kPairs = 4, kQ = 4;      // 16-byte loads of P, elements of Q per thread
constexpr int kLds = 3 << (kTile - 1); // with the stride's padding

template <int Y>
__global__ __launch_bounds__(256) void k_rowsum(RowsumDesc d) {
  constexpr int kRed = 256 * Y > kLds ? 256 * Y : kLds;
  __shared__ float2 Ps[kRed];  // the tile; at the end the threads' sums
  __shared__ float2 Qs[256 * kQ];
  __shared__ uint32_t off_lo[64], off_hi[32];
  __shared__ uint16_t to_lo[64], to_hi[32];
  const int tid = threadIdx.x;
  const int XT = 1 << d.xt, ZT = 1 << d.zt, stride = XT > 1 ? XT + 1 : 1;
  const int elems = 1 << (d.xt + d.zt);
  // tile element -> offset in P, place in LDS; both linear in the bits
  for (int i = tid; i < 96; i += 256) {
    const uint64_t at = pdep_r(i < 64 ? (uint64_t)i : (uint64_t)(i - 64) << 6, d.tile);
    int x = 0, z = 0;
    uint64_t mx = d.px, mz = d.pz;
    for (int j = 0; j < d.xt; ++j, mx &= mx - 1) x |= at & mx & (0 - mx) ? 1 << j : 0;
    for (int j = 0; j < d.zt; ++j, mz &= mz - 1) z |= at & mz & (0 - mz) ? 1 << j : 0;
    (i < 64 ? off_lo[i] : off_hi[i - 64]) = (uint32_t)at;
    (i < 64 ? to_lo[i] : to_hi[i - 64]) = (uint16_t)(z * stride + x);
  }
  __syncthreads();
  uint32_t poff[kPairs], pto[kPairs];
  uint32_t step = 0;  // from the first element of a pair to the second, in LDS
  step = to_lo[1];
#pragma unroll
  for (int i = 0; i < kPairs; ++i) {
    const int e = 2 * (tid + 256 * i) & (elems - 1);
    poff[i] = off_lo[e & 63] | off_hi[e >> 6];
    pto[i] = to_lo[e & 63] + to_hi[e >> 6];
  }
  uint64_t qoff[kQ];
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const int f = tid + 256 * i;
    qoff[i] = pdep_r((uint64_t)(f & (Y - 1)), d.qy) | pdep_r((uint64_t)(f / Y) & (ZT - 1), d.qz);
  }
  const uint64_t zstep = pdep_r((uint64_t)ZT, d.pz), qstep = pdep_r((uint64_t)ZT, d.qz);
  const int zchunks = 1 << (d.zb - d.zt);
  const int64_t xtiles = int64_t(1) << (d.xb - d.xt), units = xtiles * d.nb;
  const int x = tid & (XT - 1), part = tid >> d.xt, parts = XT < 256 ? 256 >> d.xt : 1;

  uint64_t ocol[Y];
#pragma unroll
  for (int y = 0; y < Y; ++y) ocol[y] = pdep_r((uint64_t)y, d.oy);
  const uint64_t orow = pdep_r((uint64_t)x & 255, d.ox);

  float4 p[kPairs];
  float2 q[kQ];
  auto load = [&](int64_t u, uint64_t zp, uint64_t zq) {
    const int64_t b = u >> (d.xb - d.xt);
    const float2* P = d.P + b * d.sP + (pdep_r((uint64_t)(u & (xtiles - 1)) << d.xt, d.px) | zp);
    const float2* Q = d.Q + b * d.sQ + zq;
#pragma unroll
    for (int i = 0; i < kPairs; ++i)
      if (2 * (tid + 256 * i) < elems) p[i] = *reinterpret_cast<const float4*>(P + poff[i]);
#pragma unroll
    for (int i = 0; i < kQ; ++i)
      if (tid + 256 * i < ZT * Y) q[i] = Q[qoff[i]];
  };
  int64_t u = blockIdx.x;
  uint64_t zp = 0, zq = 0;
  if (u < units) load(u, 0, 0);
  for (; u < units; u += gridDim.x) {
    float2* O = d.out + (u >> (d.xb - d.xt)) * d.sO + pdep_r((uint64_t)(u & (xtiles - 1)) << d.xt, d.ox);
    float2 sum[Y];
#pragma unroll
    for (int y = 0; y < Y; ++y) sum[y] = make_float2(0.f, 0.f);
    for (int c = 0; c < zchunks; ++c) {
      __syncthreads();  // the tile before is no longer read
#pragma unroll
      for (int i = 0; i < kPairs; ++i)
        if (2 * (tid + 256 * i) < elems) {
          Ps[pto[i]] = make_float2(p[i].x, d.conj_p ? -p[i].y : p[i].y);
          Ps[pto[i] + step] = make_float2(p[i].z, d.conj_p ? -p[i].w : p[i].w);
        }
#pragma unroll
      for (int i = 0; i < kQ; ++i)
        if (tid + 256 * i < ZT * Y) Qs[tid + 256 * i] = make_float2(q[i].x, d.conj_q ? -q[i].y : q[i].y);
      zp = madd_r(zp, zstep, d.pz);  // back at 0 after the last
      zq = madd_r(zq, qstep, d.qz);
      const int64_t next = c + 1 < zchunks ? u : u + gridDim.x;
      if (next < units) load(next, zp, zq);
      __syncthreads();
      // rows past the 256th only where one tile holds the sum: row by row
      for (int x0 = 0; x0 < XT; x0 += 256) {
        float2 acc[Y];
#pragma unroll
        for (int y = 0; y < Y; ++y) acc[y] = make_float2(0.f, 0.f);
#pragma unroll(Y > 4 ? 1 : 4)
        for (int z = part; z < ZT; z += parts) {
          const float2 a = Ps[z * stride + x0 + (x & 255)];
#pragma unroll
          for (int y = 0; y < Y; ++y) {
            const float2 b = Qs[z * Y + y];
            acc[y].x += fmaf(a.x, b.x, -(a.y * b.y));
            acc[y].y += fmaf(a.y, b.x, a.x * b.y);
          }
        }
        if (XT > 256) {
          float2* R = O + (pdep_r((uint64_t)x0, d.ox) | orow);
#pragma unroll
          for (int y = 0; y < Y; ++y) R[ocol[y]] = acc[y];
        } else {
#pragma unroll
          for (int y = 0; y < Y; ++y) {
            sum[y].x += acc[y].x;
            sum[y].y += acc[y].y;
          }
        }
      }
    }
    if (XT > 256) continue;
    if (parts > 1) {
      __syncthreads();
#pragma unroll
      for (int y = 0; y < Y; ++y) Ps[(part * Y + y) * XT + x] = sum[y];
      __syncthreads();
    }
    if (parts > 1) {
      for (int o = tid; o < XT * Y; o += 256) {
        const int r = o / Y, y = o & (Y - 1);
        float2 v = make_float2(0.f, 0.f);
        for (int w = 0; w < parts; ++w) {
          const float2 s = Ps[(w * Y + y) * XT + r];
          v.x += s.x;
          v.y += s.y;
        }
        O[pdep_r((uint64_t)r, d.ox) | pdep_r((uint64_t)y, d.oy)] = v;
      }
    } else {
#pragma unroll
      for (int y = 0; y < Y; ++y) O[orow | ocol[y]] = sum[y];
    }
  }
}

}  // namespace

// Rows from P when it has at most 16 columns to multiply, else from Q.
bool rowsum_fits(const GenericDesc& g, RowsumDesc& d) {
  const bool swap = g.yb() > 4;
  d.xb = swap ? g.yb() : g.xb();
  d.yb = swap ? g.xb() : g.yb();
  d.zb = g.zb();
  if (d.yb > 4 || d.xb + d.zb < 6 || d.xb + d.zb > 31) return false;
  d.P = swap ? g.Q : g.P;
  d.Q = swap ? g.P : g.Q;
  d.sP = swap ? g.sQ : g.sP;
  d.sQ = swap ? g.sP : g.sQ;
  d.px = swap ? g.qy : g.px;
  d.pz = swap ? g.qz : g.pz;
  d.qy = swap ? g.px : g.qy;
  d.qz = swap ? g.pz : g.qz;
  d.ox = swap ? g.oy : g.ox;
  d.oy = swap ? g.ox : g.oy;
  d.out = g.out;
  d.sO = g.sO;
  d.conj_p = swap && g.conjQ();
  d.conj_q = !swap && g.conjQ();
  d.nb = g.nb;
  // 64 rows, more where the sum is short; fewer, down to 16, while the tiles of
  // rows are below four a CU
  d.xt = std::min(d.xb, d.zb <= 2 ? kTile - d.zb : std::min(8, std::max(6, kTile - d.zb)));
  while (d.xt > 4 && (int64_t(d.nb) << (d.xb - d.xt)) < 1024) --d.xt;
  d.zt = std::min(d.zb, std::min(kTile - d.xt, 10 - d.yb));
  uint64_t mx = 0, mz = 0, rx = d.px, rz = d.pz;
  for (int j = 0; j < d.xt; ++j, rx &= rx - 1) mx |= rx & (0 - rx);
  for (int j = 0; j < d.zt; ++j, rz &= rz - 1) mz |= rz & (0 - rz);
  d.tile = mx | mz;
  // pairs of neighbours: the lowest address bit is the tile's
  return (d.tile & 1) && (int64_t(d.nb) << (d.xb - d.xt)) >= 256;
}

void launch_rowsum(const RowsumDesc& d, hipStream_t st) {
  const dim3 grid((unsigned)std::min<int64_t>(int64_t(d.nb) << (d.xb - d.xt), 2048));
  switch (d.yb) {
    case 0: hipLaunchKernelGGL(k_rowsum<1>, grid, dim3(256), 0, st, d); break;
    case 1: hipLaunchKernelGGL(k_rowsum<2>, grid, dim3(256), 0, st, d); break;
    case 2: hipLaunchKernelGGL(k_rowsum<4>, grid, dim3(256), 0, st, d); break;
    case 3: hipLaunchKernelGGL(k_rowsum<8>, grid, dim3(256), 0, st, d); break;
    default: hipLaunchKernelGGL(k_rowsum<16>, grid, dim3(256), 0, st, d); break;
  }
}

}  // namespace ltn
