// Device helpers shared by the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "philox.hpp"

namespace smg {

constexpr int TPB = 256;

__device__ __forceinline__ int wrapm(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// Quotient and remainder by d, using a shift when d is a power of two (lg2 >= 0).
__device__ __forceinline__ uint32_t udiv(uint32_t a, uint32_t d, int lg2) {
  return lg2 >= 0 ? (a >> lg2) : a / d;
}

// 1D prolongation weights for the fine cells 2J-1, 2J, 2J+1, 2J+2 around coarse cell J.
template <typename T = double>
__device__ __forceinline__ T pw(int i) { return (i == 1 || i == 2) ? T(0.75) : T(0.25); }

// XCD-aware work-group numbering.  The dispatcher deals work-groups to the 8 XCDs round-robin
// by linear id, and each XCD has its own L2.  Renumbering so that XCD k runs the k-th
// contiguous eighth of the grid keeps neighbouring tiles (which share halo rows and planes)
// on one L2.  A bijection on [0, total); the ragged tail beyond a multiple of 8 keeps its ids.
constexpr uint32_t kXcds = 8;
struct Blk3 {
  uint32_t x, y, z;
};
__device__ __forceinline__ Blk3 xcd_block() {
  const uint32_t gx = gridDim.x, gy = gridDim.y, gz = gridDim.z;
  const uint32_t total = gx * gy * gz;
  uint32_t lin = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const uint32_t per = total / kXcds;
  if (lin < per * kXcds) lin = (lin % kXcds) * per + lin / kXcds;
  Blk3 b;
  b.x = lin % gx;
  const uint32_t r = lin / gx;
  b.y = r % gy;
  b.z = r / gy;
  return b;
}

// q = v / d, r = v % d for v >= 0 and a wave-uniform d > 0: a shift and a mask when d is a power
// of two (the usual level extents), else the division.
__device__ __forceinline__ void divmod_uniform(int v, int d, int& q, int& r) {
  if ((d & (d - 1)) == 0) {
    const int lg = __builtin_ctz((unsigned)d);
    q = v >> lg;
    r = v & (d - 1);
  } else {
    q = v / d;
    r = v - q * d;
  }
}

// Periodic index of a staged halo position: v mod n for -n <= v < 2n.  A tile that overhangs
// a small level may stage positions further out; no cell inside the level reads them (a
// stencil reaches at most two cells, and n >= 4), so they are clamped into range instead of
// reduced by a division.
__device__ __forceinline__ int wrap_near(int v, int n) {
  if (v < 0) v += n;
  if (v >= n) v -= n;
  return v < n ? v : n - 1;
}

// Sum over the work-group of TPB threads in a fixed order (the total is in thread 0): the 64 lanes
// of a wave by exchanges, the waves through sh.  Called by every thread, once per use of sh.
__device__ __forceinline__ double block_sum(double v, double (&sh)[TPB / 64]) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// The two in-plane sums of a cell's row of A on a Galerkin level, p0 = (m_y (x) m_x) x and p1 =
// (a_y (x) m_x + m_y (x) a_x) x over the 5 x 5 window of plane P, in index order.  The Galerkin
// operator of the wall-bounded Laplacian is a Kronecker sum, A = a_z (x) m_y (x) m_x + m_z (x)
// (a_y (x) m_x + m_y (x) a_x), with 5-point periodic 1D stencils s1d = (m_x, a_x, m_y, a_y)
// (offsets -2..2, uniform over the level): each row of the plane is reduced with m_x and a_x, then
// the plane with m_y and a_y, 65 FMAs.  P is a tile in LDS, element ys[dy] * sy + xs[dx].
template <typename T>
__device__ __forceinline__ T gal_plane(const T* __restrict__ P, int sy, const int* xs,
                                       const int* ys, const T* s1d, T& p1) {
  T q0[5], q1[5];
#pragma unroll
  for (int dy = 0; dy < 5; ++dy) {
    const T* row = P + (size_t)ys[dy] * sy;
    T sm = 0, sa = 0;
#pragma unroll
    for (int dx = 0; dx < 5; ++dx) {
      const T v = row[xs[dx]];
      sm = fma(s1d[dx], v, sm);
      sa = fma(s1d[5 + dx], v, sa);
    }
    q0[dy] = sm;
    q1[dy] = sa;
  }
  T p0 = 0, pa = 0, pb = 0;
#pragma unroll
  for (int dy = 0; dy < 5; ++dy) {
    p0 = fma(s1d[10 + dy], q0[dy], p0);
    pa = fma(s1d[15 + dy], q0[dy], pa);
    pb = fma(s1d[10 + dy], q1[dy], pb);
  }
  p1 = pa + pb;
  return p0;
}

// b_c = P^T r at coarse cell (X,Y,Z): 4x4x4 fine window 2J-1..2J+2 per axis, weights
// (1/4, 3/4, 3/4, 1/4); on the wall axis the fine cell next to a wall carries 1/2.
template <typename T>
__device__ __forceinline__ T restrict_at(const T* __restrict__ R, int sy, int sz, int nxf, int nyf,
                                         int nzf, int X, int Y, int Z) {
  const int nzc = nzf >> 1;
  T acc = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int zf = 2 * Z - 1 + c;
    if (zf < 0 || zf >= nzf) continue;
    T wz = pw<T>(c);
    if ((Z == 0 && zf == 0) || (Z == nzc - 1 && zf == nzf - 1)) wz = T(0.5);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int yf = wrapm(2 * Y - 1 + b, nyf);
      const T* Rr = R + (size_t)zf * sz + (size_t)yf * sy;
      T s = 0;
#pragma unroll
      for (int a = 0; a < 4; ++a) s = fma(pw<T>(a), Rr[wrapm(2 * X - 1 + a, nxf)], s);
      acc = fma(wz * pw<T>(b), s, acc);
    }
  }
  return acc;
}

// (P e) at fine cell (xf, yf, zf): trilinear, 3/4 to the own parent and 1/4 to the next one;
// beyond a wall the ghost parent carries -e, so the wall-layer cell gets 1/2 e.
template <typename T>
__device__ __forceinline__ T prolong_at(const T* __restrict__ E, int sy, int sz, int xf, int yf,
                                        int zf, int nxc, int nyc, int nzc) {
  const int X0 = xf >> 1, Y0 = yf >> 1, Z0 = zf >> 1;
  const int X1 = wrapm((xf & 1) ? X0 + 1 : X0 - 1, nxc);
  const int Y1 = wrapm((yf & 1) ? Y0 + 1 : Y0 - 1, nyc);
  int Z1 = (zf & 1) ? Z0 + 1 : Z0 - 1;
  T wz0 = T(0.75), wz1 = T(0.25);
  if (Z1 < 0 || Z1 >= nzc) {
    wz0 = T(0.5);
    wz1 = T(0);
    Z1 = Z0;
  }
  const T* r00 = E + (size_t)Z0 * sz + (size_t)Y0 * sy;
  const T* r01 = E + (size_t)Z0 * sz + (size_t)Y1 * sy;
  const T* r10 = E + (size_t)Z1 * sz + (size_t)Y0 * sy;
  const T* r11 = E + (size_t)Z1 * sz + (size_t)Y1 * sy;
  const T q = T(0.75), o = T(0.25);
  const T p0 = q * (q * r00[X0] + o * r00[X1]) + o * (q * r01[X0] + o * r01[X1]);
  const T p1 = q * (q * r10[X0] + o * r10[X1]) + o * (q * r11[X0] + o * r11[X1]);
  return wz0 * p0 + wz1 * p1;
}

}  // namespace smg
