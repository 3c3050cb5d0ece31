// SELM coupling kernels (Sec. "Discretization of SELM Hydrodynamic Coupling Tensor"; Sec.
// "Generation of the Stochastic Driving Fields Accounting for Thermal Fluctuations").
//
// Velocity fields are three cell-centred components, natural layout [3][nz][ny][nx].  The
// discrete divergence is D u = delta_x u_x + delta_y u_y + delta_z u_z with delta_x, delta_y the
// periodic forward differences and delta_z = a_z^{1/2} (the symmetric square root of the 1D
// wall operator, a dense nz x nz table S), so that D D^T = A and the projection
// P = I - D^T A^-1 D commutes with the viscous operator.  Gamma interpolates with Peskin's
// 4-point function (cells beyond a no-slip wall are antisymmetric ghosts of their mirrors).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.hpp"
#include "selm.hpp"

namespace smg {
namespace {

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + TPB - 1) / TPB); }

// The wall transform S v down the z columns: acc[j] = sum_k S[z0 + j][k] v[k][col], the terms in
// the order of k.  A lane carries ZT layers of its column, so an entry of v is loaded once per
// ZT products, and the rows of S (uniform over a wave) come through the scalar cache, KU entries
// of each row at a time.  The four waves of a work-group take the same 64 columns, ZT layers
// each, and share the columns' lines in the CU's cache.  128^3 (537 MFLOP): 45-48 us a call, bound
// by the latency of the scalar loads (with the next entries of v prefetched 57-61 us); one output
// a thread loaded each entry of v for one product and took 249-264 us.
constexpr int kSelmKU = 4;
template <int ZT>
__device__ __forceinline__ void wall_transform(double (&acc)[ZT], const double* __restrict__ v,
                                               const double* S, int z0, int nz, size_t plane) {
  typedef const __attribute__((address_space(4))) double* cptr;
  const cptr R = (cptr)(S + (size_t)z0 * nz);
#pragma unroll
  for (int j = 0; j < ZT; ++j) acc[j] = 0.0;
  int k = 0;
  for (; k + kSelmKU <= nz; k += kSelmKU) {
    double c[kSelmKU];
#pragma unroll
    for (int q = 0; q < kSelmKU; ++q) c[q] = v[(size_t)(k + q) * plane];
#pragma unroll
    for (int q = 0; q < kSelmKU; ++q)
#pragma unroll
      for (int j = 0; j < ZT; ++j) acc[j] = fma(R[j * nz + k + q], c[q], acc[j]);
  }
  for (; k < nz; ++k) {
    const double c = v[(size_t)k * plane];
#pragma unroll
    for (int j = 0; j < ZT; ++j) acc[j] = fma(R[j * nz + k], c, acc[j]);
  }
}

// This thread's (x, y) column and first layer; false beyond the columns or layers.
template <int ZT>
__device__ __forceinline__ bool wall_tile(int nx, int ny, int nz, uint32_t& col, int& z0) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  col = blockIdx.x * 64 + (threadIdx.x & 63);
  z0 = ((int)blockIdx.y * (TPB / 64) + wave) * ZT;
  return z0 < nz && col < (uint32_t)nx * ny;
}

// div = D u
template <int ZT>
__global__ __launch_bounds__(TPB) void k_selm_div(double* __restrict__ div,
                                                   const double* __restrict__ u,
                                                   const double* __restrict__ S, int nx, int ny,
                                                   int nz, double inv_h) {
  uint32_t col;
  int z0;
  if (!wall_tile<ZT>(nx, ny, nz, col, z0)) return;
  const size_t plane = (size_t)nx * ny, N = plane * nz;
  double acc[ZT];
  wall_transform<ZT>(acc, u + 2 * N + col, S, z0, nz, plane);
  const int y = (int)(col / nx), x = (int)(col - (uint32_t)y * nx);
  const uint32_t xp = col - x + (x + 1 == nx ? 0 : x + 1);
  const uint32_t yp = (uint32_t)(y + 1 == ny ? 0 : y + 1) * nx + x;
#pragma unroll
  for (int j = 0; j < ZT; ++j) {
    const size_t o = (size_t)(z0 + j) * plane;
    const double *ux = u + o, *uy = u + N + o;
    double d = (ux[xp] - ux[col]) * inv_h;
    d += (uy[yp] - uy[col]) * inv_h;
    div[o + col] = d + acc[j];
  }
}

// out = u - D^T p: delta_x^T p = (p[x-1] - p[x]) / h, the same in y, and S p in z (S symmetric)
// (out may be u: each thread reads and writes the same entries)
template <int ZT>
__global__ __launch_bounds__(TPB) void k_selm_grad_sub(double* out, const double* u,
                                                        const double* __restrict__ p,
                                                        const double* __restrict__ S, int nx,
                                                        int ny, int nz, double inv_h) {
  uint32_t col;
  int z0;
  if (!wall_tile<ZT>(nx, ny, nz, col, z0)) return;
  const size_t plane = (size_t)nx * ny, N = plane * nz;
  double acc[ZT];
  wall_transform<ZT>(acc, p + col, S, z0, nz, plane);
  const int y = (int)(col / nx), x = (int)(col - (uint32_t)y * nx);
  const uint32_t xm = col - x + (x == 0 ? nx - 1 : x - 1);
  const uint32_t ym = (uint32_t)(y == 0 ? ny - 1 : y - 1) * nx + x;
#pragma unroll
  for (int j = 0; j < ZT; ++j) {
    const size_t o = (size_t)(z0 + j) * plane;
    const double* P = p + o;
    const double pc = P[col];
    const size_t i = o + col;
    const double u0 = u[i], u1 = u[N + i], u2 = u[2 * N + i];
    out[i] = u0 - (P[xm] - pc) * inv_h;
    out[N + i] = u1 - (P[ym] - pc) * inv_h;
    out[2 * N + i] = u2 - acc[j];
  }
}

// Peskin's 4-point immersed-boundary function phi(r)
__device__ __forceinline__ double peskin4(double r) {
  r = fabs(r);
  if (r < 1.0) return (3.0 - 2.0 * r + sqrt(1.0 + 4.0 * r - 4.0 * r * r)) * 0.125;
  if (r < 2.0) return (5.0 - 2.0 * r - sqrt(-7.0 + 12.0 * r - 4.0 * r * r)) * 0.125;
  return 0.0;
}

// The stencil cell q = 0..63 of a point (4 x 4 x 4 cells from the first cell whose centre is
// within two widths) and its weight; a cell beyond a wall folds onto its mirror with a minus
// sign (antisymmetric ghost).
struct StencilCell {
  int64_t cell;
  double w;
};
__device__ __forceinline__ StencilCell stencil_cell(const double* __restrict__ X, int k, int q,
                                                    int nx, int ny, int nz, double inv_h) {
  const double px = X[3 * k] * inv_h, py = X[3 * k + 1] * inv_h, pz = X[3 * k + 2] * inv_h;
  const int ix = (int)floor(px - 0.5) - 1 + (q & 3);
  const int iy = (int)floor(py - 0.5) - 1 + ((q >> 2) & 3);
  int iz = (int)floor(pz - 0.5) - 1 + (q >> 4);
  double w = peskin4(ix + 0.5 - px) * peskin4(iy + 0.5 - py) * peskin4(iz + 0.5 - pz);
  if (iz < 0) {
    iz = -1 - iz;
    w = -w;
  } else if (iz >= nz) {
    iz = 2 * nz - 1 - iz;
    w = -w;
  }
  if (iz < 0 || iz >= nz) {  // a point outside the channel: no weight, no access out of range
    iz = 0;
    w = 0.0;
  }
  const int jx = ((ix % nx) + nx) % nx, jy = ((iy % ny) + ny) % ny;
  StencilCell s;
  s.cell = ((int64_t)iz * ny + jy) * nx + jx;
  s.w = w;
  return s;
}

// f += scale * Gamma^T F (one thread per (point, stencil cell); points may share cells, so the
// adds are atomic)
__global__ __launch_bounds__(TPB) void k_selm_spread(double* __restrict__ f,
                                                      const double* __restrict__ X,
                                                      const double* __restrict__ F, int m, int nx,
                                                      int ny, int nz, double inv_h, double scale) {
  const int t = blockIdx.x * TPB + threadIdx.x;
  if (t >= 64 * m) return;
  const int k = t >> 6, q = t & 63;
  const StencilCell s = stencil_cell(X, k, q, nx, ny, nz, inv_h);
  const int64_t N = (int64_t)nx * ny * nz;
  for (int c = 0; c < 3; ++c) atomicAdd(&f[c * N + s.cell], scale * s.w * F[3 * k + c]);
}

// V = scale * Gamma u: one wave per point, lane q = stencil cell, sums by a fixed shuffle tree
__global__ __launch_bounds__(TPB) void k_selm_interp(double* __restrict__ V,
                                                      const double* __restrict__ X,
                                                      const double* __restrict__ u, int m, int nx,
                                                      int ny, int nz, double inv_h, double scale) {
  const int k = (blockIdx.x * TPB + threadIdx.x) >> 6;
  const int q = threadIdx.x & 63;
  if (k >= m) return;
  const StencilCell s = stencil_cell(X, k, q, nx, ny, nz, inv_h);
  const int64_t N = (int64_t)nx * ny * nz;
  double v[3];
  for (int c = 0; c < 3; ++c) v[c] = s.w * u[c * N + s.cell];
  for (int off = 32; off >= 1; off >>= 1)
    for (int c = 0; c < 3; ++c) v[c] += __shfl_xor(v[c], off, 64);
  if (q == 0)
    for (int c = 0; c < 3; ++c) V[3 * k + c] = scale * v[c];
}

// X += dt V + sqrt(dt) g (Euler-Maruyama)
__global__ __launch_bounds__(TPB) void k_selm_em(double* __restrict__ X,
                                                  const double* __restrict__ V,
                                                  const double* __restrict__ g, int n, double dt,
                                                  double sdt) {
  const int i = blockIdx.x * TPB + threadIdx.x;
  if (i < n) X[i] = X[i] + dt * V[i] + sdt * g[i];
}

}  // namespace

// Runs go with the layers per lane and the grid of a wall transform: the most of 8, 4, 2 and 1
// that divides nz, so that no tile overhangs (16 layers need more scalar registers for S than a
// wave has).
template <typename F>
static hipError_t with_wall_tile(int nx, int ny, int nz, F go) {
  auto run = [&](auto zt) {
    constexpr int ZT = decltype(zt)::value;
    constexpr int per = ZT * (TPB / 64);
    go(zt, dim3((unsigned)(((int64_t)nx * ny + 63) / 64), (unsigned)((nz + per - 1) / per)));
  };
  if (nz % 8 == 0) run(std::integral_constant<int, 8>());
  else if (nz % 4 == 0) run(std::integral_constant<int, 4>());
  else if (nz % 2 == 0) run(std::integral_constant<int, 2>());
  else run(std::integral_constant<int, 1>());
  return hipGetLastError();
}

hipError_t launch_selm_div(double* div, const double* u, const double* S, int nx, int ny, int nz,
                           double h, hipStream_t s) {
  return with_wall_tile(nx, ny, nz, [&](auto zt, dim3 grid) {
    k_selm_div<decltype(zt)::value><<<grid, TPB, 0, s>>>(div, u, S, nx, ny, nz, 1.0 / h);
  });
}

hipError_t launch_selm_grad_sub(double* out, const double* u, const double* p, const double* S,
                                int nx, int ny, int nz, double h, hipStream_t s) {
  return with_wall_tile(nx, ny, nz, [&](auto zt, dim3 grid) {
    k_selm_grad_sub<decltype(zt)::value><<<grid, TPB, 0, s>>>(out, u, p, S, nx, ny, nz, 1.0 / h);
  });
}

hipError_t launch_selm_spread(double* f, const double* X, const double* F, int m, int nx, int ny,
                              int nz, double h, double scale, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  k_selm_spread<<<blocks_for(64 * (int64_t)m), TPB, 0, s>>>(f, X, F, m, nx, ny, nz, 1.0 / h,
                                                           scale);
  return hipGetLastError();
}

hipError_t launch_selm_interp(double* V, const double* X, const double* u, int m, int nx, int ny,
                              int nz, double h, double scale, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  k_selm_interp<<<blocks_for(64 * (int64_t)m), TPB, 0, s>>>(V, X, u, m, nx, ny, nz, 1.0 / h,
                                                           scale);
  return hipGetLastError();
}

hipError_t launch_selm_em(double* X, const double* V, const double* g, int n, double dt,
                          hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_selm_em<<<blocks_for(n), TPB, 0, s>>>(X, V, g, n, dt, sqrt(dt));
  return hipGetLastError();
}

}  // namespace smg
