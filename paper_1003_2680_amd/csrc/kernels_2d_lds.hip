// LDS-resident kernels of the two-dimensional sampler: several level-0 sweeps (with the transfers
// beside them) per launch on strips of rows, and the bottom of the V-cycle in one work-group per
// chain.  Fields: natural layout [ncomp][nz][nx], float64; operators as in kernels2d.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "block_update.hpp"
#include "device_common.hpp"
#include "kernels2d.hpp"

namespace smg {
namespace {

// ---------------------------------------------------------------------------------- level 0
// Up to kMaxPoint2 point passes of level 0 in one launch, with the prolongation in front of them
// or the residual restriction behind.  A pass reads one row beyond the cells it draws, so a work-
// group that owns `rows` rows starts from a window of halo rows on either side (one per pass, two
// more for the restriction) and every pass draws one row less at each end; the rows outside its
// own are drawn again by their owners from the same inputs and noise.  Since a group's window
// holds rows that others write, x is read from one field and written to another.
//
// What bounds it: the launch on small grids (128 x 128 x 8 chains: four passes and the transfer
// beside them 12 us; in six launches they took 31 us, most of it launch and load latency), the
// noise arithmetic of the redrawn rows on large ones.
constexpr int P2_TPB = 512;

struct Window2 {
  int lo, hi;  // rows held in LDS
};
__device__ __forceinline__ Window2 window2(int z0, int rows, int halo, int nz) {
  return Window2{max(z0 - halo, 0), min(z0 + rows + halo, nz)};
}

// -h^2 (A x) at a cell as a sum of differences to its neighbours (nw: its walls).  On tall grids the
// field is smooth and large, and the differences keep the digits that 4 x - (sum of neighbours)
// rounds away: over 24 grids of 16 to 244 rows the samples and states are off by 5.0e-15 in the mean
// with that form and by 4.0e-15 with this one (512 x 512 x 64 chains take 1 % more).
__device__ __forceinline__ double laplace(const double* row, int x, int nx, bool below, bool above,
                                          int& nw) {
  const double c = row[x];
  const double l = row[x == 0 ? nx - 1 : x - 1] - c, r = row[x + 1 == nx ? 0 : x + 1] - c;
  const double d = below ? row[x - nx] - c : -2.0 * c, u = above ? row[x + nx] - c : -2.0 * c;
  nw = (below ? 0 : 1) + (above ? 0 : 1);
  return (l + r) + (d + u);
}

template <bool NOISE>
__global__ __launch_bounds__(P2_TPB) void k2_level0(Point2Args a, NoiseArgs na) {
  extern __shared__ double xs[];
  const uint32_t comp = blockIdx.y;
  const int nx = a.nx, nz = a.nz, nh = nx >> 1;
  const int64_t N = (int64_t)nx * nz;
  const int z0 = blockIdx.x * a.rows, z1 = min(z0 + a.rows, nz);
  const int halo = a.npass + (a.bc ? 2 : 0);
  const Window2 w = window2(z0, a.rows, halo, nz);
  const double* src = a.src + comp * N;
  const double* B = a.b ? a.b + comp * N : nullptr;
  for (int q = threadIdx.x; q < (w.hi - w.lo) * nx; q += P2_TPB) {
    double v = src[(int64_t)w.lo * nx + q];
    if (a.e) {  // x += P e (bilinear on cell centres, the wall ghost -c)
      int zr, x;
      divmod_uniform(q, nx, zr, x);
      const int z = w.lo + zr, nxc = nx >> 1, nzc = nz >> 1;
      const int X0 = x >> 1, Z0 = z >> 1;
      const int X1 = wrapm((x & 1) ? X0 + 1 : X0 - 1, nxc);
      int Z1 = (z & 1) ? Z0 + 1 : Z0 - 1;
      double wz0 = 0.75, wz1 = 0.25;
      if (Z1 < 0 || Z1 >= nzc) {
        wz0 = 0.5;
        wz1 = 0.0;
        Z1 = Z0;
      }
      const double* E = a.e + (int64_t)comp * nxc * nzc;
      const double r0 = 0.75 * E[(int64_t)Z0 * nxc + X0] + 0.25 * E[(int64_t)Z0 * nxc + X1];
      const double r1 = 0.75 * E[(int64_t)Z1 * nxc + X0] + 0.25 * E[(int64_t)Z1 * nxc + X1];
      v += wz0 * r0 + wz1 * r1;
    }
    xs[q] = v;
  }
  __syncthreads();
  for (int p = 0; p < a.npass; ++p) {
    const int colour = a.post ? 1 - (p & 1) : p & 1;
    const uint32_t sid =
        (na.sid & ~0xFFFFF0u) | ((uint32_t)(a.slot0 + (p >> 1)) << 4) | ((uint32_t)colour << 12);
    // rows drawn: one less per pass at each end that is not a wall
    const int left = halo - 1 - p;
    const int a0 = max(z0 - left, 0), a1 = min(z0 + a.rows + left, nz);
    // sites a0 nh .. a1 nh - 1 of the colour; call q holds sites 2q and 2q + 1
    const int s0 = a0 * nh, s1 = a1 * nh;
    for (int q = (s0 >> 1) + threadIdx.x; 2 * q < s1; q += P2_TPB) {
      double zn[2] = {0.0, 0.0};
      if (NOISE) normal_pair(na, sid, comp, (uint32_t)q, zn[0], zn[1]);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int s = 2 * q + t;
        if (s < s0 || s >= s1) continue;
        int z, j;
        divmod_uniform(s, nh, z, j);
        const int x = 2 * j + ((colour + z) & 1);
        const double* row = xs + (z - w.lo) * nx;
        int nw;
        const double x0 = row[x], lap = laplace(row, x, nx, z > 0, z + 1 < nz, nw);
        double v = lap * a.ih2;
        if (B) v += B[(int64_t)z * nx + x];
        v = fma(v, a.inv_d[nw], x0);
        if (NOISE) v = fma(a.sig[nw], zn[t], v);
        xs[(z - w.lo) * nx + x] = v;
      }
    }
    __syncthreads();
  }
  double* dst = a.dst + comp * N;
  for (int q = threadIdx.x; q < (z1 - z0) * nx; q += P2_TPB) {
    const double v = xs[(z0 - w.lo) * nx + q];
    dst[(int64_t)z0 * nx + q] = v;
    if (a.out) a.out[comp * N + (int64_t)z0 * nx + q] = v;
  }
  if (!a.bc) return;
  // b_c = P^T (b - A x) for the coarse rows of the owned pairs of rows, and x_c = 0
  const int nxc = nx >> 1, nzc = nz >> 1;
  for (int q = threadIdx.x; q < ((z1 - z0) >> 1) * nxc; q += P2_TPB) {
    int Zr, X;
    divmod_uniform(q, nxc, Zr, X);
    const int Z = (z0 >> 1) + Zr;
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int z = 2 * Z - 1 + i;
      if (z < 0 || z >= nz) continue;
      double wz = pw(i);
      if ((Z == 0 && z == 0) || (Z == nzc - 1 && z == nz - 1)) wz = 0.5;
      const double* row = xs + (z - w.lo) * nx;
      double s = 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int x = wrapm(2 * X - 1 + c, nx);
        int nw;
        double r = laplace(row, x, nx, z > 0, z + 1 < nz, nw) * a.ih2;
        if (B) r += B[(int64_t)z * nx + x];
        s = fma(pw(c), r, s);
      }
      acc = fma(wz, s, acc);
    }
    const int64_t at = (int64_t)comp * nxc * nzc + (int64_t)Z * nxc + X;
    a.bc[at] = acc;
    if (a.xc) a.xc[at] = 0.0;
  }
}

// ------------------------------------------------------------------- noise of the bottom levels
// One thread per 2 x 2 block and sweep: the block's four normals (calls 2 bid, 2 bid + 1) as
// sqrt(kT) L_BB^-T n in the level's layout.  Grid: blocks of the largest level, levels, slot *
// ncomp + component.
__global__ __launch_bounds__(TPB) void k2_noise(const Bot2Args* __restrict__ ap, NoiseArgs na) {
  const Bot2Args& a = *ap;
  const Bot2Level& L = a.lv[blockIdx.y];
  const uint32_t slot = blockIdx.z / (uint32_t)a.ncomp, comp = blockIdx.z % (uint32_t)a.ncomp;
  const int nbx = L.nx >> 1, nblk = nbx * (L.nz >> 1);
  const int bid = blockIdx.x * TPB + threadIdx.x;
  if (L.kind != KIND_BLOCK || bid >= nblk) return;
  const int bz = bid / nbx, bx = bid - bz * nbx;
  const uint32_t colour = (bx & 1) + 2 * (bz & 1);
  const uint32_t sid = (uint32_t)(a.level0 + blockIdx.y) | (slot << 4) | (colour << 12);
  double n[4];
  normal_pair(na, sid, comp, 2 * (uint32_t)bid, n[0], n[1]);
  normal_pair(na, sid, comp, 2 * (uint32_t)bid + 1, n[2], n[3]);
  const double* W = L.bfac + (int64_t)bz * 32 + 16;
  double* out = L.noise + ((int64_t)slot * a.ncomp + comp) * L.nx * L.nz;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    double e = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) e = fma(W[k * 4 + j], n[j], e);
    out[(int64_t)(2 * bz + (k >> 1)) * L.nx + 2 * bx + (k & 1)] = na.sqkT * e;
  }
}

// ------------------------------------------------------------------------------------ the bottom
// Every level from the bottom one down and back up, one work-group per chain, with x (rows with
// two periodic halo cells per side) and b in LDS, as the three-dimensional bottom: the passes are
// shaped for latency (DPP exchanges between a block's four lanes, lane bits kx, kz; immediate
// offsets into the rows; noise of the next pass loaded during this one).  At 128 x 128 x 8 chains
// the two halves take 31 us each and a cycle 6 launches and 100 us; with a launch per colour (4.9
// us) it was 51 launches and 237 us.
constexpr int B2_TPB = 1024;

// A x at a block's cell, shared by the two cells of a column: of their six rows 2 bz - 2 .. 2 bz
// + 3 the lane of cell row kz reduces rows 3 kz + m along x and weights them for its own cell and
// for its partner's (packed factors zw: own0, own1, oth0, oth1 of m = 0 .. 2 and a zero each).
struct Weights2 {
  double z[12], f[4];  // the lane's packed z-factors and its row of A_BB^-1 (lane order)
};
__device__ __forceinline__ void load_weights2(Weights2& w, const double* row, int kx, int kz) {
  const double* z = row + 16 + kz * 16;
  const double* F = row + (kx + 2 * kz) * 4;
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) w.z[q * 3 + m] = z[q * 4 + m];
#pragma unroll
  for (int m = 0; m < 4; ++m) w.f[m] = F[m];
}
__device__ __forceinline__ double bot2_update(const double* X, const int (&ro)[3],
                                              const double* s1d, const Weights2& w, int own,
                                              double bk, double noise) {
  double win[3][5];
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int d = 0; d < 5; ++d) win[m][d] = X[ro[m] + d];
  const double xk = X[own];
  double self = 0.0, part = 0.0;
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const double e = win[m][0] + win[m][4], d = win[m][1] + win[m][3], c = win[m][2];
    const double rm = fma(s1d[0], e, fma(s1d[1], d, s1d[2] * c));
    const double ra = fma(s1d[5], e, fma(s1d[6], d, s1d[7] * c));
    self = fma(w.z[m], rm, fma(w.z[3 + m], ra, self));
    part = fma(w.z[6 + m], rm, fma(w.z[9 + m], ra, part));
  }
  const double res = bk - (self + dpp_lane<DPP_XOR2>(part));
  double v0 = fma(w.f[0], res, xk), v1 = noise;
  v1 = fma(w.f[1], dpp_lane<DPP_XOR1>(res), v1);
  v0 = fma(w.f[2], dpp_lane<DPP_XOR2>(res), v0);
  v1 = fma(w.f[3], dpp_lane<DPP_XOR3>(res), v1);
  return v0 + v1;
}

__device__ __forceinline__ void bot2_store(double* X, int p, int x, int nx, double v) {
  X[p] = v;
  if (x < 2) X[p + nx] = v;
  if (x >= nx - 2) X[p - nx] = v;
}

typedef const __attribute__((address_space(1))) double* gdbl;

template <bool NOISE>
__device__ __forceinline__ void bot2_sweeps(double* X, const double* B, const Bot2Level& L,
                                            const double* tab, int slot0, int nslot, bool post,
                                            gdbl Z, int64_t slot_stride) {
  if (nslot == 0) return;
  double s1d[10];
#pragma unroll
  for (int q = 0; q < 10; ++q) s1d[q] = L.s1d[q];
  const int nx = L.nx, nz = L.nz, RS = L.rs, nbz = nz >> 1, nbx2 = nx >> 2;
  const int tid = (int)threadIdx.x, kx = tid & 1, kz = (tid >> 1) & 1;
  const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);
  int i, j0;
  divmod_uniform(tid >> 2, nbx2, j0, i);
  const int x0 = 4 * i + kx;
  const int steps = 4 * nslot;
  auto layers = [&](int cz) { return (nbz + 1 - cz) >> 1; };
  auto colour_of = [&](int st) { return post ? 3 - (st & 3) : st & 3; };
  // rounds over a colour: block rows j0, j0 + stride, ... (levels of more than 256 blocks a colour)
  const int stride = (B2_TPB >> 2) / nbx2;
  const bool one = layers(0) <= stride;
  auto noise_at = [&](int st, int j) {
    const int c = colour_of(st), cx = c & 1, cz = c >> 1;
    const int z = 2 * (2 * (j < layers(cz) ? j : 0) + cz) + kz;
    return Z[(int64_t)(slot0 + (st >> 2)) * slot_stride + (z < nz ? z : 0) * nx + x0 + 2 * cx];
  };
  double next = 0.0;
  const bool lane_in = j0 < stride;  // lanes past the last whole block row
  if (NOISE && one) next = noise_at(0, j0);
  Weights2 w;  // shared by the two passes of a cz when a lane has one cell per pass
#pragma unroll 1
  for (int st = 0; st < steps; ++st) {
    const int c = colour_of(st), cx = c & 1, cz = c >> 1;
    const double cur = next;
    if (NOISE && one && st + 1 < steps) next = noise_at(st + 1, j0);
    const int nl = layers(cz);
    if (wave0 < 4 * nbx2 * min(nl, stride)) {
      for (int jb = 0; jb < nl; jb += stride) {
        const bool active = lane_in && jb + j0 < nl;
        const int bz = 2 * (active ? jb + j0 : 0) + cz, z = 2 * bz + kz;
        int ro[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          int r = 2 * bz - 2 + 3 * kz + m;
          r = r < 0 ? 0 : (r >= nz ? nz - 1 : r);  // beyond a wall: factor 0
          ro[m] = r * RS + x0 + 2 * cx;
        }
        if (!one || (st & 1) == 0) load_weights2(w, tab + nz * 10 + bz * 48, kx, kz);
        const int own = z * RS + x0 + 2 * cx + 2, cell = z * nx + x0 + 2 * cx;
        double n = cur;
        if (NOISE && !one) n = noise_at(st, jb + j0);
        const double v = bot2_update(X, ro, s1d, w, own, B[cell], n);
        if (active) bot2_store(X, own, x0 + 2 * cx, nx, v);
      }
    }
    __syncthreads();
  }
}

// r = b - A x for rows za .. zb - 1 into R (row za first)
__device__ __forceinline__ void bot2_residual(double* R, const double* X, const double* B,
                                              const Bot2Level& L, const double* tab, int za,
                                              int zb) {
  const int nx = L.nx, nz = L.nz;
  for (int q = threadIdx.x; q < (zb - za) * nx; q += B2_TPB) {
    int zr, x;
    divmod_uniform(q, nx, zr, x);
    const int z = za + zr;
    const double* zt = tab + z * 10;
    double acc = 0.0;
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      int r = z + m - 2;
      r = r < 0 ? 0 : (r >= nz ? nz - 1 : r);
      const double* v = X + r * L.rs + x;
      const double e = v[0] + v[4], d = v[1] + v[3], c = v[2];
      const double rm = fma(L.s1d[0], e, fma(L.s1d[1], d, L.s1d[2] * c));
      const double ra = fma(L.s1d[5], e, fma(L.s1d[6], d, L.s1d[7] * c));
      acc = fma(zt[m], rm, fma(zt[5 + m], ra, acc));
    }
    R[q] = B[z * nx + x] - acc;
  }
}

template <bool NOISE>
__global__ __launch_bounds__(B2_TPB) void k2_bottom(const Bot2Args* __restrict__ ap, int part,
                                                     NoiseArgs na) {
  extern __shared__ double sm2[];
  const Bot2Args& a = *ap;
  const uint32_t comp = blockIdx.x;
  const int tid = threadIdx.x;
  double* R = sm2 + a.r_off;
  // fields and tables ([zt nz*10][per block row: A_BB^-1 in lane order 16, packed z-factors 32])
  for (int i = 0; i < a.nlev; ++i) {
    const Bot2Level& L = a.lv[i];
    const int n = L.nx * L.nz, nx = L.nx, halo = L.kind == KIND_BLOCK ? 2 : 0;
    double* x = sm2 + L.x_off;
    double* b = sm2 + L.b_off;
    if (part != BOT_UP) {
      for (int q = tid; q < L.nz * L.rs; q += B2_TPB) x[q] = 0.0;
      if (i == 0) {
        const gdbl bg = (gdbl)L.bg + (int64_t)comp * n;
        for (int q = tid; q < n; q += B2_TPB) b[q] = bg[q];
      }
    } else {
      const gdbl xg = (gdbl)L.xg + (int64_t)comp * n, bg = (gdbl)L.bg + (int64_t)comp * n;
      for (int q = tid; q < n; q += B2_TPB) {
        int z, xx;
        divmod_uniform(q, nx, z, xx);
        if (L.kind == KIND_BLOCK) {
          bot2_store(x, z * L.rs + xx + halo, xx, nx, xg[q]);
          b[q] = bg[q];
        } else {
          x[q] = xg[q];
        }
      }
    }
    if (L.kind == KIND_BLOCK) {
      double* t = sm2 + L.tab_off;
      const gdbl src = (gdbl)L.tab;
      for (int q = tid; q < L.nz * 10 + (L.nz >> 1) * 48; q += B2_TPB) t[q] = src[q];
    } else if (NOISE && part == BOT_WHOLE) {
      // the normals of the coarsest draw, which depend on nothing above it
      const uint32_t sid = (uint32_t)(a.level0 + i) | (1u << 24);
      for (int q = tid; 2 * q < n; q += B2_TPB) {
        double z0, z1;
        normal_pair(na, sid, comp, (uint32_t)q, z0, z1);
        b[n + 2 * q] = z0;
        if (2 * q + 1 < n) b[n + 2 * q + 1] = z1;
      }
    }
  }
  __syncthreads();
  int last = a.nlev - 1;
  for (int i = 0; i < a.nlev && part != BOT_UP; ++i) {
    const Bot2Level& L = a.lv[i];
    const int n = L.nx * L.nz;
    double* x = sm2 + L.x_off;
    double* b = sm2 + L.b_off;
    if (part == BOT_DOWN && i > 0) {
      double* bg = L.bg + (int64_t)comp * n;
      for (int q = tid; q < n; q += B2_TPB) bg[q] = b[q];
    }
    if (L.kind == KIND_CHOL) {
      if (part == BOT_DOWN) return;
      // G lanes per row (a power of two, G <= 32) split the columns of the dense factors
      const gdbl ainv = (gdbl)a.ainv, wl = (gdbl)a.w;
      int G = 1;
      while (G < 32 && 2 * G * n <= B2_TPB) G *= 2;
      const int g = tid % G;
      for (int row = tid / G; row < n; row += B2_TPB / G) {
        double acc = 0.0, an = 0.0;
#pragma unroll 8
        for (int jj = g; jj < n; jj += G) {
          acc = fma(ainv[(int64_t)jj * n + row], b[jj], acc);
          if (NOISE && jj >= row) an = fma(wl[(int64_t)jj * n + row], b[n + jj], an);
        }
        for (int off = G / 2; off >= 1; off >>= 1) {
          acc += __shfl_xor(acc, off, G);
          if (NOISE) an += __shfl_xor(an, off, G);
        }
        if (NOISE) acc = fma(na.sqkT, an, acc);
        if (g == 0) x[row] = acc;
      }
      __syncthreads();
      last = i;
      break;
    }
    const double* tab = sm2 + L.tab_off;
    const gdbl Z = (gdbl)L.noise + (int64_t)comp * n;
    const int64_t zs = (int64_t)a.ncomp * n;
    bot2_sweeps<NOISE>(x, b, L, tab, 0, a.nu1, false, Z, zs);
    if (i == a.nlev - 1) {  // smoothing-only coarsest level: the post-sweeps follow at once
      bot2_sweeps<NOISE>(x, b, L, tab, a.nu1, a.nu2, true, Z, zs);
      last = i;
      break;
    }
    if (part == BOT_DOWN) {
      double* xg = L.xg + (int64_t)comp * n;
      for (int q = tid; q < n; q += B2_TPB) {
        int z, xx;
        divmod_uniform(q, L.nx, z, xx);
        xg[q] = x[z * L.rs + xx + 2];
      }
    }
    // b_{i+1} = P^T (b_i - A_i x_i), half of the coarse rows at a time (the residual of a half,
    // with a row beyond either end, fits the scratch field)
    const Bot2Level& C = a.lv[i + 1];
    double* bc = sm2 + C.b_off;
    const int half = (C.nz + 1) >> 1;
    for (int h = 0; h < 2; ++h) {
      const int Za = h * half, Zb = min(C.nz, Za + half);
      if (Zb <= Za) continue;
      const int za = max(2 * Za - 1, 0), zb = min(2 * Zb + 1, L.nz);
      bot2_residual(R, x, b, L, tab, za, zb);
      __syncthreads();
      for (int q = tid; q < (Zb - Za) * C.nx; q += B2_TPB) {
        int Zr, X;
        divmod_uniform(q, C.nx, Zr, X);
        const int Zc = Za + Zr;
        double acc = 0.0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int z = 2 * Zc - 1 + m;
          if (z < 0 || z >= L.nz) continue;
          double wz = pw(m);
          if ((Zc == 0 && z == 0) || (Zc == C.nz - 1 && z == L.nz - 1)) wz = 0.5;
          double s = 0.0;
#pragma unroll
          for (int d = 0; d < 4; ++d)
            s = fma(pw(d), R[(z - za) * L.nx + wrapm(2 * X - 1 + d, L.nx)], s);
          acc = fma(wz, s, acc);
        }
        bc[Zc * C.nx + X] = acc;
      }
      __syncthreads();
    }
  }
  for (int i = last - 1; i >= 0; --i) {
    const Bot2Level& L = a.lv[i];
    const Bot2Level& C = a.lv[i + 1];
    const int n = L.nx * L.nz;
    double* x = sm2 + L.x_off;
    const double* xc = sm2 + C.x_off + (C.kind == KIND_BLOCK ? 2 : 0);
    for (int q = tid; q < n; q += B2_TPB) {
      int z, xx;
      divmod_uniform(q, L.nx, z, xx);
      const int X0 = xx >> 1, Z0 = z >> 1;
      const int X1 = wrapm((xx & 1) ? X0 + 1 : X0 - 1, C.nx);
      int Z1 = (z & 1) ? Z0 + 1 : Z0 - 1;
      double wz0 = 0.75, wz1 = 0.25;
      if (Z1 < 0 || Z1 >= C.nz) {
        wz0 = 0.5;
        wz1 = 0.0;
        Z1 = Z0;
      }
      const double r0 = 0.75 * xc[Z0 * C.rs + X0] + 0.25 * xc[Z0 * C.rs + X1];
      const double r1 = 0.75 * xc[Z1 * C.rs + X0] + 0.25 * xc[Z1 * C.rs + X1];
      const int p = z * L.rs + xx + 2;
      bot2_store(x, p, xx, L.nx, x[p] + (wz0 * r0 + wz1 * r1));
    }
    __syncthreads();
    bot2_sweeps<NOISE>(x, sm2 + L.b_off, L, sm2 + L.tab_off, a.nu1, a.nu2, true,
                       (gdbl)L.noise + (int64_t)comp * n, (int64_t)a.ncomp * n);
  }
  const Bot2Level& L0 = a.lv[0];
  const int n0 = L0.nx * L0.nz, halo = L0.kind == KIND_BLOCK ? 2 : 0;
  double* xg = L0.xg + (int64_t)comp * n0;
  for (int q = tid; q < n0; q += B2_TPB) {
    int z, xx;
    divmod_uniform(q, L0.nx, z, xx);
    xg[q] = sm2[L0.x_off + z * L0.rs + xx + halo];
  }
}

}  // namespace

hipError_t launch2_level0(const Point2Args& args, int ncomp, double kT, bool noise,
                          const NoiseArgs& na, hipStream_t s) {
  Point2Args a = args;
  const int halo = a.npass + (a.bc ? 2 : 0);
  a.rows = level0_rows(a.nx, a.nz, ncomp, a.npass, a.bc != nullptr);
  if (a.rows == 0 || a.npass > kMaxPoint2) return hipErrorNotSupported;
  for (int nw = 0; nw < 3; ++nw) {
    a.inv_d[nw] = 1.0 / ((4 + nw) * a.ih2);
    a.sig[nw] = sqrt(kT / ((4 + nw) * a.ih2));
  }
  const size_t lds = (size_t)std::min(a.rows + 2 * halo, a.nz) * a.nx * sizeof(double);
  dim3 grid((a.nz + a.rows - 1) / a.rows, ncomp);
  if (noise) k2_level0<true><<<grid, P2_TPB, lds, s>>>(a, na);
  else k2_level0<false><<<grid, P2_TPB, lds, s>>>(a, na);
  return hipGetLastError();
}

hipError_t launch2_noise(const Bot2Args* dev, const Bot2Args& host, const NoiseArgs& na,
                         hipStream_t s) {
  int most = 0;
  for (int i = 0; i < host.nlev; ++i)
    if (host.lv[i].kind == KIND_BLOCK) most = std::max(most, host.lv[i].nx * host.lv[i].nz / 4);
  if (most == 0 || host.nu1 + host.nu2 == 0) return hipSuccess;
  dim3 grid((most + TPB - 1) / TPB, host.nlev, (host.nu1 + host.nu2) * host.ncomp);
  k2_noise<<<grid, TPB, 0, s>>>(dev, na);
  return hipGetLastError();
}

hipError_t launch2_bottom(const Bot2Args* dev, const Bot2Args& host, int part, bool noise,
                          const NoiseArgs& na, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)k2_bottom<true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess)
      e = hipFuncSetAttribute((const void*)k2_bottom<false>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  if (host.lds > kBot2LdsMax) return hipErrorInvalidValue;
  if (noise) k2_bottom<true><<<host.ncomp, B2_TPB, host.lds, s>>>(dev, part, na);
  else k2_bottom<false><<<host.ncomp, B2_TPB, host.lds, s>>>(dev, part, na);
  return hipGetLastError();
}

}  // namespace smg
