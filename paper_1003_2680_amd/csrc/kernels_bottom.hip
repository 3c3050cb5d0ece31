// The LDS-resident bottom of the V-cycle (Alg. 3 below the tiled levels): every level of at most
// 4096 cells and the coarsest exact draw, one work-group per component, in one launch.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "block_update.hpp"
#include "device_common.hpp"
#include "kernels.hpp"

namespace smg {
namespace {

// One work-group per component runs every level from the bottom level down to the coarsest
// and back up, with x, b and a scratch field of each level in LDS; only b of the bottom level
// comes from global memory and only its x goes back.  Colour passes are separated by
// work-group barriers instead of kernel launches.  The coarsest draw is FP64 in every mode.
//
// What bounds it: the serial chain of 8 (nu1 + nu2) colour passes per level on one compute
// unit, so a pass is shaped for latency.  The exchanges of partial sums between a block's eight
// lanes and the eight-value sum of its solve are DPP moves, never LDS permutes; the x rows carry
// two halo cells per side, so a row's five reads are one address with immediate offsets; the
// z-factors and the block's A_BB^-1 row stay in registers over the four passes that share them;
// and the noise of a pair of passes is loaded while the pair before runs.  The 16^3 .. 4^3 bottom
// takes 88 us a launch (FP64): a 16^3 pass 1.3 us, an 8^3 pass 0.55 us.  With indexed window
// reads, permutes and a noise load inside each pass it took 203 us.
constexpr int BOT_TPB = 512;

// Pointers read from a level descriptor are taken into the global address space: a load through a
// generic pointer also counts as an LDS access, so every barrier's wait for LDS would wait for
// the noise prefetched over it.
template <typename T>
using gptr = const __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gptr<T> global_ptr(const void* p) {
  return (gptr<T>)(const T*)p;
}

// The lane's cell within its block, its share s of the cell's planes, and the block's place
// among the blocks of one colour: bx = 2 i + cx, by = 2 j + cy, bz = 2 l + cz.
struct BotLane {
  int kx, ky, kz, s, i, j, l;
};
template <int SPLIT>
__device__ __forceinline__ BotLane bot_lane(const BotLevel& L, int t) {
  BotLane g;
  g.kx = t & 1;
  g.ky = (t >> 1) & 1;
  g.kz = (t >> 2) & 1;
  g.s = SPLIT == 4 ? (t >> 4) & 3 : 0;
  const int nbx2 = L.nx >> 2, nby2 = L.ny >> 2;
  int rest;
  // SPLIT 4: a wave is two blocks, their lanes next to each other as in SPLIT 1
  const int blk = SPLIT == 4 ? ((t >> 6) << 1) | ((t >> 3) & 1) : t >> 3;
  divmod_uniform(blk, nbx2, rest, g.i);
  divmod_uniform(rest, nby2, g.l, g.j);
  return g;
}

template <typename T, int SPLIT, bool INDEX>
__device__ __forceinline__ BlockWeights<T, SPLIT, INDEX> bot_weights(int nz, int sz, const T* tab,
                                                              const BotLane& g, int bz) {
  BlockWeights<T, SPLIT, INDEX> w;
  const T* row = tab + nz * 10 + bz * kBotRow;
  block_weights<T, SPLIT>(w, row, row + 64, g.kx, g.ky, g.kz, g.s);
#pragma unroll
  for (int p = 0; p < BlockWeights<T, SPLIT, INDEX>::P; ++p) {
    int pz = 2 * bz - 2 + 3 * g.kz + (SPLIT == 4 ? g.s : p);
    pz = pz < 0 ? 0 : (pz >= nz ? nz - 1 : pz);
    w.po[p] = pz * sz;
  }
  return w;
}

// x value at LDS element p (row position x) and its copy in the row's halo, if it has one
template <typename T>
__device__ __forceinline__ void bot_store(T* X, int p, int x, int nx, T v) {
  X[p] = v;
  if (x < 2) X[p + nx] = v;
  if (x >= nx - 2) X[p - nx] = v;
}

// Sweeps slot0 .. slot0 + nslot - 1 of a block level.  Z: the level's pregenerated noise of this
// component (natural layout), slot s at s * slot_stride.  A sweep is four pairs of passes (the
// two cx of one cy, cz).  ONE: every lane has at most one cell (SPLIT 4: a quarter of one) per
// pass, and its addresses and factors are formed once per level, cz or pair.  SPLIT 4 is for
// levels whose colours fill a quarter of the work-group or less, 8^3 and smaller: a pass there
// is one wave's chain of instructions, and four waves share it plane by plane (8^3: 1.05 -> 0.72
// us per pass, and 0.55 with the bank-free strides).  Without ONE
// (the flat levels whose nz is not a multiple of four, where one layer parity holds more than
// half of the blocks) the work-group goes over the colour in rounds.
template <typename T, int KIND, int SPLIT, bool ONE>
__device__ __forceinline__ void bot_sweeps_as(T* X, const T* B, const BotLevel& L, const T* tab,
                                              int slot0, int nslot, bool post, gptr<T> Z,
                                              size_t slot_stride) {
  constexpr bool NOISE = KIND == CYCLE_NOISE, INDEX = index_order<T, KIND>;
  using Weights = BlockWeights<T, SPLIT, INDEX>;
  T s1d[20];
#pragma unroll
  for (int q = 0; q < 20; ++q) s1d[q] = (T)L.s1d[q];  // uniform: scalar registers
  const int nx = L.nx, ny = L.ny, nz = L.nz, sy = L.sy, sz = L.sz;
  const int nbz = nz >> 1;
  const int tid = (int)threadIdx.x;
  const int steps = 4 * nslot;  // (slot, cz, cy) in sweep order
  auto cz_of = [&](int st) { return post ? 1 - ((st >> 1) & 1) : (st >> 1) & 1; };
  auto cy_of = [&](int st) { return post ? 1 - (st & 1) : st & 1; };
  auto layers = [&](int cz) { return (nbz + 1 - cz) >> 1; };  // block layers of this parity
  auto rows = [&](const BotLane& g, int cy, int (&ro)[3]) {
    const int y = 4 * g.j + 2 * cy + g.ky;
#pragma unroll
    for (int r = 0; r < 3; ++r)
      ro[r] = wrapm(y + (g.ky ? 2 - r : r - 2), ny) * sy + 4 * g.i + g.kx;
  };
  auto pass = [&](const BotLane& g, const Weights& w, const int (&ro)[3], int own,
                  int cell, int cx, bool active, T noise) {
    const int d = 2 * cx;
    const T v = block_update<T, SPLIT, true>(X + d, ro, s1d, w, own, B[cell + d], noise);
    if (active) bot_store(X, own + d, 4 * g.i + g.kx + d, nx, v);
  };
  if constexpr (ONE) {
    const BotLane g = bot_lane<SPLIT>(L, tid);
    // lanes past the level's blocks take part in the exchanges on cells of layer 0
    auto bz_of = [&](int cz) { return 2 * (g.l < layers(cz) ? g.l : 0) + cz; };
    int ro0[3], ro1[3];
    rows(g, 0, ro0);
    rows(g, 1, ro1);
    // kept as they are, not formed again in every pass
#pragma unroll
    for (int r = 0; r < 3; ++r) asm volatile("" : "+v"(ro0[r]), "+v"(ro1[r]));
    const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    const int per_layer = (nx >> 2) * (ny >> 2) * 8 * SPLIT;
    // the cell of (cx, cy) = (0, 0) within its z-plane: in LDS strides and natural
    const int y0 = 4 * g.j + g.ky, x0 = 4 * g.i + g.kx;
    const int own0 = y0 * sy + x0 + kBotHalo, nat0 = y0 * nx + x0, plane = nx * ny;
    auto noise_of = [&](int st, T& n0, T& n1) {
      const int z = 2 * bz_of(cz_of(st)) + g.kz;
      const gptr<T> p = Z + (size_t)(slot0 + (st >> 2)) * slot_stride;
      const int at = (z < nz ? z : 0) * plane + nat0 + 2 * nx * cy_of(st);
      n0 = p[at];
      n1 = p[at + 2];
    };
    T n0 = T(0), n1 = T(0);
    // a wave past the level's blocks only keeps the barriers: it would take issue slots from the
    // waves that have work
    if (wave0 >= per_layer * layers(0)) {
      for (int st = 0; st < steps; ++st) {
        if (layers(cz_of(st)) == 0) continue;
        __syncthreads();
        __syncthreads();
      }
      return;
    }
    if (NOISE) noise_of(0, n0, n1);
    Weights w;
    int zown = 0, znat = 0;
#pragma unroll 1
    for (int st = 0; st < steps; ++st) {
      const T c0 = n0, c1 = n1;
      if (NOISE && st + 1 < steps) noise_of(st + 1, n0, n1);
      const int cz = cz_of(st), cy = cy_of(st);
      if (layers(cz) == 0) continue;  // one block layer: no blocks of this parity
      const bool active = g.l < layers(cz) && g.s == 0;
      if ((st & 1) == 0) {
        const int bz = bz_of(cz);
        w = bot_weights<T, SPLIT, INDEX>(nz, sz, tab, g, bz);
        zown = (2 * bz + g.kz) * sz + own0;
        znat = (2 * bz + g.kz) * plane + nat0;
      }
      int ro[3];
#pragma unroll
      for (int r = 0; r < 3; ++r) ro[r] = cy ? ro1[r] : ro0[r];
      const int own = zown + (cy ? 2 * sy : 0), cell = znat + (cy ? 2 * nx : 0);
      const int cx = post ? 1 : 0;
      pass(g, w, ro, own, cell, cx, active, post ? c1 : c0);
      __syncthreads();
      pass(g, w, ro, own, cell, cx ^ 1, active, post ? c0 : c1);
      __syncthreads();
    }
  } else {
    const int per_layer = (nx >> 2) * (ny >> 2) * 8;
#pragma unroll 1
    for (int st = 0; st < steps; ++st) {
      const int cz = cz_of(st), cy = cy_of(st);
#pragma unroll 1
      for (int q = 0; q < 2; ++q) {
        const int cx = post ? 1 - q : q;
#pragma unroll 1
        for (int base = 0; base < per_layer * layers(cz); base += BOT_TPB) {
          const BotLane g = bot_lane<SPLIT>(L, base + tid);
          const bool active = g.l < layers(cz);
          const int bz = 2 * (active ? g.l : 0) + cz;
          const Weights w = bot_weights<T, SPLIT, INDEX>(nz, sz, tab, g, bz);
          int ro[3];
          rows(g, cy, ro);
          const int y = 4 * g.j + 2 * cy + g.ky, z = 2 * bz + g.kz, x = 4 * g.i + g.kx;
          const int cell = (z * ny + y) * nx + x;
          T n = T(0);
          if (NOISE) n = Z[(size_t)(slot0 + (st >> 2)) * slot_stride + cell + 2 * cx];
          pass(g, w, ro, z * sz + y * sy + x + kBotHalo, cell, cx, active, n);
        }
        __syncthreads();
      }
    }
  }
}

template <typename T, int KIND>
__device__ __forceinline__ void bot_sweeps(T* X, const T* B, const BotLevel& L, const T* tab,
                                           int slot0, int nslot, bool post, gptr<T> Z,
                                           size_t slot_stride) {
  if (nslot == 0) return;
  // lanes of the larger layer parity's colours
  const int lanes = (L.nx >> 2) * (L.ny >> 2) * (((L.nz >> 1) + 1) >> 1) * 8;
  if (4 * lanes <= BOT_TPB)
    bot_sweeps_as<T, KIND, 4, true>(X, B, L, tab, slot0, nslot, post, Z, slot_stride);
  else if (lanes <= BOT_TPB)
    bot_sweeps_as<T, KIND, 1, true>(X, B, L, tab, slot0, nslot, post, Z, slot_stride);
  else
    bot_sweeps_as<T, KIND, 1, false>(X, B, L, tab, slot0, nslot, post, Z, slot_stride);
}

// r = b - A x on a block level in LDS, in index order (the FP32 chain): a thread takes a
// column of cells (or a part of one, so that the whole work-group has work) and marches up z,
// forming each plane's two in-plane sums once and keeping the five that the current cell reaches.
template <typename T>
__device__ __forceinline__ void bot_residual(T* R, const T* X, const T* B, const BotLevel& L,
                                             const T* tab) {
  T s1d[20];
#pragma unroll
  for (int q = 0; q < 20; ++q) s1d[q] = (T)L.s1d[q];
  const int nx = L.nx, ny = L.ny, nz = L.nz, sy = L.sy, sz = L.sz;
  const int ncol = nx * ny;
  int parts = BOT_TPB / ncol;
  parts = parts < 1 ? 1 : (parts > nz ? nz : parts);
  const int len = (nz + parts - 1) / parts;
  for (int t = threadIdx.x; t < ncol * parts; t += BOT_TPB) {
    int part, col, x, y;
    divmod_uniform(t, ncol, part, col);
    divmod_uniform(col, nx, y, x);
    int ro[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) ro[d] = wrapm(y + d - 2, ny) * sy;
    const int xs[5] = {x, x + 1, x + 2, x + 3, x + 4};
    const int z0 = part * len, z1 = z0 + len < nz ? z0 + len : nz;
    T p0[5], p1[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) p0[d] = p1[d] = T(0);
#pragma unroll 1
    for (int zz = z0 - 2; zz < z1 + 2; ++zz) {
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        p0[d] = p0[d + 1];
        p1[d] = p1[d + 1];
      }
      const T* P = X + (zz < 0 ? 0 : (zz >= nz ? nz - 1 : zz)) * sz;  // beyond a wall: factor 0
      p0[4] = gal_plane<T>(P, 1, xs, ro, s1d, p1[4]);
      const int z = zz - 2;
      if (z < z0) continue;
      const T* zr = tab + z * 10;
      T acc0 = T(0), acc1 = T(0);
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        acc0 = fma(zr[d], p0[d], acc0);
        acc1 = fma(zr[5 + d], p1[d], acc1);
      }
      const int q = z * ncol + col;
      R[q] = B[q] - (acc0 + acc1);
    }
  }
}

// b_c = P^T (b - A x) from a block level in LDS, axis by axis: P^T folds into the 1D stencils of
// A's Kronecker sum, eight taps per coarse position around 2X - 3 .. 2X + 4, so x is read 4 times
// per cell and axis pair instead of 25 and no residual is stored.  R (n elements) holds first the
// two x-folded fields on (nx/2, ny, nz), then the three xy-folded ones on (nx/2, ny/2, nz): those of
// m_y m_x, of a_y m_x + m_y a_x, and of b.  16^3 FP64: 4.7 us (forming the residual of every
// cell by a march up z and restricting it took 11.5); 8^3: 2.0 (6.2).
template <typename T>
__device__ __forceinline__ void bot_restrict(T* bc, T* R, const T* X, const T* B,
                                             const BotLevel& L, const T* tab) {
  using V2 = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
  const int nx = L.nx, ny = L.ny, nz = L.nz, hx = nx >> 1, hy = ny >> 1;
  const int tid = (int)threadIdx.x;
  // taps t and 7 - t are equal: sum_c w_c s[t - 3 - c], w = (1/4, 3/4, 3/4, 1/4) at c = -1 .. 2
  auto fold = [](const double* q, T (&m)[4]) {
    const T s0 = (T)q[0], s1 = (T)q[1], s2 = (T)q[2];
    m[0] = T(0.25) * s0;
    m[1] = fma(T(0.25), s1, T(0.75) * s0);
    m[2] = fma(T(0.25), s2, T(0.75) * (s0 + s1));
    m[3] = fma(T(0.25), s0 + s1, T(0.75) * (s1 + s2)) ;
  };
  {
    T m[4], am[4];
    fold(L.s1d, m);
    fold(L.s1d + 5, am);
    const int items = hx * ny * nz;
    T* U = R;
    T* V = R + items;
    for (int it = tid; it < items; it += BOT_TPB) {
      int r, Xc, y, z;
      divmod_uniform(it, hx, r, Xc);
      divmod_uniform(r, ny, z, y);
      const T* row = X + z * L.sz + y * L.sy + kBotHalo;
      const V2 v0 = *reinterpret_cast<const V2*>(row + 2 * Xc - 2);
      const V2 v1 = *reinterpret_cast<const V2*>(row + 2 * Xc);
      const V2 v2 = *reinterpret_cast<const V2*>(row + 2 * Xc + 2);
      // the halo holds two cells a side: the outermost taps of the end cells wrap by hand
      const T lo = row[Xc == 0 ? nx - 3 : 2 * Xc - 3], hi = row[Xc == hx - 1 ? 2 : 2 * Xc + 4];
      const T e0 = lo + hi, e1 = v0.x + v2.y, e2 = v0.y + v2.x, e3 = v1.x + v1.y;
      U[it] = fma(m[0], e0, fma(m[1], e1, fma(m[2], e2, m[3] * e3)));
      V[it] = fma(am[0], e0, fma(am[1], e1, fma(am[2], e2, am[3] * e3)));
    }
  }
  __syncthreads();
  const int items2 = hx * hy * nz, col = hx * hy;
  {
    T m[4], am[4];
    fold(L.s1d + 10, m);
    fold(L.s1d + 15, am);
    const T* U = R;
    const T* V = R + 2 * items2;
    constexpr int PER = 4096 / 4 / BOT_TPB;
    T p0[PER], p1[PER], p2[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int it = tid + k * BOT_TPB;
      if (it >= items2) break;
      int r, Xc, Y, z;
      divmod_uniform(it, hx, r, Xc);
      divmod_uniform(r, hy, z, Y);
      const int base = z * ny;
      T a0 = T(0), a1 = T(0);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int y0 = wrapm(2 * Y - 3 + t, ny), y1 = wrapm(2 * Y + 4 - t, ny);
        const T u = U[(base + y0) * hx + Xc] + U[(base + y1) * hx + Xc];
        const T v = V[(base + y0) * hx + Xc] + V[(base + y1) * hx + Xc];
        a0 = fma(m[t], u, a0);
        a1 = fma(am[t], u, fma(m[t], v, a1));
      }
      p0[k] = a0;
      p1[k] = a1;
      const int xl = Xc == 0 ? nx - 1 : 2 * Xc - 1, xh = Xc == hx - 1 ? 0 : 2 * Xc + 2;
      T bs[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {  // the inner two rows (3/4), the outer two (1/4)
        T s = T(0), o = T(0);
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const int y = q == 0 ? 2 * Y + d : wrapm(2 * Y - 1 + 3 * d, ny);
          const T* row = B + (base + y) * nx;
          const V2 c = *reinterpret_cast<const V2*>(row + 2 * Xc);
          s += c.x + c.y;
          o += row[xl] + row[xh];
        }
        bs[q] = fma(T(0.75), s, T(0.25) * o);
      }
      p2[k] = fma(T(0.75), bs[0], T(0.25) * bs[1]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int it = tid + k * BOT_TPB;
      if (it >= items2) break;
      R[it] = p0[k];
      R[items2 + it] = p1[k];
      R[2 * items2 + it] = p2[k];
    }
  }
  __syncthreads();
  const int nzc = nz >> 1;
  for (int it = tid; it < col * nzc; it += BOT_TPB) {
    int Z, q;
    divmod_uniform(it, col, Z, q);
    T p0[8], p1[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      int z = 2 * Z - 3 + t;
      z = z < 0 ? 0 : (z >= nz ? nz - 1 : z);  // beyond a wall: factor 0
      p0[t] = R[z * col + q];
      p1[t] = R[items2 + z * col + q];
    }
    T acc = T(0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int z = 2 * Z - 1 + c;
      if (z < 0 || z >= nz) continue;
      const T* zr = tab + z * 10;
      T s = R[2 * items2 + z * col + q];
#pragma unroll
      for (int d = 0; d < 5; ++d) s = fma(-zr[d], p0[c + d], fma(-zr[5 + d], p1[c + d], s));
      T wz = pw<T>(c);
      if ((Z == 0 && c == 1) || (Z == nzc - 1 && c == 2)) wz = T(0.5);
      acc = fma(wz, s, acc);
    }
    bc[it] = acc;
  }
}

// Level 0 in the bottom: the red-black point heat bath of a hierarchy of at most 4096 cells, its
// state in LDS in the split layout (natural, no halo: consecutive lanes touch consecutive words).
// A thread owns the sites p = tid + k BOT_TPB of either colour, so a site's row, plane and wall
// are found once, and the normals of a pass are loaded while the pass before runs.  A launch per
// colour pass and transfer of such a grid is all latency: a 16^3 cycle took 75 us in 12 launches
// and takes 49 in two (noise 4.6, this one 44.0; a sample's export is a third, 4.5), of which the
// point level 16: a pass 0.55 us, the folded restriction 3.8 (a residual and its window sums 4.8),
// the prolongation 1.8.
constexpr int PT_PER = 4096 / 2 / BOT_TPB;
template <typename T>
struct PointSites {
  int p[PT_PER], n[PT_PER], s[PT_PER], u[PT_PER], d[PT_PER];  // the site, its y and z neighbours
  int o[PT_PER][2];      // per colour: the x-neighbour beside entry p of the other colour
  int nat[PT_PER][2];    // per colour: the site's natural index
  int wall[PT_PER];      // bit 0: at the top, bit 1: at the bottom
  int nsite;
  __device__ __forceinline__ void init(const BotLevel& L) {
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));  // formed anew by each leg: not kept over the levels between
    const int nh = L.nx >> 1, ny = L.ny, nz = L.nz, plane = nh * ny;
    nsite = plane * nz;
#pragma unroll
    for (int k = 0; k < PT_PER; ++k) {
      p[k] = tid + k * BOT_TPB;
      const int q = p[k] < nsite ? p[k] : 0;  // lanes past the sites stay in range
      int row, j, z, y;
      divmod_uniform(q, nh, row, j);
      divmod_uniform(row, ny, z, y);
      n[k] = q + (y + 1 == ny ? nh - plane : nh);
      s[k] = q + (y == 0 ? plane - nh : -nh);
      u[k] = z + 1 < nz ? q + plane : q;
      d[k] = z > 0 ? q - plane : q;
      wall[k] = (z + 1 >= nz ? 1 : 0) | (z == 0 ? 2 : 0);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int xs = (y + z + c) & 1;  // x = 2j + xs: neighbours j and j + 1 or j - 1
        o[k][c] = xs ? (j + 1 == nh ? q - j : q + 1) : (j == 0 ? q + nh - 1 : q - 1);
        nat[k][c] = row * L.nx + 2 * j + xs;
      }
    }
  }
};

// The normals of colour pass q of the sweeps slot0 .. of a leg.
template <typename T>
__device__ __forceinline__ void point_noise(T (&z)[PT_PER], const PointSites<T>& S, gptr<T> Z,
                                            size_t slot_stride, int slot0, int q, bool post) {
  const int colour = post ? 1 - (q & 1) : q & 1;
  const gptr<T> P = Z + (size_t)(slot0 + (q >> 1)) * slot_stride + (size_t)colour * S.nsite;
#pragma unroll
  for (int k = 0; k < PT_PER; ++k) z[k] = P[S.p[k] < S.nsite ? S.p[k] : 0];
}

// Sweeps slot0 .. slot0 + nslot - 1; z holds the normals of the first pass (point_noise).  VEC: the
// order of the sums in the colour-pass launches (launch_rb_pass), whose bits these are.
template <typename T, int KIND, bool VEC>
__device__ __forceinline__ void point_sweeps_as(T* X, const T* B, bool has_b, const BotLevel& L,
                                             const PointSites<T>& S, T (&z)[PT_PER], gptr<T> Z,
                                             size_t slot_stride, int slot0, int nslot, bool post) {
  constexpr bool NOISE = KIND == CYCLE_NOISE;
  const int nsite = S.nsite;
  T dg[10];
#pragma unroll
  for (int e = 0; e < 10; ++e) dg[e] = (T)L.s1d[e];  // uniform: scalar registers
#pragma unroll 1
  for (int q = 0; q < 2 * nslot; ++q) {
    const int c = post ? 1 - (q & 1) : q & 1;
    T zn[PT_PER];
#pragma unroll
    for (int k = 0; k < PT_PER; ++k) zn[k] = z[k];
    if (NOISE && q + 1 < 2 * nslot) point_noise<T>(z, S, Z, slot_stride, slot0, q + 1, post);
    T* xc = X + c * nsite;
    const T* xo = X + (1 - c) * nsite;
    const T* bc = B + c * nsite;
#pragma unroll
    for (int k = 0; k < PT_PER; ++k) {
      if (k * BOT_TPB >= nsite) break;
      const bool top = S.wall[k] & 1, low = S.wall[k] & 2;
      const int own = S.p[k] < nsite ? S.p[k] : 0, ox = c ? S.o[k][1] : S.o[k][0];
      const T sx = xo[own] + xo[ox];
      const T sxy = sx + (xo[S.n[k]] + xo[S.s[k]]);
      T sum;
      if (VEC)
        sum = sxy + fma(xo[S.u[k]], top ? T(0) : T(1), xo[S.d[k]] * (low ? T(0) : T(1)));
      else
        sum = (sxy + (top ? T(0) : xo[S.u[k]])) + (low ? T(0) : xo[S.d[k]]);
      const int nw = (int)top + (int)low;
      auto by_walls = [&](T d6, T d7, T d8) { return nw == 0 ? d6 : (nw == 1 ? d7 : d8); };
      const T rhs = has_b ? fma(sum, dg[9], bc[own]) : sum * dg[9];
      const T idg = by_walls(dg[0], dg[1], dg[2]);
      T v = has_b || !VEC ? rhs * idg : sum * by_walls(dg[6], dg[7], dg[8]);
      if (NOISE) {
        const T sig = by_walls(dg[3], dg[4], dg[5]);
        v = VEC ? fma(sig, zn[k], v) : fma(rhs, idg, sig * zn[k]);
      }
      if (S.p[k] < nsite) xc[own] = v;
    }
    __syncthreads();
  }
}

template <typename T, int KIND>
__device__ __forceinline__ void point_sweeps(T* X, const T* B, bool has_b, const BotLevel& L,
                                              const PointSites<T>& S, T (&z)[PT_PER], gptr<T> Z,
                                              size_t slot_stride, int slot0, int nslot, bool post) {
  if ((L.nx >> 1) % (16 / (int)sizeof(T)) == 0)
    point_sweeps_as<T, KIND, true>(X, B, has_b, L, S, z, Z, slot_stride, slot0, nslot, post);
  else
    point_sweeps_as<T, KIND, false>(X, B, has_b, L, S, z, Z, slot_stride, slot0, nslot, post);
}

// R = b - A x in natural layout.
template <typename T>
__device__ __forceinline__ void point_residual(T* R, const T* X, const T* B, bool has_b,
                                               const BotLevel& L, const PointSites<T>& S) {
  const int nsite = S.nsite;
  const T ih2 = (T)L.s1d[9];
#pragma unroll
  for (int k = 0; k < PT_PER; ++k) {
    if (S.p[k] >= nsite) break;
    const bool top = S.wall[k] & 1, low = S.wall[k] & 2;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const T* xo = X + (1 - c) * nsite;
      T sn = (xo[S.p[k]] + xo[S.o[k][c]]) + (xo[S.s[k]] + xo[S.n[k]]);
      if (!top) sn += xo[S.u[k]];
      if (!low) sn += xo[S.d[k]];
      const T t = fma(-T(6 + (int)top + (int)low), X[c * nsite + S.p[k]], sn);
      R[S.nat[k][c]] = has_b ? fma(t, ih2, B[c * nsite + S.p[k]]) : t * ih2;
    }
  }
}

// (P^T R)(X, Y, Z) in index order: column sums first, as k_restrict_residual0 adds them.
template <typename T>
__device__ __forceinline__ T point_restrict(const T* R, int nx, int ny, int nz, int X, int Y,
                                            int Z) {
  int xs[4], ys[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    xs[d] = wrapm(2 * X - 1 + d, nx);
    ys[d] = wrapm(2 * Y - 1 + d, ny) * nx;
  }
  T acc = T(0);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int z = 2 * Z - 1 + c;
    if (z < 0 || z >= nz) continue;
    const T* P = R + z * nx * ny;
    T cs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      T s = T(0);
#pragma unroll
      for (int b = 0; b < 4; ++b) s = fma(pw<T>(b), P[ys[b] + xs[q]], s);
      cs[q] = s * pw<T>(q);
    }
    T wz = pw<T>(c);
    if ((Z == 0 && z == 0) || (Z == (nz >> 1) - 1 && z == nz - 1)) wz = T(0.5);
    acc = fma(wz, (cs[0] + cs[1]) + (cs[2] + cs[3]), acc);
  }
  return acc;
}

// b_1 = P^T (b - A x) axis by axis, the sums of k_fold_residual0 in its order: per fine row and
// coarse column u = Px^T x and s = Px^T (b - a_x x), per coarse row p and q of them, then the six
// planes of a layer.  R (n elements) holds first u, s on (nx/2, ny, nz), then p, q on (nx/2, ny/2, nz).
template <typename T>
__device__ __forceinline__ void point_fold(T* bc, T* R, const T* X, const T* B, bool has_b,
                                           const BotLevel& L, const PointSites<T>& S) {
  const int nh = L.nx >> 1, ny = L.ny, nz = L.nz, nyc = ny >> 1, nzc = nz >> 1;
  const int tid = (int)threadIdx.x, nsite = S.nsite, half = nsite >> 1, col = nh * nyc;
  const T ih2 = (T)L.s1d[9];
  const T q1 = T(0.25), q3 = T(0.75), d1 = T(0.25) * ih2, d2 = T(0.5) * ih2;
#pragma unroll
  for (int k = 0; k < PT_PER; ++k) {
    const int it = S.p[k];
    if (it >= nsite) break;
    // even cells 2j of the row are entries of colour (y + z) & 1, odd ones of the other
    const int odd = S.nat[k][0] & 1;
    const int l = odd ? S.o[k][1] : S.o[k][0], r = odd ? S.o[k][0] : S.o[k][1];
    const T *E = X + odd * nsite, *O = X + (1 - odd) * nsite;
    const T m = E[it] + O[it], n = O[l] + E[r];
    T s = fma(d1, n + (E[l] + O[r]), -d2 * m);
    if (has_b) {
      const T *Eb = B + odd * nsite, *Ob = B + (1 - odd) * nsite;
      s += fma(q3, Eb[it] + Ob[it], q1 * (Ob[l] + Eb[r]));
    }
    R[it] = fma(q3, m, q1 * n);
    R[nsite + it] = s;
  }
  __syncthreads();
  constexpr int PER = 4096 / 4 / BOT_TPB;
  T p[PER], q[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int it = tid + k * BOT_TPB;
    if (it >= half) break;
    int r, Xc, Y, z;
    divmod_uniform(it, nh, r, Xc);
    divmod_uniform(r, nyc, z, Y);
    T u[6], s[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      const int at = (z * ny + wrapm(2 * Y - 2 + d, ny)) * nh + Xc;
      u[d] = R[at];
      s[d] = R[nsite + at];
    }
    const T mid = u[2] + u[3], near = u[1] + u[4], far = u[0] + u[5];
    p[k] = fma(q3, mid, q1 * near);
    q[k] = fma(q3, s[2] + s[3], q1 * (s[1] + s[4])) + fma(d1, near + far, -d2 * mid);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int it = tid + k * BOT_TPB;
    if (it >= half) break;
    R[it] = p[k];
    R[half + it] = q[k];
  }
  __syncthreads();
  for (int it = tid; it < col * nzc; it += BOT_TPB) {
    int Z, c;
    divmod_uniform(it, col, Z, c);
    const T mid = d2 + (Z == 0 ? d1 : T(0)) + (Z == nzc - 1 ? d1 : T(0));
    T acc = T(0);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      const int f = 2 * Z - 2 + d;
      if (f < 0 || f >= nz) continue;
      acc = fma(d == 2 || d == 3 ? -mid : d1, R[f * col + c], acc);
      T w = d == 1 || d == 4 ? q1 : q3;
      if ((d == 2 && Z == 0) || (d == 3 && Z == nzc - 1)) w = T(0.5);
      if (d > 0 && d < 5) acc = fma(w, R[half + f * col + c], acc);
    }
    bc[it] = acc;
  }
}

// POINT: the first level may be a point level (level 0).
template <typename T, int KIND, bool POINT>
__device__ __forceinline__ void bottom_body(const BotArgs& a, const uint32_t comp,
                                            const NoiseArgs& na, int part_b) {
  constexpr bool NOISE = KIND == CYCLE_NOISE;
  const int part = part_b & 3;
  const bool has_b = part_b & kBotHasB;
  extern __shared__ char smraw[];
  T* sm = reinterpret_cast<T*>(smraw);
  const int tid = threadIdx.x;
  const BotLevel& L0 = a.lv[0];
  const int n0 = L0.nx * L0.ny * L0.nz;
  const bool below = part_b & kBotBelow;
  const bool point = POINT && L0.kind == KIND_POINT && !below;
  const int first = point || below ? 1 : 0;  // the first level in the natural layout
  const gptr<T> pn = global_ptr<T>(L0.noise) + (size_t)comp * n0;
  const size_t pstride = (size_t)a.ncomp * n0;
  auto point_load = [&](const PointSites<T>& ps) {
    T* X = sm + a.lds_off[0];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const size_t at = ((size_t)c * a.ncomp + comp) * ps.nsite;
      const gptr<T> xg = global_ptr<T>(L0.xg) + at, bg = global_ptr<T>(L0.bg) + at;
#pragma unroll
      for (int k = 0; k < PT_PER; ++k) {
        if (ps.p[k] >= ps.nsite) break;
        X[c * ps.nsite + ps.p[k]] = xg[ps.p[k]];
        if (has_b) X[n0 + c * ps.nsite + ps.p[k]] = bg[ps.p[k]];
      }
    }
  };
  auto point_store = [&](const PointSites<T>& ps) {
    const T* X = sm + a.lds_off[0];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      T* xg = (T*)L0.xg + ((size_t)c * a.ncomp + comp) * ps.nsite;
#pragma unroll
      for (int k = 0; k < PT_PER; ++k)
        if (ps.p[k] < ps.nsite) xg[ps.p[k]] = X[c * ps.nsite + ps.p[k]];
    }
  };
  // element of the LDS field x for the natural index q of level L, halo copies beside it
  auto place = [](const BotLevel& L, int q, int& x) {
    int y, z, r;
    divmod_uniform(q, L.nx, r, x);
    divmod_uniform(r, L.ny, z, y);
    return z * L.sz + y * L.sy + x + (L.kind == KIND_BLOCK ? kBotHalo : 0);
  };
  if (part == BOT_UP) {  // x and b of every block level, and the coarsest x, as BOT_DOWN left them
    for (int i = first; i < a.nlev; ++i) {
      const BotLevel& L = a.lv[i];
      const int n = L.nx * L.ny * L.nz;
      T* xi = sm + a.lds_off[i];
      const gptr<T> xg = global_ptr<T>(L.xg) + (size_t)comp * n;
      const gptr<T> bg = global_ptr<T>(L.bg) + (size_t)comp * n;
      for (int q = tid; q < n; q += BOT_TPB) {
        int x;
        const int p = place(L, q, x);
        if (L.kind == KIND_BLOCK) {
          bot_store(xi, p, x, L.nx, (T)xg[q]);
          xi[L.nz * L.sz + q] = bg[q];
        } else {
          xi[p] = xg[q];
        }
      }
    }
  } else if (!point) {
    const BotLevel& L = a.lv[first];
    const int n = L.nx * L.ny * L.nz;
    T* x0 = sm + a.lds_off[first];
    for (int q = tid; q < L.nz * L.sz; q += BOT_TPB) x0[q] = T(0);
    T* b0 = x0 + L.nz * L.sz;
    const gptr<T> bg = global_ptr<T>(L.bg) + (size_t)comp * n;
    for (int q = tid; q < n; q += BOT_TPB) b0[q] = bg[q];
  }
  // operator tables of the block levels (bot_table_elems) at tab_off[i]; the normals
  // of the coarsest draw, which depend on nothing above it
  for (int i = first; i < a.nlev; ++i) {
    const BotLevel& L = a.lv[i];
    if (L.kind == KIND_BLOCK) {
      const int nz = L.nz;
      T* t = sm + a.tab_off[i];
      const gptr<T> zt = global_ptr<T>(L.zt), bf = global_ptr<T>(L.bfac);
      for (int q = tid; q < nz * 10; q += BOT_TPB) t[q] = zt[q];
      for (int q = tid; q < (nz / 2) * kBotRow; q += BOT_TPB) {
        const int bz = q / kBotRow, e = q - bz * kBotRow;
        t[nz * 10 + q] = bf[bz * kBlockRow<T> + (e < 64 ? e : e - 64 + kBlockZ)];
      }
    } else if (NOISE && part == BOT_WHOLE) {
      const int n = L.nx * L.ny * L.nz;
      T* ri = sm + a.lds_off[i] + 2 * n;
      const uint32_t sid = (uint32_t)(a.level0 + i) | (1u << 24);
      for (int q = tid; 2 * q < n; q += BOT_TPB) {
        double z0, z1;
        normal_pair(na, sid, comp, (uint32_t)q, z0, z1);
        ri[2 * q] = (T)z0;
        if (2 * q + 1 < n) ri[2 * q + 1] = (T)z1;
      }
    }
  }
  __syncthreads();
  int last = a.nlev - 1;
  T pz[PT_PER] = {};  // the point level's normals of its next pass
  if (point && part != BOT_UP) {
    PointSites<T> ps;
    ps.init(L0);
    T* X = sm + a.lds_off[0];
    if (NOISE && a.nu1 > 0) point_noise<T>(pz, ps, pn, pstride, 0, 0, false);
    point_load(ps);
    __syncthreads();
    point_sweeps<T, KIND>(X, X + n0, has_b, L0, ps, pz, pn, pstride, 0, a.nu1, false);
    if (NOISE && part != BOT_DOWN && a.nu2 > 0)
      point_noise<T>(pz, ps, pn, pstride, a.nu1, 0, true);
    if (a.nlev == 1) {
      // smoothing-only: the post-sweeps follow at once
      point_sweeps<T, KIND>(X, X + n0, has_b, L0, ps, pz, pn, pstride, a.nu1, a.nu2, true);
      point_store(ps);
      return;
    }
    if (part == BOT_DOWN) point_store(ps);
    // b_1 = P^T (b - A x), x_1 = 0, added up as the launch of this restriction does
    // (launch_restrict_residual0)
    const BotLevel& C = a.lv[1];
    T* xc = sm + a.lds_off[1];
    T* bc = xc + C.nz * C.sz;
    for (int q = tid; q < C.nz * C.sz; q += BOT_TPB) xc[q] = T(0);
    if (!index_order<T, KIND> && (L0.nx >> 1) % 2 == 0) {
      point_fold<T>(bc, X + 2 * n0, X, X + n0, has_b, L0, ps);
    } else {
      point_residual<T>(X + 2 * n0, X, X + n0, has_b, L0, ps);
      __syncthreads();
      for (int q = tid; q < C.nx * C.ny * C.nz; q += BOT_TPB) {
        int Xc, Y, Z, r;
        divmod_uniform(q, C.nx, r, Xc);
        divmod_uniform(r, C.ny, Z, Y);
        bc[q] = point_restrict<T>(X + 2 * n0, L0.nx, L0.ny, L0.nz, Xc, Y, Z);
      }
    }
    __syncthreads();
  }
  for (int i = first; i < a.nlev && part != BOT_UP; ++i) {
    const BotLevel& L = a.lv[i];
    const int n = L.nx * L.ny * L.nz;
    T* xi = sm + a.lds_off[i];
    T* bi = xi + L.nz * L.sz;
    T* ri = bi + n;
    if (part == BOT_DOWN && i > 0) {
      T* bg = (T*)L.bg + (size_t)comp * n;
      for (int q = tid; q < n; q += BOT_TPB) bg[q] = bi[q];
    }
    if (L.kind == KIND_CHOL) {
      if (part == BOT_DOWN) return;
      // exact draw x = A_c^-1 b + sqrt(kT) L_c^-T n (natural layout on this level).  G lanes
      // per row (a power of two, G <= 32) split the columns, so that every lane has only n/G
      // loads of the dense factors in its chain; their sums meet by shuffles
      const gptr<double> ainv = global_ptr<double>(a.ainv), wl = global_ptr<double>(a.w);
      int G = 1;
      while (G < 32 && 2 * G * n <= BOT_TPB) G *= 2;
      const int part = tid % G;
      for (int row = tid / G; row < n; row += BOT_TPB / G) {
        double acc = 0.0, an = 0.0;
#pragma unroll 8
        for (int jj = part; jj < n; jj += G) {
          acc = fma(ainv[(size_t)jj * n + row], (double)bi[jj], acc);
          if (NOISE && jj >= row) an = fma(wl[(size_t)jj * n + row], (double)ri[jj], an);
        }
        for (int off = G / 2; off >= 1; off >>= 1) {
          acc += __shfl_xor(acc, off, G);
          if (NOISE) an += __shfl_xor(an, off, G);
        }
        if (NOISE) acc = fma(na.sqkT, an, acc);
        if (part == 0) xi[row] = (T)acc;
      }
      __syncthreads();
      last = i;
      break;
    }
    const T* tab = sm + a.tab_off[i];
    const gptr<T> Z = global_ptr<T>(L.noise) + (size_t)comp * n;
    const size_t zs = (size_t)a.ncomp * n;
    bot_sweeps<T, KIND>(xi, bi, L, tab, 0, a.nu1, false, Z, zs);
    if (i == a.nlev - 1) {
      // smoothing-only coarsest level: the post-sweeps follow at once
      bot_sweeps<T, KIND>(xi, bi, L, tab, a.nu1, a.nu2, true, Z, zs);
      last = i;
      break;
    }
    if (part == BOT_DOWN) {
      T* xg = (T*)L.xg + (size_t)comp * n;
      for (int q = tid; q < n; q += BOT_TPB) {
        int x;
        xg[q] = xi[place(L, q, x)];
      }
    }
    // b_{i+1} = P^T (b_i - A_i x_i), x_{i+1} = 0
    const BotLevel& C = a.lv[i + 1];
    T* xc = sm + a.lds_off[i + 1];
    for (int q = tid; q < C.nz * C.sz; q += BOT_TPB) xc[q] = T(0);
    T* bc = xc + C.nz * C.sz;
    if constexpr (index_order<T, KIND>) {
      bot_residual<T>(ri, xi, bi, L, tab);
      __syncthreads();
      for (int q = tid; q < C.nx * C.ny * C.nz; q += BOT_TPB) {
        int Xc, Y, Z, r;
        divmod_uniform(q, C.nx, r, Xc);
        divmod_uniform(r, C.ny, Z, Y);
        bc[q] = restrict_at<T>(ri, L.nx, L.nx * L.ny, L.nx, L.ny, L.nz, Xc, Y, Z);
      }
    } else {
      bot_restrict<T>(bc, ri, xi, bi, L, tab);
    }
    __syncthreads();
  }
  for (int i = last - 1; i >= first; --i) {
    const BotLevel& L = a.lv[i];
    const BotLevel& C = a.lv[i + 1];
    const int n = L.nx * L.ny * L.nz;
    T* xi = sm + a.lds_off[i];
    const T* xc = sm + a.lds_off[i + 1] + (C.kind == KIND_BLOCK ? kBotHalo : 0);
    for (int q = tid; q < n; q += BOT_TPB) {
      int x, y, z, r;
      divmod_uniform(q, L.nx, r, x);
      divmod_uniform(r, L.ny, z, y);
      const int p = z * L.sz + y * L.sy + x + kBotHalo;
      bot_store(xi, p, x, L.nx,
                xi[p] + prolong_at<T>(xc, C.sy, C.sz, x, y, z, C.nx, C.ny, C.nz));
    }
    __syncthreads();
    bot_sweeps<T, KIND>(xi, xi + L.nz * L.sz, L, sm + a.tab_off[i], a.nu1, a.nu2, true,
                         global_ptr<T>(L.noise) + (size_t)comp * n, (size_t)a.ncomp * n);
  }
  if (point) {
    T* X = sm + a.lds_off[0];
    PointSites<T> ps;
    ps.init(L0);
    if (part == BOT_UP) {
      if (NOISE && a.nu2 > 0) point_noise<T>(pz, ps, pn, pstride, a.nu1, 0, true);
      point_load(ps);
      __syncthreads();
    }
    // x += P e; with post-sweeps colour 1, drawn afresh by their first pass, needs none
    const BotLevel& C = a.lv[1];
    const T* xc = sm + a.lds_off[1] + (C.kind == KIND_BLOCK ? kBotHalo : 0);
    for (int c = 0; c < (a.nu2 > 0 ? 1 : 2); ++c)
#pragma unroll
      for (int k = 0; k < PT_PER; ++k) {
        if (ps.p[k] >= ps.nsite) break;
        int x, y, z, r;
        divmod_uniform(c ? ps.nat[k][1] : ps.nat[k][0], L0.nx, r, x);
        divmod_uniform(r, L0.ny, z, y);
        X[c * ps.nsite + ps.p[k]] +=
            prolong_at<T>(xc, C.sy, C.sz, x, y, z, C.nx, C.ny, C.nz);
      }
    __syncthreads();
    point_sweeps<T, KIND>(X, X + n0, has_b, L0, ps, pz, pn, pstride, a.nu1, a.nu2, true);
    point_store(ps);
    return;
  }
  const BotLevel& L = a.lv[first];
  const int n = L.nx * L.ny * L.nz;
  T* xg = (T*)L.xg + (size_t)comp * n;
  for (int q = tid; q < n; q += BOT_TPB) {
    int x;
    xg[q] = sm[a.lds_off[first] + place(L, q, x)];
  }
}

// One hierarchy, one work-group per component.
template <typename T, int KIND, bool POINT>
__global__ __launch_bounds__(BOT_TPB)
__attribute__((amdgpu_waves_per_eu(2, 2))) void k_bottom(const BotArgs* __restrict__ ap, int c0,
                                                    int part, NoiseArgs na) {
  bottom_body<T, KIND, POINT>(*ap, c0 + (int)blockIdx.x, na, part);
}

// Several hierarchies (of any sizes) in one launch: work-group w runs component wg >> 16 of
// item wg & 0xffff, with that item's level descriptors and noise keys, so the latency-bound
// bottoms of uneven instances overlap instead of running one launch after another.
template <typename T, int KIND, bool POINT>
__global__ __launch_bounds__(BOT_TPB)
__attribute__((amdgpu_waves_per_eu(2, 2))) void k_bottom_multi(BotMultiArgs m) {
  const uint32_t w = m.wg[blockIdx.x];
  const BotMultiItem& it = m.it[w & 0xffffu];
  NoiseArgs na;
  na.k0 = it.k0;
  na.k1 = it.k1;
  na.sid = 0;
  na.c2 = it.c2;
  na.c3 = it.c3;
  na.sqkT = it.sqkT;
  na.chains = it.chains;
  na.comps_per_chain = it.cpc;
  na.cpc_magic = it.cpc_magic;
  na.bm = m.bm;
  bottom_body<T, KIND, POINT>(*it.args, w >> 16, na, it.part);
}

}  // namespace

// The kernels with dynamic LDS of up to 160 KB (the attribute is set once a process each).
template <typename K>
static hipError_t big_lds(K k, bool& set) {
  if (set) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute((const void*)k,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  set = e == hipSuccess;
  return e;
}

template <typename T>
hipError_t launch_bottom(const BotArgs* a, int ncomp, int c0, size_t lds, int kind, bool point,
                         int part, const NoiseArgs& na, hipStream_t s) {
  hipError_t rc = hipSuccess;
  auto go = [&](auto kd, auto pt) -> hipError_t {
    static bool set = false;
    auto k = k_bottom<T, decltype(kd)::value, decltype(pt)::value>;
    const hipError_t e = big_lds(k, set);
    if (e != hipSuccess) return e;
    k<<<ncomp, BOT_TPB, lds, s>>>(a, c0, part, na);
    return hipGetLastError();
  };
  by_kind<T>(kind, [&](auto kd) {
    rc = point ? go(kd, std::true_type()) : go(kd, std::false_type());
  });
  return rc;
}

template <typename T>
hipError_t launch_bottom_multi(const BotMultiArgs& m, int nwg, size_t lds, int kind, bool point,
                               hipStream_t s) {
  if (nwg <= 0) return hipSuccess;
  if (nwg > kBotMultiWG || m.nitems > kBotMultiItems) return hipErrorInvalidValue;
  hipError_t rc = hipSuccess;
  auto go = [&](auto kd, auto pt) -> hipError_t {
    static bool set = false;
    auto k = k_bottom_multi<T, decltype(kd)::value, decltype(pt)::value>;
    const hipError_t e = big_lds(k, set);
    if (e != hipSuccess) return e;
    k<<<nwg, BOT_TPB, lds, s>>>(m);
    return hipGetLastError();
  };
  by_kind<T>(kind, [&](auto kd) {
    rc = point ? go(kd, std::true_type()) : go(kd, std::false_type());
  });
  return rc;
}

#define SMG_INST(T)                                                                  \
  template hipError_t launch_bottom<T>(const BotArgs*, int, int, size_t, int, bool,  \
                                       int, const NoiseArgs&, hipStream_t);          \
  template hipError_t launch_bottom_multi<T>(const BotMultiArgs&, int, size_t, int,  \
                                             bool, hipStream_t);
SMG_INST(double)
SMG_INST(float)
#undef SMG_INST

}  // namespace smg
