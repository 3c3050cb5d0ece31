// The LDS-resident bottom of the V-cycle (Alg. 3 below the tiled levels): every level of at most
// 4096 cells and the coarsest exact draw, one work-group per component, in one launch.
#include <hip/hip_runtime.h>

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
// takes 92 us (FP64, inside the kernel; FP32 76 us): a 16^3 pass 1.3 us, an 8^3 pass 0.55 us.
// With indexed window reads, permutes and a noise load inside each pass it took 203 us.
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

template <typename T, int SPLIT>
__device__ __forceinline__ BlockWeights<T, SPLIT> bot_weights(int nz, int sz, const T* tab,
                                                              const BotLane& g, int bz) {
  BlockWeights<T, SPLIT> w;
  const T* row = tab + nz * 10 + bz * kBotRow;
  block_weights<T, SPLIT>(w, row, row + 64, g.kx, g.ky, g.kz, g.s);
#pragma unroll
  for (int p = 0; p < BlockWeights<T, SPLIT>::P; ++p) {
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
template <typename T, bool NOISE, int SPLIT, bool ONE>
__device__ __forceinline__ void bot_sweeps_as(T* X, const T* B, const BotLevel& L, const T* tab,
                                              int slot0, int nslot, bool post, gptr<T> Z,
                                              size_t slot_stride) {
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
  auto pass = [&](const BotLane& g, const BlockWeights<T, SPLIT>& w, const int (&ro)[3], int own,
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
    BlockWeights<T, SPLIT> w;
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
        w = bot_weights<T, SPLIT>(nz, sz, tab, g, bz);
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
          const BlockWeights<T, SPLIT> w = bot_weights<T, SPLIT>(nz, sz, tab, g, bz);
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

template <typename T, bool NOISE>
__device__ __forceinline__ void bot_sweeps(T* X, const T* B, const BotLevel& L, const T* tab,
                                           int slot0, int nslot, bool post, gptr<T> Z,
                                           size_t slot_stride) {
  if (nslot == 0) return;
  // lanes of the larger layer parity's colours
  const int lanes = (L.nx >> 2) * (L.ny >> 2) * (((L.nz >> 1) + 1) >> 1) * 8;
  if (4 * lanes <= BOT_TPB)
    bot_sweeps_as<T, NOISE, 4, true>(X, B, L, tab, slot0, nslot, post, Z, slot_stride);
  else if (lanes <= BOT_TPB)
    bot_sweeps_as<T, NOISE, 1, true>(X, B, L, tab, slot0, nslot, post, Z, slot_stride);
  else
    bot_sweeps_as<T, NOISE, 1, false>(X, B, L, tab, slot0, nslot, post, Z, slot_stride);
}

// r = b - A x on a block level in LDS: a thread takes a column of cells (or a part of one, so
// that the whole work-group has work) and marches up z, forming each plane's two in-plane sums
// once and keeping the five that the current cell reaches.
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
    for (int d = 0; d < 5; ++d) ro[d] = wrapm(y + d - 2, ny) * sy + x;
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
      T rm[5], ra[5];
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        const T* v = P + ro[d];
        const T e = v[0] + v[4], f = v[1] + v[3], c = v[2];
        rm[d] = fma(s1d[0], e, fma(s1d[1], f, s1d[2] * c));
        ra[d] = fma(s1d[5], e, fma(s1d[6], f, s1d[7] * c));
      }
      const T* my = s1d + 10;
      const T* ay = s1d + 15;
      T a0 = my[2] * rm[2], a1 = ay[2] * rm[2], a2 = my[2] * ra[2];
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        a0 = fma(my[d], rm[d] + rm[4 - d], a0);
        a1 = fma(ay[d], rm[d] + rm[4 - d], a1);
        a2 = fma(my[d], ra[d] + ra[4 - d], a2);
      }
      p0[4] = a0;
      p1[4] = a1 + a2;
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

template <typename T, bool NOISE>
__device__ __forceinline__ void bottom_body(const BotArgs& a, const uint32_t comp,
                                            const NoiseArgs& na, int part) {
  extern __shared__ char smraw[];
  T* sm = reinterpret_cast<T*>(smraw);
  const int tid = threadIdx.x;
  const BotLevel& L0 = a.lv[0];
  const int n0 = L0.nx * L0.ny * L0.nz;
  // element of the LDS field x for the natural index q of level L, halo copies beside it
  auto place = [](const BotLevel& L, int q, int& x) {
    int y, z, r;
    divmod_uniform(q, L.nx, r, x);
    divmod_uniform(r, L.ny, z, y);
    return z * L.sz + y * L.sy + x + (L.kind == KIND_BLOCK ? kBotHalo : 0);
  };
  if (part == BOT_UP) {  // x and b of every block level, and the coarsest x, as BOT_DOWN left them
    for (int i = 0; i < a.nlev; ++i) {
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
  } else {
    T* x0 = sm + a.lds_off[0];
    for (int q = tid; q < L0.nz * L0.sz; q += BOT_TPB) x0[q] = T(0);
    T* b0 = x0 + L0.nz * L0.sz;
    const gptr<T> bg = global_ptr<T>(a.b_in) + (size_t)comp * n0;
    for (int q = tid; q < n0; q += BOT_TPB) b0[q] = bg[q];
  }
  // operator tables of the block levels (bot_table_elems) at tab_off[i]; the normals
  // of the coarsest draw, which depend on nothing above it
  for (int i = 0; i < a.nlev; ++i) {
    const BotLevel& L = a.lv[i];
    if (L.kind == KIND_BLOCK) {
      const int nz = L.nz;
      T* t = sm + a.tab_off[i];
      const gptr<T> zt = global_ptr<T>(L.zt), bf = global_ptr<T>(L.bfac);
      for (int q = tid; q < nz * 10; q += BOT_TPB) t[q] = zt[q];
      for (int q = tid; q < (nz / 2) * kBotRow; q += BOT_TPB) {
        const int bz = q / kBotRow, e = q - bz * kBotRow;
        t[nz * 10 + q] = bf[bz * kBlockRow + (e < 64 ? e : e - 64 + kBlockZ)];
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
  for (int i = 0; i < a.nlev && part != BOT_UP; ++i) {
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
    bot_sweeps<T, NOISE>(xi, bi, L, tab, 0, a.nu1, false, Z, zs);
    if (i == a.nlev - 1) {
      // smoothing-only coarsest level: the post-sweeps follow at once
      bot_sweeps<T, NOISE>(xi, bi, L, tab, a.nu1, a.nu2, true, Z, zs);
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
    bot_residual<T>(ri, xi, bi, L, tab);
    __syncthreads();
    const BotLevel& C = a.lv[i + 1];
    T* xc = sm + a.lds_off[i + 1];
    T* bc = xc + C.nz * C.sz;
    for (int q = tid; q < C.nz * C.sz; q += BOT_TPB) xc[q] = T(0);
    for (int q = tid; q < C.nx * C.ny * C.nz; q += BOT_TPB) {
      int X, Y, Z2, r;
      divmod_uniform(q, C.nx, r, X);
      divmod_uniform(r, C.ny, Z2, Y);
      bc[q] = restrict_at<T>(ri, L.nx, L.nx * L.ny, L.nx, L.ny, L.nz, X, Y, Z2);
    }
    __syncthreads();
  }
  for (int i = last - 1; i >= 0; --i) {
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
    bot_sweeps<T, NOISE>(xi, xi + L.nz * L.sz, L, sm + a.tab_off[i], a.nu1, a.nu2, true,
                         global_ptr<T>(L.noise) + (size_t)comp * n, (size_t)a.ncomp * n);
  }
  for (int q = tid; q < n0; q += BOT_TPB) {
    int x;
    ((T*)a.x_out)[(size_t)comp * n0 + q] = sm[a.lds_off[0] + place(L0, q, x)];
  }
}

// One hierarchy, one work-group per component.
template <typename T, bool NOISE>
__global__ __launch_bounds__(BOT_TPB)
__attribute__((amdgpu_waves_per_eu(2, 2))) void k_bottom(const BotArgs* __restrict__ ap, int c0,
                                                    int part, NoiseArgs na) {
  bottom_body<T, NOISE>(*ap, c0 + (int)blockIdx.x, na, part);
}

// Several hierarchies (of any sizes) in one launch: work-group w runs component wg >> 16 of
// item wg & 0xffff, with that item's level descriptors and noise keys, so the latency-bound
// bottoms of uneven instances overlap instead of running one launch after another.
template <typename T, bool NOISE>
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
  bottom_body<T, NOISE>(*it.args, w >> 16, na, it.part);
}

}  // namespace

template <typename T>
hipError_t launch_bottom(const BotArgs* a, int ncomp, int c0, size_t lds, bool noise, int part,
                         const NoiseArgs& na, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)k_bottom<T, true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess)
      e = hipFuncSetAttribute((const void*)k_bottom<T, false>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  if (noise) k_bottom<T, true><<<ncomp, BOT_TPB, lds, s>>>(a, c0, part, na);
  else k_bottom<T, false><<<ncomp, BOT_TPB, lds, s>>>(a, c0, part, na);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_bottom_multi(const BotMultiArgs& m, int nwg, size_t lds, bool noise,
                               hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)k_bottom_multi<T, true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess)
      e = hipFuncSetAttribute((const void*)k_bottom_multi<T, false>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  if (nwg <= 0) return hipSuccess;
  if (nwg > kBotMultiWG || m.nitems > kBotMultiItems) return hipErrorInvalidValue;
  if (noise) k_bottom_multi<T, true><<<nwg, BOT_TPB, lds, s>>>(m);
  else k_bottom_multi<T, false><<<nwg, BOT_TPB, lds, s>>>(m);
  return hipGetLastError();
}

#define SMG_INST(T)                                                                  \
  template hipError_t launch_bottom<T>(const BotArgs*, int, int, size_t, bool, int,  \
                                       const NoiseArgs&, hipStream_t);               \
  template hipError_t launch_bottom_multi<T>(const BotMultiArgs&, int, size_t, bool, \
                                             hipStream_t);
SMG_INST(double)
SMG_INST(float)
#undef SMG_INST

}  // namespace smg
