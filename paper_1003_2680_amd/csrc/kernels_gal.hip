// Galerkin-level kernels: 2x2x2 block heat bath, residual, restriction, prolongation and the
// coarsest exact draw (the LDS-resident bottom of the V-cycle is in kernels_bottom.hip).
//
// Sec. "Stochastic Multigrid Methods": the coarse operators are Galerkin, A^(l+1) = P^T A^(l) P,
// which makes them 81-point (level 1) and 125-point (deeper) stencils.  Two cells of one
// red-black colour are coupled there, so each colour class is a set of 2x2x2 blocks
// (colour (bx%2) + 2(by%2) + 4(bz%2)); blocks of one colour are >= 3 cells apart and every
// block is redrawn from its exact 8-variable conditional law.
#include <hip/hip_runtime.h>

#include <algorithm>

#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"

namespace smg {
namespace {

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + TPB - 1) / TPB); }

// Block-level noise for whole sweeps, ready for the block passes: one thread per block draws
// the block's eight normals (Philox calls 4 bid .. 4 bid + 3, cells k = 2m, 2m+1 of call m) and
// writes sqrt(kT) L_BB^-T n, L_BB^-T being upper triangular.  When a wave's 64 blocks lie in
// one block row (the level's blocks per layer a multiple of 64) the factor rows are uniform
// and are read with scalar loads as FMA operands.  Grid: x over the blocks of one (sweep slot,
// component) of the largest level, y = level entry, z = slot * nact + component.
template <typename T, bool UNIFORM>
__device__ __forceinline__ void colour_block_noise(const T* __restrict__ W, const T (&n)[8],
                                                   T (&e)[8]) {
  typedef const __attribute__((address_space(4))) T* cptr;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    T acc = 0;
#pragma unroll
    for (int j = k; j < 8; ++j) acc = fma(UNIFORM ? ((cptr)W)[k * 8 + j] : W[k * 8 + j], n[j], acc);
    e[k] = acc;
  }
}

// POINT: some entry is a point level (with its branch the FP64 form has 78 registers, 68 without: one
// wave a SIMD less, 2 % of the time of 128^3 x 24).
template <typename T, bool POINT>
__global__ __launch_bounds__(TPB) void k_level_noise(NoiseGenArgs a, NoiseArgs na) {
  using V2 = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
  const NoiseLevel& L = a.lv[blockIdx.y];
  const uint32_t N = (uint32_t)L.nx * L.ny * L.nz;
  const uint32_t bid = blockIdx.x * TPB + threadIdx.x;  // block within (slot, comp)
  const uint32_t s = blockIdx.z / (uint32_t)a.nact;
  const uint32_t comp = blockIdx.z - s * (uint32_t)a.nact;
  if (POINT && !L.bfac) {
    // a point level: N/4 calls a colour, four of the N/2 a thread, neighbours side by side
    const uint32_t per = (N / 2 + 3) / 4;
    if (bid >= per || (int)s >= L.nslot) return;
    T* out = (T*)L.out + ((size_t)s * a.ncomp + comp) * N;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uint32_t q = bid + m * per, c = q >= N / 4 ? 1u : 0u;
      if (q >= N / 2) return;
      const uint32_t sid = (uint32_t)L.level | ((uint32_t)(L.slot0 + s) << 4) | (c << 12);
      T z0, z1;
      if constexpr (sizeof(T) == 8) normal_pair_notable(na, sid, comp, q - c * (N / 4), z0, z1);
      else normal_pair_t<T>(na, sid, comp, q - c * (N / 4), z0, z1);
      V2 v;
      v.x = z0;
      v.y = z1;
      *reinterpret_cast<V2*>(out + 2 * q) = v;
    }
    return;
  }
  if (bid >= (N >> 3) || (int)s >= L.nslot) return;
  const uint32_t nbx = (uint32_t)L.nx >> 1, nby = (uint32_t)L.ny >> 1;
  const uint32_t bz = udiv(bid, nbx * nby, L.lg_bxy);
  const uint32_t rem = bid - bz * nbx * nby;
  const uint32_t by = udiv(rem, nbx, L.lg_bx);
  const uint32_t bx = rem - by * nbx;
  const int colour = (bx & 1) + 2 * (by & 1) + 4 * (bz & 1);
  const uint32_t sid = (uint32_t)L.level | ((uint32_t)(L.slot0 + s) << 4) | ((uint32_t)colour << 12);
  T n[8], e[8];
#pragma unroll
  for (int m = 0; m < 4; ++m) normal_pair_t<T>(na, sid, comp, 4 * bid + m, n[2 * m], n[2 * m + 1]);
  if ((nbx * nby) % 64 == 0) {
    const uint32_t bzu = __builtin_amdgcn_readfirstlane(bz);
    colour_block_noise<T, true>((const T*)L.bfac + (size_t)bzu * kBlockRow<T> + 64, n, e);
  } else {
    colour_block_noise<T, false>((const T*)L.bfac + (size_t)bz * kBlockRow<T> + 64, n, e);
  }
  const T sq = (T)na.sqkT;
  T* out = (T*)L.out + ((size_t)s * a.ncomp + comp) * N;
#pragma unroll
  for (int m = 0; m < 4; ++m) {  // cells k = 2m, 2m+1: one row of the block (dy, dz) = (m&1, m>>1)
    const uint32_t c0 = ((2 * bz + (m >> 1)) * L.ny + (2 * by + (m & 1))) * L.nx + 2 * bx;
    V2 v;
    v.x = sq * e[2 * m];
    v.y = sq * e[2 * m + 1];
    *reinterpret_cast<V2*>(out + c0) = v;
  }
}

// One block-colour pass, LDS-staged.  A work-group owns a TI x TJ tile of the colour's blocks in
// one block layer (bz = 2l + colour/4) and stages the box of cells within 2 of them
// ((4TI+2) x (4TJ+2) x 6, periodic in x and y, wall planes clamped: their z-factors are zero)
// with coalesced row loads; the 125-point rows are then gathered from LDS.  The box never
// contains another work-group's blocks of this colour (blocks of one colour are >= 3 cells
// apart), so staging and the writes of other work-groups do not overlap.
// Tile shapes (blocks per work-group along x, y): 4x4 (128 threads), 4x2 (one wavefront) and
// 8x4 (256 threads); the shape changes only the work distribution, never a result.
constexpr int TILE_D = 6;

// The pass of one work-group: wg = (tile, block layer l, component).
template <typename T, int KIND, int TILE_I, int TILE_J>
__device__ __forceinline__ void block_tile_body(T* __restrict__ xg, const T* __restrict__ bg,
                                                const T* __restrict__ s1d,
                                                const T* __restrict__ bfac, int nx, int ny,
                                                int nz, uint32_t N, int colour, int nbx2,
                                                int nby2, int ntx, const T* __restrict__ zn,
                                                const Blk3 wg) {
  constexpr bool NOISE = KIND == CYCLE_NOISE;
  // rows of 2 mod 4 elements (see block_plane_stride)
  constexpr int TILE_W = 4 * TILE_I + 2, TILE_H = 4 * TILE_J + 2;
  constexpr int TILE_TPB = TILE_I * TILE_J * 8;
  constexpr int TP = block_plane_stride(TILE_H * TILE_W + 1, sizeof(T));  // + a pad element
  __shared__ T Tl[TILE_D * TP];
  const uint32_t comp = wg.z;
  const int l = wg.y;
  const int ti = wg.x % ntx, tj = wg.x / ntx;
  const int cx = colour & 1, cy = (colour >> 1) & 1;
  const int bz = 2 * l + (colour >> 2);
  const int i0 = ti * TILE_I, j0 = tj * TILE_J;
  const int x0 = 4 * i0 + 2 * cx - 2, y0 = 4 * j0 + 2 * cy - 2, z0 = 2 * bz - 2;
  T* X = xg + (size_t)comp * N;
  const int tid = threadIdx.x;
  // this lane's cell: its b and noise loads go out before the tile is staged
  const int k = tid & 7;
  const int il = (tid >> 3) % TILE_I, jl = (tid >> 3) / TILE_I;
  const int i = i0 + il, j = j0 + jl;
  const bool active = i < nbx2 && j < nby2;
  const int bx = 2 * i + cx, by = 2 * j + cy;
  const int kx = k & 1, ky = (k >> 1) & 1, kz = k >> 2;
  const int tx = 4 * il + 2 + kx, ty = 4 * jl + 2 + ky, tz = 2 + kz;
  const int gcx = 2 * bx + kx, gcy = 2 * by + ky, gcz = 2 * bz + kz;
  const uint32_t cell = ((uint32_t)gcz * ny + gcy) * nx + gcx;
  T bk = 0, nrm = 0;
  if (active) {
    bk = bg[(size_t)comp * N + cell];
    if (NOISE) nrm = zn[(size_t)comp * N + cell];
  }
  // stage the box: each thread owns up to PPT (x, y) positions of a plane and loads them in all
  // TILE_D planes; every load is issued before the first LDS store, so the work-group waits for
  // global memory once, and the index arithmetic is done once per position, not per element
  constexpr int PLANE = TILE_W * TILE_H;
  constexpr int PPT = (PLANE + TILE_TPB - 1) / TILE_TPB;
  int goff[PPT], loff[PPT];
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    const int pos = tid + p * TILE_TPB;
    const int sx = pos % TILE_W, sy = pos / TILE_W;
    // positions past the plane store into its pad element: no branch
    loff[p] = pos < PLANE ? pos : PLANE;
    goff[p] = pos < PLANE ? wrap_near(y0 + sy, ny) * nx + wrap_near(x0 + sx, nx) : 0;
  }
  T stage[TILE_D][PPT];
#pragma unroll
  for (int sz = 0; sz < TILE_D; ++sz) {
    int gz = z0 + sz;
    gz = gz < 0 ? 0 : (gz >= nz ? nz - 1 : gz);
    const T* P = X + (size_t)gz * nx * ny;
#pragma unroll
    for (int p = 0; p < PPT; ++p) stage[sz][p] = P[goff[p]];  // goff = 0 (in range) if unused
  }
#pragma unroll
  for (int sz = 0; sz < TILE_D; ++sz)
#pragma unroll
    for (int p = 0; p < PPT; ++p) Tl[sz * TP + loff[p]] = stage[sz][p];
  __syncthreads();
  BlockWeights<T, 1, index_order<T, KIND>> w;
  const T* row = bfac + (size_t)bz * kBlockRow<T>;
  block_row_weights<T>(w, row, kx, ky, kz);
#pragma unroll
  for (int m = 0; m < 3; ++m) w.po[m] = (3 * kz + m) * TP;
  const Stencils<T> st = load_stencils(s1d);
  int ro[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) ro[r] = (ty + (ky ? 2 - r : r - 2)) * TILE_W + tx - 2;
  const T v = block_update<T, 1, false>(Tl, ro, st.v, w, tz * TP + ty * TILE_W + tx, bk, nrm);
  if (active) X[cell] = v;
}

template <typename T, int KIND, int TILE_I, int TILE_J>
__global__ __launch_bounds__(TILE_I * TILE_J * 8) void k_block_tile(T* __restrict__ xg,
                                                          const T* __restrict__ bg,
                                                          const T* __restrict__ s1d,
                                                          const T* __restrict__ bfac, int nx,
                                                          int ny, int nz, uint32_t N, int colour,
                                                          int nbx2, int nby2, int ntx,
                                                          const T* __restrict__ zn) {
  block_tile_body<T, KIND, TILE_I, TILE_J>(xg, bg, s1d, bfac, nx, ny, nz, N, colour, nbx2,
                                            nby2, ntx, zn, xcd_block());
}

// Half a sweep in one launch: the four block colours of one layer parity cz, in sweep order (cy 0
// then 1, within each cx 0 then 1; reversed in a post-sweep).  A block row depends on the rows of
// the other cy on both sides, so a work-group that owns a pair of block rows of one layer over
// the whole (periodic) x-extent also draws the row of the first cy beyond its own (which it does
// not store), and then all the rows that its second cy needs are in its tile.  Every value is
// computed from the same inputs by the same arithmetic as in four single-colour passes, so the
// result is theirs, bit for bit.  The rows a work-group stages are rewritten by its neighbours in
// the same launch, so the layers are read from one field and written to another: xs holds this
// parity's layers before the half-sweep, xo the other parity's, xn receives this parity's.
//
// The tile is HALF_ROWS cell rows of the layer's six planes with two periodic halo cells per row
// side; the first row is the cell row 4 j0 - 2 (pre) or 4 j0 - 4 (post), so that the rows of the
// first cy start at 2 and those of the second at 4 in both.
//
// What bounds it: the launch and the latency of the staging loads, on the levels of few
// components it is used for.  A two-colour launch takes nearly as long (5.9 us at 32^3 x 3, FP64;
// a half-sweep 8.4 us), and a sweep needs four of those: 23.6 -> 16.8 us.
template <typename T, int KIND>
__device__ __forceinline__ void block_half_body(const HalfItem<T>& h, int cz, bool post,
                                                const Blk3 wg) {
  constexpr bool NOISE = KIND == CYCLE_NOISE;
  extern __shared__ char smraw[];
  T* Tl = reinterpret_cast<T*>(smraw);
  const int nx = h.nx, ny = h.ny, nz = h.nz;
  const size_t base = (size_t)wg.z * h.N;
  const int bz = 2 * (int)wg.y + cz, j0 = (int)wg.x;
  const int RS = nx + 2 * kBotHalo + 2;
  const int TP = h.TP;
  const int y0 = 4 * j0 - (post ? 4 : 2), z0 = 2 * bz - 2;
  const int tid = threadIdx.x, nthr = (int)blockDim.x;
  const int kx = tid & 1, ky = (tid >> 1) & 1, kz = (tid >> 2) & 1;
  int il, jl;
  divmod_uniform(tid >> 3, nx >> 2, jl, il);
  const int jr = jl <= 1 ? jl : 0;  // lanes past the tile read inside it and store nothing
  const int gcz = 2 * bz + kz;
  // this lane's cells: row jr of the first cy, then of the second, each at cx = 0 and 1
  uint32_t cell[2];
  T b[2][2], n[2][2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int gy = wrap_near(y0 + 2 + 2 * q + 4 * jr + ky, ny);
    cell[q] = ((uint32_t)gcz * ny + gy) * nx + 4 * il + kx;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      b[q][c] = h.b[base + cell[q] + 2 * c];
      n[q][c] = NOISE ? h.zn[base + cell[q] + 2 * c] : T(0);
    }
  }
  // stage: at most three positions of a plane per thread (10 nx positions, 4 nx threads); all
  // their loads in all six planes are issued before the first store
  constexpr int PPT = 3;
  const int plane = nx * HALF_ROWS;
  int goff[PPT], loff[PPT], hoff[PPT];
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    const int pos = tid + p * nthr;
    const bool in = pos < plane;
    int py, px;
    divmod_uniform(pos, nx, py, px);
    loff[p] = in ? py * RS + px + kBotHalo : -1;
    hoff[p] = px < 2 ? nx : (px >= nx - 2 ? -nx : 0);
    goff[p] = in ? wrap_near(y0 + py, ny) * nx + px : 0;
  }
  T stage[TILE_D][PPT];
#pragma unroll
  for (int sz = 0; sz < TILE_D; ++sz) {
    int gz = z0 + sz;
    gz = gz < 0 ? 0 : (gz >= nz ? nz - 1 : gz);
    const T* S = ((gz >> 1) & 1) == cz ? h.xs : h.xo;
    const T* Pl = S + base + (size_t)gz * ny * nx;
#pragma unroll
    for (int p = 0; p < PPT; ++p) stage[sz][p] = Pl[goff[p]];  // goff = 0 (in range) if unused
  }
#pragma unroll
  for (int sz = 0; sz < TILE_D; ++sz)
#pragma unroll
    for (int p = 0; p < PPT; ++p)
      if (loff[p] >= 0) {
        Tl[sz * TP + loff[p]] = stage[sz][p];
        if (hoff[p]) Tl[sz * TP + loff[p] + hoff[p]] = stage[sz][p];
      }
  __builtin_amdgcn_sched_barrier(0);
  BlockWeights<T, 1, index_order<T, KIND>> w;
  const T* row = h.bfac + (size_t)bz * kBlockRow<T>;
  block_row_weights<T>(w, row, kx, ky, kz);
#pragma unroll
  for (int m = 0; m < 3; ++m) w.po[m] = (3 * kz + m) * TP;
  __syncthreads();
  const Stencils<T> s1d = load_stencils(h.s1d);
  const int wave_row = __builtin_amdgcn_readfirstlane(jl);  // the wave's first block row
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int rows = 2 - q;
    const int ty = 2 + 2 * q + 4 * jr + ky;
    int ro[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) ro[r] = (ty + (ky ? 2 - r : r - 2)) * RS + 4 * il + kx;
    const int at = (2 + kz) * TP + ty * RS + 4 * il + kx + kBotHalo;
    const bool draws = jl < rows;
    // the row beyond the group's own: the second of a pre-sweep's first cy, the first of a post's
    const bool stores = draws && (q == 1 || jl == (post ? 1 : 0));
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (wave_row < rows) {  // whole waves without a row only keep the barrier
        const int cx = post ? 1 - c : c, d = 2 * cx;
        const T v = block_update<T, 1, false>(Tl + d, ro, s1d.v, w, at, cx ? b[q][1] : b[q][0],
                                              cx ? n[q][1] : n[q][0]);
        if (draws) {
          const int x = 4 * il + kx + d;
          T* t = Tl + at + d;
          t[0] = v;
          if (x < 2) t[nx] = v;
          if (x >= nx - 2) t[-nx] = v;
          if (stores) h.xn[base + cell[q] + d] = v;
        }
      }
      if (q == 0 || c == 0) __syncthreads();
    }
  }
}

// Half-sweeps of the levels of several hierarchies (or of one) in one launch: the flat grid
// concatenates the items' (row group, layer, component) grids in XCD-aware order; the block size
// and the LDS are the largest the items need.
template <typename T, int KIND>
__global__ __launch_bounds__(HALF_TPB, 3) void k_block_half(HalfArgs<T> m) {
  const uint32_t lin = xcd_block().x;
  int i = 0;
  while (i + 1 < m.nitems && lin >= m.begin[i + 1]) ++i;
  const HalfItem<T>& it = m.it[i];
  const uint32_t local = lin - m.begin[i];
  Blk3 wg;
  wg.x = local % (uint32_t)it.ngx;
  const uint32_t rest = local / (uint32_t)it.ngx;
  wg.y = rest % (uint32_t)it.nbzc;
  wg.z = rest / (uint32_t)it.nbzc;
  block_half_body<T, KIND>(it, m.cz, m.post != 0, wg);
}

// Two block colours c and c ^ 1 in one launch.  They differ only in the parity of bx, so a
// block of colour c ^ 1 depends on colour-c blocks only through its x-neighbours in the same
// block row and layer.  A work-group owns PJ (4, 2 or 1: see pair_rows) block rows
// by = 2 (j0 + jl) + cy of one block layer bz = 2 l + cz over the whole x-extent (periodic: two
// halo cells per row side), stages the cells within two of them ((4 PJ + 2) rows of 6 planes, wall
// planes clamped), draws colour c into the tile, then colour c ^ 1 from the updated tile, and
// writes both.  No other work-group stages a cell that this one writes (rows of parity cy are
// four cells apart, and rows and layers of the other parity are not written), and every value is
// computed by the arithmetic of the single-colour pass from the same inputs, so the result is that
// of the two single-colour passes in order.  FP64, 64^3 x 24, two rows a group: 28 us a launch
// (before the DPP exchanges, the bank-free plane stride and the packed factors 32 us; VALU
// instructions per wave 753 -> 610, LDS cycles 8.2 M -> 6.1 M a launch).
template <typename T, int KIND>
__device__ __forceinline__ void block_pair_body(const HalfItem<T>& h, int c_first, const Blk3 wg) {
  constexpr bool NOISE = KIND == CYCLE_NOISE;
  extern __shared__ char smraw[];
  T* Tl = reinterpret_cast<T*>(smraw);
  const int nx = h.nx, ny = h.ny, nz = h.nz, PJ = h.P, TP = h.TP;
  const size_t base = (size_t)wg.z * h.N;
  const int cy = (c_first >> 1) & 1, cz = c_first >> 2;
  const int bz = 2 * (int)wg.y + cz, j0 = (int)wg.x * PJ;
  const int H = 4 * PJ + 2, RS = nx + 2 * kBotHalo + 2;
  const int y0 = 4 * j0 + 2 * cy - 2, z0 = 2 * bz - 2;
  const int nthr = (int)blockDim.x;  // >= 2 nx PJ
  T* X = h.xn + base;
  const int tid = threadIdx.x;
  const int kx = tid & 1, ky = (tid >> 1) & 1, kz = (tid >> 2) & 1;
  const int nbx2 = nx >> 2;
  int il, jl;
  divmod_uniform(tid >> 3, nbx2, jl, il);
  const bool active = jl < PJ && j0 + jl < (ny >> 2);
  // lanes past the group's rows take row 0 for addressing only
  const int jr = jl < PJ ? jl : 0;
  const int ty = 4 * jr + 2 + ky;
  const int gcy = wrap_near(y0 + ty, ny), gcz = 2 * bz + kz;
  const uint32_t cell = ((uint32_t)gcz * ny + gcy) * nx + 4 * il + kx;  // at cx = 0
  const T b0 = h.b[base + cell], b1 = h.b[base + cell + 2];
  const T n0 = NOISE ? h.zn[base + cell] : T(0), n1 = NOISE ? h.zn[base + cell + 2] : T(0);
  // stage: a plane has nx (4 PJ + 2) positions and the group 2 nx PJ threads, so every thread
  // owns at most three positions; all their loads in all six planes are issued before the first
  // store, so the group waits for memory once
  constexpr int PPT = 3;
  const int plane = nx * H;
  int goff[PPT], loff[PPT], hoff[PPT];
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    const int pos = tid + p * nthr;
    const bool in = pos < plane;
    int py, px;
    divmod_uniform(pos, nx, py, px);
    loff[p] = in ? py * RS + px + kBotHalo : -1;
    hoff[p] = px < 2 ? nx : (px >= nx - 2 ? -nx : 0);
    goff[p] = in ? wrap_near(y0 + py, ny) * nx + px : 0;
  }
  T stage[TILE_D][PPT];
#pragma unroll
  for (int sz = 0; sz < TILE_D; ++sz) {
    int gz = z0 + sz;
    gz = gz < 0 ? 0 : (gz >= nz ? nz - 1 : gz);
    const T* Pl = X + (size_t)gz * ny * nx;
#pragma unroll
    for (int p = 0; p < PPT; ++p) stage[sz][p] = Pl[goff[p]];  // goff = 0 (in range) if unused
  }
#pragma unroll
  for (int sz = 0; sz < TILE_D; ++sz)
#pragma unroll
    for (int p = 0; p < PPT; ++p)
      if (loff[p] >= 0) {
        Tl[sz * TP + loff[p]] = stage[sz][p];
        if (hoff[p]) Tl[sz * TP + loff[p] + hoff[p]] = stage[sz][p];
      }
  __builtin_amdgcn_sched_barrier(0);
  BlockWeights<T, 1, index_order<T, KIND>> w;
  const T* row = h.bfac + (size_t)bz * kBlockRow<T>;
  block_row_weights<T>(w, row, kx, ky, kz);
#pragma unroll
  for (int m = 0; m < 3; ++m) w.po[m] = (3 * kz + m) * TP;
  __syncthreads();
  const Stencils<T> s1d = load_stencils(h.s1d);
  const int cx0 = c_first & 1;
  int ro[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) ro[r] = (ty + (ky ? 2 - r : r - 2)) * RS + 4 * il + kx;
  const int at = (2 + kz) * TP + ty * RS + 4 * il + kx + kBotHalo;
  // colour c is written into the tile in place: blocks of one colour never read each other's
  // cells, and the eight lanes of a block are one wave, whose reads precede its writes
  {
    const int d = 2 * cx0, x = 4 * il + kx + d;
    const T v = block_update<T, 1, false>(Tl + d, ro, s1d.v, w, at, cx0 ? b1 : b0, cx0 ? n1 : n0);
    if (active) {
      T* t = Tl + at + d;
      t[0] = v;
      if (x < 2) t[nx] = v;
      if (x >= nx - 2) t[-nx] = v;
      X[cell + d] = v;
    }
  }
  __syncthreads();
  {
    const int d = 2 - 2 * cx0;
    const T v = block_update<T, 1, false>(Tl + d, ro, s1d.v, w, at, cx0 ? b0 : b1, cx0 ? n0 : n1);
    if (active) X[cell + d] = v;
  }
}

// Two-colour launches of the levels of several hierarchies (or of one) in one launch, as
// k_block_half.
template <typename T, int KIND>
__global__ __launch_bounds__(HALF_TPB) void k_block_pair(HalfArgs<T> m) {
  const uint32_t lin = xcd_block().x;
  int i = 0;
  while (i + 1 < m.nitems && lin >= m.begin[i + 1]) ++i;
  const HalfItem<T>& it = m.it[i];
  const uint32_t local = lin - m.begin[i];
  Blk3 wg;
  wg.x = local % (uint32_t)it.ngx;
  const uint32_t rest = local / (uint32_t)it.ngx;
  wg.y = rest % (uint32_t)it.nbzc;
  wg.z = rest / (uint32_t)it.nbzc;
  block_pair_body<T, KIND>(it, m.cz, wg);
}

// The same pass for several levels of different hierarchies (one colour) in one launch: the
// one-dimensional grid is the concatenation of every item's (tile, layer, component) grid, in
// XCD-aware order; a work-group finds its item from the offsets and runs the item's pass.
template <typename T, int KIND, int TILE_I, int TILE_J>
__global__ __launch_bounds__(TILE_I * TILE_J * 8) void k_block_tile_multi(BlockMultiArgs<T> m) {
  const uint32_t lin = xcd_block().x;
  int i = 0;
  while (i + 1 < m.nitems && lin >= m.begin[i + 1]) ++i;
  const BlockMultiItem<T>& it = m.it[i];
  const uint32_t local = lin - m.begin[i];
  const uint32_t tiles = (uint32_t)it.ntx * (uint32_t)it.nty;
  Blk3 wg;
  wg.x = local % tiles;
  const uint32_t rest = local / tiles;
  wg.y = rest % (uint32_t)it.nbzc;
  wg.z = rest / (uint32_t)it.nbzc;
  block_tile_body<T, KIND, TILE_I, TILE_J>(it.x, it.b, it.s1d, it.bfac, it.nx, it.ny,
                                            it.nz, it.N, m.colour, it.nbx2, it.nby2, it.ntx,
                                            it.zn, wg);
}

// r = b - A x on a Galerkin level, LDS-tiled: a work-group owns GR_X x GR_Y x GR_Z cells and
// stages the box within 2 of them; a thread takes a z-column of GR_Z cells and forms each of
// the GR_Z + 4 staged planes' two partial sums once, adding them into every cell of the
// column they reach, plane by plane in index order.
constexpr int GR_X = 16, GR_Y = 16, GR_Z = 4;
constexpr int GR_SX = GR_X + 4, GR_SY = GR_Y + 4, GR_SZ = GR_Z + 4;

template <typename T>
__global__ __launch_bounds__(TPB) void k_residual_gal_tile(T* __restrict__ r,
                                                            const T* __restrict__ xg,
                                                            const T* __restrict__ bg,
                                                            const T* __restrict__ s1d,
                                                            const T* __restrict__ zt, int nx,
                                                            int ny, int nz, int ntx) {
  __shared__ T Xs[GR_SZ * GR_SY * GR_SX];
  const Blk3 wg = xcd_block();
  const uint32_t comp = wg.z;
  const int X0 = (wg.x % ntx) * GR_X, Y0 = (wg.x / ntx) * GR_Y, Z0 = wg.y * GR_Z;
  const size_t N = (size_t)nx * ny * nz;
  const T* X = xg + comp * N;
  const int tid = threadIdx.x;
  {
    constexpr int PLANE = GR_SX * GR_SY;
    constexpr int PPT = (PLANE + TPB - 1) / TPB;
    int goff[PPT], loff[PPT];
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
      const int pos = tid + p * TPB;
      const int sx = pos % GR_SX, sy = pos / GR_SX;
      loff[p] = pos < PLANE ? sy * GR_SX + sx : -1;
      goff[p] = pos < PLANE ? wrap_near(Y0 - 2 + sy, ny) * nx + wrap_near(X0 - 2 + sx, nx) : 0;
    }
    T st[GR_SZ][PPT];
#pragma unroll
    for (int sz = 0; sz < GR_SZ; ++sz) {
      int gz = Z0 - 2 + sz;
      gz = gz < 0 ? 0 : (gz >= nz ? nz - 1 : gz);
#pragma unroll
      for (int p = 0; p < PPT; ++p) st[sz][p] = X[(size_t)gz * nx * ny + goff[p]];
    }
#pragma unroll
    for (int sz = 0; sz < GR_SZ; ++sz)
#pragma unroll
      for (int p = 0; p < PPT; ++p)
        if (loff[p] >= 0) Xs[sz * PLANE + loff[p]] = st[sz][p];
  }
  __syncthreads();
  const int lx = tid % GR_X, ly = tid / GR_X;
  const int cx = X0 + lx, cy = Y0 + ly;
  const int xs[5] = {lx, lx + 1, lx + 2, lx + 3, lx + 4};
  const int ys[5] = {ly, ly + 1, ly + 2, ly + 3, ly + 4};
  const int kmax = nz - Z0 < GR_Z ? nz - Z0 : GR_Z;
  T acc0[GR_Z], acc1[GR_Z];
#pragma unroll
  for (int k = 0; k < GR_Z; ++k) acc0[k] = acc1[k] = T(0);
#pragma unroll
  for (int p = 0; p < GR_SZ; ++p) {
    T p1;
    const T p0 = gal_plane<T>(Xs + p * (GR_SX * GR_SY), GR_SX, xs, ys, s1d, p1);
#pragma unroll
    for (int k = 0; k < GR_Z; ++k) {
      const int dz = p - k;  // plane offset + 2 seen from cell Z0 + k
      if (dz < 0 || dz > 4 || k >= kmax) continue;
      const T* zr = zt + (Z0 + k) * 10;
      acc0[k] = fma(zr[dz], p0, acc0[k]);
      acc1[k] = fma(zr[5 + dz], p1, acc1[k]);
    }
  }
  if (cx >= nx || cy >= ny) return;
#pragma unroll
  for (int k = 0; k < GR_Z; ++k) {
    if (k >= kmax) break;
    const size_t i = comp * N + ((size_t)(Z0 + k) * ny + cy) * nx + cx;
    r[i] = bg[i] - (acc0[k] + acc1[k]);
  }
}

// b_c = P^T (b - A x) on a Galerkin level axis by axis, and x_c = 0: as k_fold_residual0, with the
// eight-tap folds of m and a along x and y (symmetric: four coefficients each) and the rows of a_z
// and m_z along z.  A fine row leaves u = Px^T m_x x, v = Px^T a_x x and w = Px^T b per coarse
// column, these p0 = Py^T m_y u, p1 = Py^T (a_y u + m_y v) and q = Py^T w per coarse row; a plane's
// p0, p1 go into the five z-rows that they reach, and a finished row into its two coarse layers.
// A lane forms two coarse columns of a row from its four cells (16-byte loads) and three beside
// them on either side, from the neighbouring lanes by DPP moves and, for the end lanes of a row, by
// loads of their own.  us, residual kernel + restriction / here (FP64): 64^3 x 24 57 + 27 / 33, x 3
// 11.9 + 5.8 / 11.1, 256x256x128 73 + 35 / 36.
constexpr int FOLD_Z = 16;  // coarse layers a work-group at most
template <int RX, int NT>
struct FoldG {
  static constexpr int RY = TPB / RX;
  static constexpr int YS = 2 * RY + 6;  // rows 2Y0 - 3 .. 2Y0 + 2RY + 2
  static constexpr int ITEMS = RX * YS;
  static constexpr int LANES = RX / 2, ROWS = NT / LANES;
  static constexpr int IPT = (YS + ROWS - 1) / ROWS;
};

template <typename T, int RX, int NT>
__global__ __launch_bounds__(NT) void k_fold_residual(T* __restrict__ bc, T* __restrict__ xc,
                                                        const T* __restrict__ xg,
                                                        const T* __restrict__ bg,
                                                        const T* __restrict__ zt, int nx, int ny,
                                                        int nz, int ntx, int zper,
                                                        FoldTaps<T> m) {
  using F = FoldG<RX, NT>;
  using V2 = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
  __shared__ __attribute__((aligned(16))) T Us[2][F::ITEMS], Vs[2][F::ITEMS], Ws[2][F::ITEMS];
  __shared__ T Zt[(2 * FOLD_Z + 10) * 10];  // the z-rows that the run's planes reach
  const Blk3 wg = xcd_block();
  const uint32_t comp = wg.z;
  const int nxc = nx >> 1, nyc = ny >> 1, nzc = nz >> 1;
  const int X0 = (int)(wg.x % (uint32_t)ntx) * RX, Y0 = (int)(wg.x / (uint32_t)ntx) * F::RY;
  const int Z0 = (int)wg.y * zper, Z1 = min(Z0 + zper, nzc);
  const size_t plane = (size_t)nx * ny, N = plane * nz;
  const T *X = xg + comp * N, *B = bg + comp * N;
  const int tid = threadIdx.x;
  const int lr = tid & (F::LANES - 1);
  const bool first = lr == 0, last = lr == F::LANES - 1;
  // cell offsets within a plane: the lane's four, and the four beside them of an end lane
  uint32_t em[F::IPT], eh[F::IPT];
  int at[F::IPT];
#pragma unroll
  for (int k = 0; k < F::IPT; ++k) {
    const int row = tid / F::LANES + k * F::ROWS;
    at[k] = row < F::YS ? row * RX + 2 * lr : -1;
    const uint32_t y = (uint32_t)wrap_near(2 * Y0 - 3 + (row < F::YS ? row : 0), ny) * nx;
    int x = X0 + 2 * lr;  // lanes beyond the grid hold its periodic continuation
    x = 2 * (x < nxc ? x : (x < 2 * nxc ? x - nxc : 0));
    em[k] = y + x;
    eh[k] = y + (first ? (x == 0 ? nx - 4 : x - 4) : (x + 4 == nx ? 0 : x + 4));
  }
  V2 x0[F::IPT], x1[F::IPT], b0[F::IPT], b1[F::IPT], h0[F::IPT], h1[F::IPT], hb[F::IPT];
  auto ld = [](const T* p) { return *reinterpret_cast<const V2*>(p); };
  auto load = [&](int f) {
    const T *P = X + f * plane, *Q = B + f * plane;
#pragma unroll
    for (int k = 0; k < F::IPT; ++k) {
      x0[k] = ld(P + em[k]);
      x1[k] = ld(P + em[k] + 2);
      b0[k] = ld(Q + em[k]);
      b1[k] = ld(Q + em[k] + 2);
      if (first || last) {
        h0[k] = ld(P + eh[k]);
        h1[k] = ld(P + eh[k] + 2);
        hb[k] = ld(Q + eh[k] + (first ? 2 : 0));
      }
    }
  };
  const T q1 = T(0.25), q3 = T(0.75);
  const int lx = tid % RX, ly = tid / RX;
  const bool owner = tid < TPB && X0 + lx < nxc && Y0 + ly < nyc;
  const size_t out = (size_t)comp * nxc * nyc * nzc + (size_t)(Y0 + ly) * nxc + X0 + lx;
  const size_t cplane = (size_t)nxc * nyc;
  auto emit = [&](int Z, T a) {
    if (Z < Z0 || Z >= Z1 || !owner) return;
    bc[out + Z * cplane] = a;
    if (xc) xc[out + Z * cplane] = T(0);
  };
  // r[j]: the residual of z-row f - 2 + j so far; lo, hi: the coarse layers that it goes into
  T r[5] = {}, lo = T(0), hi = T(0);
  const int f0 = max(0, 2 * Z0 - 3), f1 = 2 * Z1 + 2;
  load(f0);
  for (int q = tid; q < (f1 - f0 + 5) * 10; q += NT) {
    const int z = min(max(f0 - 2 + q / 10, 0), nz - 1);  // a row beyond a wall is never used
    Zt[q] = zt[z * 10 + q % 10];
  }
#pragma unroll 1
  for (int f = f0; f <= f1; ++f) {
    const int buf = f & 1;
    if (f < nz) {
#pragma unroll
      for (int k = 0; k < F::IPT; ++k) {
        const T c0 = x0[k].x, c1 = x0[k].y, c2 = x1[k].x, c3 = x1[k].y;
        T l1 = dpp_lane<DPP_BEFORE>(c1), l2 = dpp_lane<DPP_BEFORE>(c2),
          l3 = dpp_lane<DPP_BEFORE>(c3);
        T r4 = dpp_lane<DPP_AFTER>(c0), r5 = dpp_lane<DPP_AFTER>(c1), r6 = dpp_lane<DPP_AFTER>(c2);
        T bl = dpp_lane<DPP_BEFORE>(b1[k].y), bh = dpp_lane<DPP_AFTER>(b0[k].x);
        l1 = first ? h0[k].y : l1;
        l2 = first ? h1[k].x : l2;
        l3 = first ? h1[k].y : l3;
        bl = first ? hb[k].y : bl;
        r4 = last ? h0[k].x : r4;
        r5 = last ? h0[k].y : r5;
        r6 = last ? h1[k].x : r6;
        bh = last ? hb[k].x : bh;
        const T ea[4] = {l1 + r4, l2 + c3, l3 + c2, c0 + c1};
        const T eb[4] = {l3 + r6, c0 + r5, c1 + r4, c2 + c3};
        V2 u, v, w;
        u.x = u.y = v.x = v.y = T(0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          u.x = fma(m.mx[t], ea[t], u.x);
          u.y = fma(m.mx[t], eb[t], u.y);
          v.x = fma(m.ax[t], ea[t], v.x);
          v.y = fma(m.ax[t], eb[t], v.y);
        }
        w.x = fma(q3, b0[k].x + b0[k].y, q1 * (bl + b1[k].x));
        w.y = fma(q3, b1[k].x + b1[k].y, q1 * (b0[k].y + bh));
        if (at[k] >= 0) {
          *reinterpret_cast<V2*>(&Us[buf][at[k]]) = u;
          *reinterpret_cast<V2*>(&Vs[buf][at[k]]) = v;
          *reinterpret_cast<V2*>(&Ws[buf][at[k]]) = w;
        }
      }
      if (f + 1 < nz && f < f1) load(f + 1);
      __syncthreads();
      if (tid >= TPB) continue;  // more lanes than columns: whole waves
      const int o = 2 * ly * RX + lx;
      T p0 = T(0), p1 = T(0);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const T u = Us[buf][o + t * RX] + Us[buf][o + (7 - t) * RX];
        const T v = Vs[buf][o + t * RX] + Vs[buf][o + (7 - t) * RX];
        p0 = fma(m.my[t], u, p0);
        p1 = fma(m.ay[t], u, fma(m.my[t], v, p1));
      }
      const T* W = &Ws[buf][o];
      r[2] += fma(q3, W[3 * RX] + W[4 * RX], q1 * (W[2 * RX] + W[5 * RX]));
      const T* zr = &Zt[(f - f0) * 10];  // row f - 2 + j holds plane f at its offset 2 - j
#pragma unroll
      for (int j = 0; j < 5; ++j) r[j] = fma(-zr[j * 10 + 4 - j], p0, fma(-zr[j * 10 + 9 - j], p1, r[j]));
    }
    // row z = f - 2 has all its planes
    const int z = f - 2, Z = z >> 1;
    if (z >= 0 && z < nz) {
      if (z & 1) {
        lo = fma(Z == nzc - 1 ? T(0.5) : q3, r[0], lo);
        hi = fma(q1, r[0], hi);
      } else {
        lo = fma(q1, r[0], lo);
        hi = fma(Z == 0 ? T(0.5) : q3, r[0], hi);
        emit(Z - 1, lo);
        lo = hi;
        hi = T(0);
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = r[j + 1];
    r[4] = T(0);
  }
  if (Z1 == nzc) emit(nzc - 1, lo);  // no plane above the layer at the upper wall
}

// b_c = P^T r, and x_c = 0 (the coarse iterate of Alg. 3 starts from zero)
template <typename T>
__global__ __launch_bounds__(TPB) void k_restrict(T* __restrict__ bc, T* __restrict__ xc,
                                                   const T* __restrict__ r, int nxf, int nyf,
                                                   int nzf, uint32_t Nf, uint32_t Nc) {
  const uint32_t comp = blockIdx.y;
  const uint32_t I = blockIdx.x * TPB + threadIdx.x;
  if (I >= Nc) return;
  const int nxc = nxf >> 1, nyc = nyf >> 1;
  const int X = I % nxc;
  const uint32_t row = I / nxc;
  const int Y = row % nyc;
  const int Z = row / nyc;
  bc[(size_t)comp * Nc + I] =
      restrict_at<T>(r + (size_t)comp * Nf, nxf, nxf * nyf, nxf, nyf, nzf, X, Y, Z);
  if (xc) xc[(size_t)comp * Nc + I] = T(0);
}

template <typename T>
__global__ __launch_bounds__(TPB) void k_prolong(T* __restrict__ x, const T* __restrict__ e,
                                                  int nxf, int nyf, int nzf, uint32_t Nf,
                                                  uint32_t Nc) {
  const uint32_t comp = blockIdx.y;
  const uint32_t i = blockIdx.x * TPB + threadIdx.x;
  if (i >= Nf) return;
  const int xf = i % nxf;
  const uint32_t row = i / nxf;
  const int yf = row % nyf;
  const int zf = row / nyf;
  const int nxc = nxf >> 1, nyc = nyf >> 1;
  x[(size_t)comp * Nf + i] +=
      prolong_at<T>(e + (size_t)comp * Nc, nxc, nxc * nyc, xf, yf, zf, nxc, nyc, nzf >> 1);
}

// x = A_c^-1 b (+ sqrt(kT) L_c^-T n) in FP64.  A work-group owns CO_ROWS rows of C components
// and splits the columns over CO_TPB / CO_ROWS lanes per row, so that the dense factors (the
// bound: 12 n^2 bytes, from L2 or memory) are read by the whole chip, in 128-byte segments, with
// eight loads per lane in flight; the components of a group share every factor element.  b and
// the normals that the rows need (columns from the first row on: L_c^-T is upper triangular) are
// staged in LDS.  A lane's columns and the order of the sums do not depend on the grid, so a
// component's draw is the same bits in any launch.
// One work-group per component took 3469 us at n = 2160 (inside the bottom kernel) and 140-230
// us at n = 512; one thread per row over n / 256 work-groups 40 us at n = 256 (eight components).
constexpr int CO_ROWS = 16, CO_TPB = 512, CO_PARTS = CO_TPB / CO_ROWS;

template <typename T, bool NOISE, int C>
__global__ __launch_bounds__(CO_TPB) void k_coarsest(T* __restrict__ xg,
                                                      const T* __restrict__ bg,
                                                      const double* __restrict__ ainv,
                                                      const double* __restrict__ w, int n,
                                                      int ncomp, bool round, NoiseArgs na) {
  extern __shared__ double sh[];  // b [C][n], normals [C][n]; then the partial sums
  const int comp0 = blockIdx.y * C;
  const int nc = min(C, ncomp - comp0);
  const int row0 = blockIdx.x * CO_ROWS;
  for (int c = 0; c < nc; ++c) {
    const T* B = bg + (size_t)(comp0 + c) * n;
    for (int i = threadIdx.x; i < n; i += CO_TPB) sh[c * n + i] = (double)B[i];
    if (NOISE) {
      double* Z = sh + (C + c) * n;
      for (int q = row0 / 2 + threadIdx.x; 2 * q < n; q += CO_TPB) {
        double z0, z1;
        normal_pair(na, na.sid, comp0 + c, (uint32_t)q, z0, z1);
        Z[2 * q] = round ? (double)(T)z0 : z0;
        if (2 * q + 1 < n) Z[2 * q + 1] = round ? (double)(T)z1 : z1;
      }
    }
  }
  for (int c = nc; c < C; ++c)  // components past the last: zeros, so that the sums need no test
    for (int i = threadIdx.x; i < n; i += CO_TPB) sh[c * n + i] = sh[(C + c) * n + i] = 0.0;
  __syncthreads();
  const int r = threadIdx.x % CO_ROWS, part = threadIdx.x / CO_ROWS;
  const int row = row0 + r, rl = min(row, n - 1);
  double acc[C], an[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = an[c] = 0.0;
#pragma unroll 8
  for (int jj = part; jj < n; jj += CO_PARTS) {
    const double a = ainv[(size_t)jj * n + rl];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = fma(a, sh[c * n + jj], acc[c]);
  }
  if (NOISE) {
    // from the lane's first column at or after row0; entries above the diagonal row are zero
#pragma unroll 8
    for (int jj = row0 + (part - row0 % CO_PARTS + CO_PARTS) % CO_PARTS; jj < n; jj += CO_PARTS) {
      const double a = jj >= rl ? w[(size_t)jj * n + rl] : 0.0;
#pragma unroll
      for (int c = 0; c < C; ++c) an[c] = fma(a, sh[(C + c) * n + jj], an[c]);
    }
  }
  __syncthreads();  // every read of b and the normals is done: the sums take their place
#pragma unroll
  for (int c = 0; c < C; ++c) {
    double v = NOISE ? fma(na.sqkT, an[c], acc[c]) : acc[c];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if ((threadIdx.x & 63) < CO_ROWS) sh[(c * (CO_TPB / 64) + threadIdx.x / 64) * CO_ROWS + r] = v;
  }
  __syncthreads();
  const int c = threadIdx.x / CO_ROWS;
  if (c < nc && row < n) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < CO_TPB / 64; ++q) v += sh[(c * (CO_TPB / 64) + q) * CO_ROWS + r];
    xg[(size_t)(comp0 + c) * n + row] = (T)v;
  }
}

}  // namespace

template <typename T, int TI, int TJ>
void launch_block_tile(T* x, const T* b, const T* s1d, const T* bfac, int nx, int ny,
                       int nz, int ncomp, int colour, int kind, const T* zn, int nbx2,
                       int nby2, int nbzc, hipStream_t s) {
  const uint32_t N = (uint32_t)nx * ny * nz;
  const int ntx = (nbx2 + TI - 1) / TI, nty = (nby2 + TJ - 1) / TJ;
  dim3 grid(ntx * nty, nbzc, ncomp);
  by_kind<T>(kind, [&](auto k) {
    k_block_tile<T, decltype(k)::value, TI, TJ><<<grid, TI * TJ * 8, 0, s>>>(
        x, b, s1d, bfac, nx, ny, nz, N, colour, nbx2, nby2, ntx, zn);
  });
}

template <typename T>
hipError_t launch_block_pass(T* x, const T* b, const T* s1d, const T* bfac, int nx,
                             int ny, int nz, int ncomp, int colour, int kind, const T* zn,
                             int tile, hipStream_t s) {
  const int nbx2 = nx / 4, nby2 = ny / 4;
  const int nbz = nz / 2;
  const int nbzc = (nbz + 1 - (colour >> 2)) / 2;
  if (nbx2 * nby2 * nbzc == 0) return hipSuccess;
  if (tile == SMG_TILE_AUTO) {
    // the largest tile (least halo per block) that still gives every compute unit two
    // work-groups
    const int64_t layers = (int64_t)nbzc * ncomp;
    const int64_t wg84 = (int64_t)((nbx2 + 7) / 8) * ((nby2 + 3) / 4) * layers;
    const int64_t wg44 = (int64_t)((nbx2 + 3) / 4) * ((nby2 + 3) / 4) * layers;
    tile = wg84 >= 512 ? SMG_TILE_8X4 : (wg44 >= 512 ? SMG_TILE_4X4 : SMG_TILE_4X2);
  }
  if (tile == SMG_TILE_4X2)
    launch_block_tile<T, 4, 2>(x, b, s1d, bfac, nx, ny, nz, ncomp, colour, kind, zn, nbx2,
                                nby2, nbzc, s);
  else if (tile == SMG_TILE_8X4)
    launch_block_tile<T, 8, 4>(x, b, s1d, bfac, nx, ny, nz, ncomp, colour, kind, zn, nbx2,
                                nby2, nbzc, s);
  else
    launch_block_tile<T, 4, 4>(x, b, s1d, bfac, nx, ny, nz, ncomp, colour, kind, zn, nbx2,
                                nby2, nbzc, s);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_block_half(const HalfPassItem<T>* items, int n, int cz, bool post, int kind,
                             hipStream_t s) {
  for (int q = 0; q < n; ++q)
    if (!half_level(items[q].nx, items[q].ny)) return hipErrorNotSupported;
  HalfArgs<T> m{};
  m.cz = cz;
  m.post = post;
  uint32_t total = 0;
  int nthr = 0;
  size_t lds = 0;
  auto flush = [&]() -> hipError_t {
    if (m.nitems == 0) return hipSuccess;
    m.begin[m.nitems] = total;
    by_kind<T>(kind, [&](auto k) {
      k_block_half<T, decltype(k)::value><<<total, nthr, lds, s>>>(m);
    });
    m.nitems = 0;
    total = 0;
    nthr = 0;
    lds = 0;
    return hipGetLastError();
  };
  for (int q = 0; q < n; ++q) {
    const HalfPassItem<T>& p = items[q];
    const int nby2 = p.ny / 4, nbzc = (p.nz / 2 + 1 - cz) / 2;
    if (nby2 * nbzc == 0 || p.ncomp == 0) continue;
    if (m.nitems == kHalfItems) {
      hipError_t e = flush();
      if (e != hipSuccess) return e;
    }
    HalfItem<T>& it = m.it[m.nitems];
    it.xs = p.xs;
    it.xo = p.xo;
    it.xn = p.xn;
    it.b = p.b;
    it.s1d = p.s1d;
    it.bfac = p.bfac;
    it.zn = p.zn;
    it.nx = p.nx;
    it.ny = p.ny;
    it.nz = p.nz;
    it.N = (uint32_t)p.nx * p.ny * p.nz;
    it.P = 1;
    it.nbzc = nbzc;
    it.ngx = nby2;
    it.TP = block_plane_stride(HALF_ROWS * (p.nx + 2 * kBotHalo + 2), sizeof(T));
    m.begin[m.nitems] = total;
    total += (uint32_t)it.ngx * nbzc * p.ncomp;
    nthr = std::max(nthr, (4 * p.nx + 63) / 64 * 64);
    lds = std::max(lds, (size_t)TILE_D * it.TP * sizeof(T));
    ++m.nitems;
  }
  return flush();
}

// (Items of one launch run with the block size and LDS of the largest.  Launches of their own for
// items of one, two and four block rows a group were no faster: batches of 32 128^3 with 4 each of
// 64^3, 48^3, 32^3 6270 us, merged 6185; 40 96^3 with 2 each of 64^3, 48^3, 32^3 4064, merged 3941;
// FP32 6215, 6161 and 4049, 3882.)
//
// Block rows per work-group of a two-colour launch: the most (4, or 2 above 64 cells in x, for
// the least staging overlap) that still gives the launch about eight work-groups per compute
// unit, else one.
inline int pair_rows(int nx, int ny, int nz, int ncomp, int c_first) {
  const int nby2 = ny / 4, nbzc = (nz / 2 + 1 - (c_first >> 2)) / 2;
  int pj = nx <= 64 ? 4 : 2;
  while (pj > 1 && (int64_t)((nby2 + pj - 1) / pj) * nbzc * ncomp < 2048) pj /= 2;
  return pj;
}

template <typename T>
hipError_t launch_block_pair(const HalfPassItem<T>* items, int n, int c_first, int kind,
                             hipStream_t s) {
  for (int q = 0; q < n; ++q)
    if (!half_level(items[q].nx, items[q].ny)) return hipErrorNotSupported;
  HalfArgs<T> m{};
  m.cz = c_first;
  uint32_t total = 0;
  int nthr = 0;
  size_t lds = 0;
  auto flush = [&]() -> hipError_t {
    if (m.nitems == 0) return hipSuccess;
    m.begin[m.nitems] = total;
    by_kind<T>(kind, [&](auto k) {
      k_block_pair<T, decltype(k)::value><<<total, nthr, lds, s>>>(m);
    });
    m.nitems = 0;
    total = 0;
    nthr = 0;
    lds = 0;
    return hipGetLastError();
  };
  for (int q = 0; q < n; ++q) {
    const HalfPassItem<T>& p = items[q];
    const int nby2 = p.ny / 4, nbzc = (p.nz / 2 + 1 - (c_first >> 2)) / 2;
    if (nby2 * nbzc == 0 || p.ncomp == 0) continue;
    if (m.nitems == kHalfItems) {
      hipError_t e = flush();
      if (e != hipSuccess) return e;
    }
    HalfItem<T>& it = m.it[m.nitems];
    it.xn = p.xn;
    it.b = p.b;
    it.s1d = p.s1d;
    it.bfac = p.bfac;
    it.zn = p.zn;
    it.nx = p.nx;
    it.ny = p.ny;
    it.nz = p.nz;
    it.N = (uint32_t)p.nx * p.ny * p.nz;
    it.P = pair_rows(p.nx, p.ny, p.nz, p.ncomp, c_first);
    it.nbzc = nbzc;
    it.ngx = (nby2 + it.P - 1) / it.P;
    it.TP = block_plane_stride((4 * it.P + 2) * (p.nx + 2 * kBotHalo + 2), sizeof(T));
    m.begin[m.nitems] = total;
    total += (uint32_t)it.ngx * nbzc * p.ncomp;
    nthr = std::max(nthr, (2 * it.P * p.nx + 63) / 64 * 64);
    lds = std::max(lds, (size_t)TILE_D * it.TP * sizeof(T));
    ++m.nitems;
  }
  return flush();
}

template <typename T, int TI, int TJ>
hipError_t launch_block_multi_tiled(const BlockPassItem<T>* items, int n, int colour, int kind,
                                    hipStream_t s) {
  BlockMultiArgs<T> m{};
  m.colour = colour;
  uint32_t total = 0;
  auto flush = [&]() -> hipError_t {
    if (m.nitems == 0) return hipSuccess;
    m.begin[m.nitems] = total;
    by_kind<T>(kind, [&](auto k) {
      k_block_tile_multi<T, decltype(k)::value, TI, TJ><<<total, TI * TJ * 8, 0, s>>>(m);
    });
    m.nitems = 0;
    total = 0;
    return hipGetLastError();
  };
  for (int q = 0; q < n; ++q) {
    const BlockPassItem<T>& p = items[q];
    const int nbx2 = p.nx / 4, nby2 = p.ny / 4;
    const int nbzc = (p.nz / 2 + 1 - (colour >> 2)) / 2;
    if (nbx2 * nby2 * nbzc == 0 || p.ncomp == 0) continue;
    const int ntx = (nbx2 + TI - 1) / TI, nty = (nby2 + TJ - 1) / TJ;
    const uint32_t wgs = (uint32_t)ntx * nty * nbzc * p.ncomp;
    if (m.nitems == kBlockMultiItems) {
      hipError_t e = flush();
      if (e != hipSuccess) return e;
    }
    BlockMultiItem<T>& it = m.it[m.nitems];
    it.x = p.x;
    it.b = p.b;
    it.s1d = p.s1d;
    it.bfac = p.bfac;
    it.zn = p.zn;
    it.nx = p.nx;
    it.ny = p.ny;
    it.nz = p.nz;
    it.N = (uint32_t)p.nx * p.ny * p.nz;
    it.nbx2 = nbx2;
    it.nby2 = nby2;
    it.nbzc = nbzc;
    it.ntx = ntx;
    it.nty = nty;
    m.begin[m.nitems] = total;
    total += wgs;
    ++m.nitems;
  }
  return flush();
}

template <typename T>
hipError_t launch_block_pass_multi(const BlockPassItem<T>* items, int n, int colour, int kind,
                                   int tile, hipStream_t s) {
  if (tile == SMG_TILE_AUTO) {
    // the rule of launch_block_pass over the work-groups of all items together
    int64_t wg84 = 0, wg44 = 0;
    for (int q = 0; q < n; ++q) {
      const int nbx2 = items[q].nx / 4, nby2 = items[q].ny / 4;
      const int64_t layers = (int64_t)((items[q].nz / 2 + 1 - (colour >> 2)) / 2) * items[q].ncomp;
      wg84 += (int64_t)((nbx2 + 7) / 8) * ((nby2 + 3) / 4) * layers;
      wg44 += (int64_t)((nbx2 + 3) / 4) * ((nby2 + 3) / 4) * layers;
    }
    tile = wg84 >= 512 ? SMG_TILE_8X4 : (wg44 >= 512 ? SMG_TILE_4X4 : SMG_TILE_4X2);
  }
  if (tile == SMG_TILE_4X2) return launch_block_multi_tiled<T, 4, 2>(items, n, colour, kind, s);
  if (tile == SMG_TILE_8X4) return launch_block_multi_tiled<T, 8, 4>(items, n, colour, kind, s);
  return launch_block_multi_tiled<T, 4, 4>(items, n, colour, kind, s);
}

hipError_t launch_residual_gal(float* r, const float* x, const float* b, const float* s1d,
                               const float* zt, int nx, int ny, int nz, int ncomp, hipStream_t s) {
  const int ntx = (nx + GR_X - 1) / GR_X, nty = (ny + GR_Y - 1) / GR_Y;
  dim3 grid(ntx * nty, (nz + GR_Z - 1) / GR_Z, ncomp);
  k_residual_gal_tile<float><<<grid, TPB, 0, s>>>(r, x, b, s1d, zt, nx, ny, nz, ntx);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fold_residual(T* bc, T* xc, const T* x, const T* b, const T* zt,
                                const FoldTaps<T>& m, int nx, int ny, int nz, int ncomp,
                                hipStream_t s) {
  const int nxc = nx >> 1, nyc = ny >> 1, nzc = nz >> 1;
  if (nx % 4 || ny % 2 || nz % 2) return hipErrorInvalidValue;
  if (nxc * nyc * nzc == 0) return hipSuccess;
  auto go = [&](auto rx) {
    constexpr int RX = decltype(rx)::value, RY = TPB / RX;
    const int ntx = (nxc + RX - 1) / RX, nty = (nyc + RY - 1) / RY;
    int zper = FOLD_Z;  // see launch_fold_residual0; six planes are a run's halo
    auto groups = [&]() { return (int64_t)ntx * nty * ((nzc + zper - 1) / zper) * ncomp; };
    while (zper > 2 && groups() < 512) zper /= 2;
    // the time is that of a run's planes one after the other: a single layer where few groups
    // share the chip (32^3 x 3: 9.0 against 10.4 us, but 64^3 x 3 14.0 against 13.3)
    if (groups() < 128) zper = 1;
    dim3 grid(ntx * nty, (nzc + zper - 1) / zper, ncomp);
    // 512 lanes (one item of a plane each) where the work-groups are few, else two items a lane
    // (64^3 x 3 11.1 / 13.3 us, 64^3 x 24 38.9 / 33.0)
    if ((int64_t)grid.x * grid.y * grid.z < 640)
      k_fold_residual<T, RX, 2 * TPB><<<grid, 2 * TPB, 0, s>>>(bc, xc, x, b, zt, nx, ny, nz, ntx,
                                                               zper, m);
    else
      k_fold_residual<T, RX, TPB><<<grid, TPB, 0, s>>>(bc, xc, x, b, zt, nx, ny, nz, ntx, zper, m);
  };
  auto cover = [&](int rx, int ry) { return (int64_t)((nxc + rx - 1) / rx) * ((nyc + ry - 1) / ry); };
  if (cover(32, 8) <= cover(16, 16)) go(std::integral_constant<int, 32>());
  else go(std::integral_constant<int, 16>());
  return hipGetLastError();
}

template <typename T>
hipError_t launch_restrict(T* bc, T* xc, const T* r, int nxf, int nyf, int nzf, int ncomp,
                           hipStream_t s) {
  const uint32_t Nf = (uint32_t)nxf * nyf * nzf;
  const uint32_t Nc = Nf / 8;
  dim3 grid(blocks_for(Nc), ncomp);
  k_restrict<T><<<grid, TPB, 0, s>>>(bc, xc, r, nxf, nyf, nzf, Nf, Nc);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_prolong(T* x, const T* e, int nxf, int nyf, int nzf, int ncomp, hipStream_t s) {
  const uint32_t Nf = (uint32_t)nxf * nyf * nzf;
  dim3 grid(blocks_for(Nf), ncomp);
  k_prolong<T><<<grid, TPB, 0, s>>>(x, e, nxf, nyf, nzf, Nf, Nf / 8);
  return hipGetLastError();
}

template <typename T, int C>
hipError_t launch_coarsest_c(T* x, const T* b, const double* ainv, const double* w, int n,
                             int ncomp, bool noise, bool round, const NoiseArgs& na,
                             hipStream_t s) {
  dim3 grid((n + CO_ROWS - 1) / CO_ROWS, (ncomp + C - 1) / C);
  const size_t sums = (size_t)C * (CO_TPB / 64) * CO_ROWS;
  const size_t lds = std::max((size_t)2 * C * n, sums) * sizeof(double);
  if (noise) k_coarsest<T, true, C><<<grid, CO_TPB, lds, s>>>(x, b, ainv, w, n, ncomp, round, na);
  else k_coarsest<T, false, C><<<grid, CO_TPB, lds, s>>>(x, b, ainv, w, n, ncomp, round, na);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_coarsest(T* x, const T* b, const double* ainv, const double* w, int n,
                           int ncomp, bool noise, bool round, const NoiseArgs& na,
                           hipStream_t s) {
  if (n > 4096) return hipErrorInvalidValue;  // 64 KB of LDS for one component
  // four components per work-group once that still leaves work for the chip: a quarter of the
  // factor traffic, while four components' b and normals fit 64 KB
  if (ncomp >= 8 && n <= 1024) return launch_coarsest_c<T, 4>(x, b, ainv, w, n, ncomp, noise, round, na, s);
  return launch_coarsest_c<T, 1>(x, b, ainv, w, n, ncomp, noise, round, na, s);
}

template <typename T>
hipError_t launch_level_noise(const NoiseGenArgs& a, const NoiseArgs& na, hipStream_t s) {
  uint32_t maxblk = 0;
  int maxslot = 0;
  bool point = false;
  for (int e = 0; e < a.nlev; ++e) {
    point = point || !a.lv[e].bfac;
    const uint32_t nb = ((uint32_t)a.lv[e].nx * a.lv[e].ny * a.lv[e].nz + 7) / 8;
    maxblk = nb > maxblk ? nb : maxblk;
    maxslot = a.lv[e].nslot > maxslot ? a.lv[e].nslot : maxslot;
  }
  if (maxblk == 0 || maxslot * a.nact == 0) return hipSuccess;
  dim3 grid(blocks_for(maxblk), a.nlev, maxslot * a.nact);
  if (point) k_level_noise<T, true><<<grid, TPB, 0, s>>>(a, na);
  else k_level_noise<T, false><<<grid, TPB, 0, s>>>(a, na);
  return hipGetLastError();
}

#define SMG_INST(T)                                                                            \
  template hipError_t launch_block_pass<T>(T*, const T*, const T*, const T*, int, int,           \
                                           int, int, int, int, const T*, int, hipStream_t);     \
  template hipError_t launch_block_half<T>(const HalfPassItem<T>*, int, int, bool, int,          \
                                           hipStream_t);                                         \
  template hipError_t launch_block_pair<T>(const HalfPassItem<T>*, int, int, int, hipStream_t);   \
  template hipError_t launch_block_pass_multi<T>(const BlockPassItem<T>*, int, int, int, int,     \
                                                 hipStream_t);                                   \
  template hipError_t launch_fold_residual<T>(T*, T*, const T*, const T*, const T*,             \
                                              const FoldTaps<T>&, int, int, int, int,          \
                                              hipStream_t);                                     \
  template hipError_t launch_restrict<T>(T*, T*, const T*, int, int, int, int, hipStream_t);    \
  template hipError_t launch_prolong<T>(T*, const T*, int, int, int, int, hipStream_t);         \
  template hipError_t launch_coarsest<T>(T*, const T*, const double*, const double*, int, int,  \
                                         bool, bool, const NoiseArgs&, hipStream_t);            \
  template hipError_t launch_level_noise<T>(const NoiseGenArgs&, const NoiseArgs&, hipStream_t);
SMG_INST(double)
SMG_INST(float)
#undef SMG_INST

}  // namespace smg
