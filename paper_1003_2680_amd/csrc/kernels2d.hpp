// Launchers of the two-dimensional sampler's kernels (kernels_2d.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "kernels.hpp"
#include "philox.hpp"

namespace smg {

// One level of the 2D hierarchy on the device: x stencils s1d = (m_x, a_x) (10 values, offsets
// -2..2), per-row z bands zt[nz][10] = (a_z[z][z-2..z+2], m_z[z][z-2..z+2]) (zero beyond the
// walls), block factors bfac[nz/2][32] = (A_BB^-1, L_BB^-T) row-major 4 x 4 (Galerkin levels).
struct Lev2 {
  int nx, nz;
  const double* s1d;
  const double* zt;
  const double* bfac;
};

// level-0 red-black point heat bath of one colour (b null = 0); noise site = lex >> 1
hipError_t launch2_point_pass(double* x, const double* b, const Lev2& L, int ncomp, int colour,
                              double kT, bool noise, const NoiseArgs& na, hipStream_t s);
// Galerkin-level 2 x 2 block heat bath of one colour (colour = bx%2 + 2 (bz%2)); noise site =
// 4 block + in-block index
hipError_t launch2_block_pass(double* x, const double* b, const Lev2& L, int ncomp, int colour,
                              double kT, bool noise, const NoiseArgs& na, hipStream_t s);
// r = b - A x (b null = 0)
hipError_t launch2_residual(double* r, const double* x, const double* b, const Lev2& L,
                            int ncomp, hipStream_t s);
// b_c = P^T r; x_c = 0 when xc is not null
hipError_t launch2_restrict(double* bc, double* xc, const double* r, int nxf, int nzf, int ncomp,
                            hipStream_t s);
// x += P e
hipError_t launch2_prolong(double* x, const double* e, int nxf, int nzf, int ncomp,
                           hipStream_t s);

// ---- several level-0 passes per launch (kernels_2d_lds.hip)
constexpr int kMaxPoint2 = 4;  // point passes per launch
struct Point2Args {
  int nx, nz, rows;      // rows: per work-group (set by the launcher)
  int npass, slot0;      // passes: two per sweep, sweep slots slot0, slot0 + 1, ...
  int post;              // colour 1 first
  double ih2;            // 1 / h^2
  double inv_d[3], sig[3];  // set by the launcher: 1 / diagonal, sqrt(kT / diagonal) by walls
  const double* src;     // [ncomp][N]
  double* dst;           // another field
  const double* b;       // right-hand side or null
  const double* e;       // coarse correction added (as P e) before the passes, or null
  double* bc;            // P^T (b - A x) after the passes, or null; xc: cleared with it, or null
  double* xc;
  double* out;           // x written there too, or null
};
// Rows a work-group owns (even; 0: the window of a row strip does not fit): as many as leave the
// launch two work-groups per compute unit, at least eight (fewer draw more rows again than they
// own) unless only four fit.  Wherever a window fits, strips are the faster form, also on chips
// full of chains, whose launches are bound by the redrawn noise: four cycles, a launch a colour /
// strips, us: 512x512 1 chain 1309 / 1230, 8 2195 / 1668, 64 9796 / 7069; 416x512 (four rows) 16
// chains 2890 / 2168, 128 15 354 / 10 667; 256x256 255 chains 8976 / 5345; 64x64 255 792 / 443.
inline int level0_rows(int nx, int nz, int ncomp, int npass, bool restricts) {
  const int halo = npass + (restricts ? 2 : 0);
  int rows = 32;
  while (rows > 4 && ((size_t)(rows + 2 * halo) * nx * 8 > 64 * 1024 ||
                      (rows > 8 && (int64_t)((nz + rows - 1) / rows) * ncomp < 512)))
    rows /= 2;
  return (size_t)(rows + 2 * halo) * nx * 8 > 64 * 1024 ? 0 : rows;
}
hipError_t launch2_level0(const Point2Args& a, int ncomp, double kT, bool noise,
                          const NoiseArgs& na, hipStream_t s);

// ---- the LDS-resident bottom (kernels_2d_lds.hip)
constexpr int kMaxBot2Levels = 8;
constexpr size_t kBot2LdsMax = 160 * 1024;
struct Bot2Level {
  int nx, nz, kind;
  int rs;                   // LDS row stride of x: nx + 6 (two halo cells per side, 2 mod 4), nx coarsest
  int x_off, b_off, tab_off;  // LDS offsets (doubles)
  double s1d[10];           // (m_x, a_x)
  const double* tab;        // device: [zt nz*10][per block row A_BB^-1 in lane order, packed factors]
  const double* bfac;       // as Lev2
  double* noise;            // [nu1 + nu2][ncomp][nx nz], pregenerated each cycle
  double* xg;               // the level's x and b in memory
  double* bg;
};
struct Bot2Args {
  int nlev, level0, nu1, nu2, ncomp;
  int r_off;                // scratch rows
  size_t lds;               // bytes
  const double* ainv;
  const double* w;
  Bot2Level lv[kMaxBot2Levels];
};
// `dev` is the device copy of `host`; part: BotPart
hipError_t launch2_noise(const Bot2Args* dev, const Bot2Args& host, const NoiseArgs& na,
                         hipStream_t s);
hipError_t launch2_bottom(const Bot2Args* dev, const Bot2Args& host, int part, bool noise,
                          const NoiseArgs& na, hipStream_t s);

}  // namespace smg
