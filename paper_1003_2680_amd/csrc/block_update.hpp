// The 2x2x2 block heat bath of a Galerkin level on cells held in LDS, shared by every kernel that
// makes block passes, so that a cell's new value is the same bits in each of them.
//
// A = a_z (x) m_y (x) m_x + m_z (x) (a_y (x) m_x + m_y (x) a_x) with symmetric 5-point periodic 1D
// stencils s1d = (m_x, a_x, m_y, a_y) (offsets -2..2, uniform over the level) and the wall-axis
// rows zt[z] = (a_z[z][z + dz], m_z[z][z + dz]).  The eight lanes of a block are consecutive, lane
// bits kx, ky, kz from the lowest (neighbouring lanes touch neighbouring cells in memory; with kx
// as the highest bit the FP64 single-colour pass of 256x256x128 took 38 instead of 31 us): both
// exchanges of partial sums (y-partner lane ^ 2, z-partner lane ^ 4) and the eight-value sum of the
// block solve are DPP moves, never LDS permutes.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace smg {

// What a cycle belongs to: a solve, a chain without noise (kT = 0) or a chain with it.
enum CycleKind { CYCLE_SOLVE = 0, CYCLE_STILL = 1, CYCLE_NOISE = 2 };

// The passes of a chain in FP32 add up in index order (row, plane, lane), one term after the other:
// a refined chain carries its rounding from cycle to cycle into an FP64 state, which therefore
// keeps the bits that the plain order of the sums gives.  FP64 sums and the FP32 correction of a
// solve, whose rounding the next residual takes back, use the shorter symmetric forms.
template <typename T, int KIND>
constexpr bool index_order = KIND != CYCLE_SOLVE && sizeof(T) == 4;

// Runs go with the kind as a constant; an FP64 chain without noise makes a solve's passes.
template <typename T, typename F>
void by_kind(int kind, F go) {
  if (kind == CYCLE_NOISE) go(std::integral_constant<int, CYCLE_NOISE>());
  else if (sizeof(T) == 4 && kind == CYCLE_STILL)
    go(std::integral_constant<int, sizeof(T) == 4 ? CYCLE_STILL : CYCLE_SOLVE>());
  else go(std::integral_constant<int, CYCLE_SOLVE>());
}

// v of another lane of the same eight: quad_perm moves for lane ^ 1, ^ 2, ^ 3 and the mirror of
// the eight lanes for lane ^ 7 (lane ^ 4 is ^ 3 of it).
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_XOR3 = 0x1B, DPP_XOR7 = 0x141;
// the lane before and after within sixteen (nothing for the first, the last)
constexpr int DPP_BEFORE = 0x111, DPP_AFTER = 0x101;
template <int CTRL>
__device__ __forceinline__ double dpp_lane(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_lane(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the same bits in each of them).
__device__ __forceinline__ unsigned lane_pairs16(unsigned v, unsigned& other) {
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  other = r[1];
  return r[0];
}
__device__ __forceinline__ unsigned lane_pairs32(unsigned v, unsigned& other) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  other = r[1];
  return r[0];
}
__device__ __forceinline__ double sum_rows(double v) {
  auto join = [](unsigned lo, unsigned hi) {
    return __longlong_as_double(((long long)hi << 32) | lo);
  };
  long long u = __double_as_longlong(v);
  unsigned l1, h1;
  unsigned l0 = lane_pairs16((unsigned)u, l1), h0 = lane_pairs16((unsigned)(u >> 32), h1);
  v = join(l0, h0) + join(l1, h1);
  u = __double_as_longlong(v);
  l0 = lane_pairs32((unsigned)u, l1);
  h0 = lane_pairs32((unsigned)(u >> 32), h1);
  return join(l0, h0) + join(l1, h1);
}
__device__ __forceinline__ float sum_rows(float v) {
  unsigned a, b;
  a = lane_pairs16(__float_as_uint(v), b);
  v = __uint_as_float(a) + __uint_as_float(b);
  a = lane_pairs32(__float_as_uint(v), b);
  return __uint_as_float(a) + __uint_as_float(b);
}

// What a lane keeps over the passes of one block layer.  Of the layer's six planes 2 bz - 2 ..
// 2 bz + 3 the lanes of cell layer kz reduce planes 3 kz + m, m = 0 .. 2: all three (SPLIT 1) or,
// where a level leaves lanes idle, one each (SPLIT 4: m = s, the fourth lane with zero factors).
// po: element offset of each plane; the plane's z-factors for the lane's own cell and for its
// z-partner's; the lane's row of A_BB^-1 in the order of the lanes ^ m.
template <typename T, int SPLIT, bool INDEX = false>
struct BlockWeights {
  static constexpr int P = SPLIT == 4 ? 1 : 3;
  int po[P];
  T own0[P], own1[P], oth0[P], oth1[P], F[8];
};
// In index order: the cell's z-factors of its five planes and its row of A_BB^-1 by cell.
template <typename T, int SPLIT>
struct BlockWeights<T, SPLIT, true> {
  static constexpr int P = SPLIT == 4 ? 1 : 3;
  int po[P];
  T z0[5], z1[5], F[8];
};
// The device table of a block layer bz (kBlockRow<T> values): A_BB^-1 with entry m of row k that of
// cell k ^ m, cells k = kx + 2 ky + 4 kz; L_BB^-T; at kBlockZ the packed z-factors of the two
// cell layers kz, own0, own1, oth0, oth1 of planes m = 0 .. 2 and a zero each; and in FP32, for sums in
// index order, the layers' own z-rows, z0 and z1 eight apart (kBlockRows), and A_BB^-1 by cell (kBlockF).
template <typename T>
constexpr int kBlockRow = sizeof(T) == 4 ? 256 : 192;
constexpr int kBlockZ = 128, kBlockRows = 160, kBlockF = 192;
// Fp, Zp: a layer's A_BB^-1 part and its packed z-factors.
template <typename T, int SPLIT, typename PT>
__device__ __forceinline__ void block_weights(BlockWeights<T, SPLIT, true>& w, const PT Fp,
                                              const PT Zp, int kx, int ky, int kz, int) {
  // of the cell's five planes kz .. kz + 4 of the layer's six, the partner reduces 3, 4 (kz 0) or
  // 1, 2 (kz 1)
  const PT own = Zp + kz * 16, par = Zp + (kz ^ 1) * 16 + 8;
#pragma unroll
  for (int d = 0; d < 5; ++d) {
    const int at = kz ? (d < 2 ? 1 + d : d - 2) : (d < 3 ? d : d - 3);
    const PT q = (kz ? d < 2 : d >= 3) ? par : own;
    w.z0[d] = q[at];
    w.z1[d] = q[4 + at];
  }
  const int k = kx + 2 * ky + 4 * kz;
#pragma unroll
  for (int m = 0; m < 8; ++m) w.F[m] = Fp[k * 8 + (m ^ k)];
}
template <typename T, int SPLIT, typename PT>
__device__ __forceinline__ void block_weights(BlockWeights<T, SPLIT, false>& w, const PT Fp,
                                              const PT Zp, int kx, int ky, int kz, int s) {
  const PT z = Zp + kz * 16 + (SPLIT == 4 ? s : 0);
#pragma unroll
  for (int p = 0; p < BlockWeights<T, SPLIT>::P; ++p) {
    w.own0[p] = z[p];
    w.own1[p] = z[4 + p];
    w.oth0[p] = z[8 + p];
    w.oth1[p] = z[12 + p];
  }
  const PT F = Fp + (kx + 2 * ky + 4 * kz) * 8;
#pragma unroll
  for (int m = 0; m < 8; ++m) w.F[m] = F[m];
}

// The same from a layer's row of the device table in memory, where the entries in index order lie
// side by side: a lane's eight factors are two wide loads, where picking them out of the lane order
// (in LDS, above) is a load each (FP32 single-colour pass of 256x256x128: 15.9 us, with those 18.3).
template <typename T, bool INDEX>
__device__ __forceinline__ void block_row_weights(BlockWeights<T, 1, INDEX>& w, const T* row, int kx,
                                                  int ky, int kz) {
  if constexpr (INDEX) {
    const T *z = row + kBlockRows + kz * 16, *F = row + kBlockF + (kx + 2 * ky + 4 * kz) * 8;
#pragma unroll
    for (int d = 0; d < 5; ++d) {
      w.z0[d] = z[d];
      w.z1[d] = z[8 + d];
    }
#pragma unroll
    for (int m = 0; m < 8; ++m) w.F[m] = F[m];
  } else {
    block_weights<T, 1>(w, row, row + kBlockZ, kx, ky, kz, 0);
  }
}

// New value of the lane's cell: x_B + A_BB^-1 (b_B - (A x)_B) + noise, which equals A_BB^-1 (b_B -
// A_B,rest x_rest) + noise: the block's own coupling cancels.  `noise` already holds the lane's
// entry of sqrt(kT) L_BB^-T n.  Every lane of the wave calls it.
//
// ro[r]: element offset of the start of the five-cell x window of row r within a plane.  The two
// cells y, y + 1 of a block column together need the six rows y - 2 .. y + 3; each lane reduces
// three of them along x, rows y_lane + s (r - 2) with s = +1 for ky = 0 and -1 for ky = 1, i.e.
// the outer three of its own window from its far edge inwards.  m_y and a_y are symmetric, so in
// that order both lanes weight row r by factor r for their own cell, and rows 1, 2 by factors 0,
// 1 for the partner's, whose share arrives by a DPP move.  The z-partners trade their planes'
// weighted sums the same way.  45 reads a lane instead of 125.
//
// PRELOAD: every read is issued before the first sum, so that a pass waits for LDS once (for
// kernels with the registers to spare).
template <typename T, int SPLIT, bool PRELOAD>
__device__ __forceinline__ T block_update(const T* X, const int (&ro)[3], const T* s1d,
                                        const BlockWeights<T, SPLIT, false>& w, int own, T bk,
                                        T noise) {
  constexpr int P = BlockWeights<T, SPLIT>::P;
  T win[P][3][5];
#pragma unroll
  for (int m = 0; m < P; ++m)
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int d = 0; d < 5; ++d) win[m][r][d] = X[w.po[m] + ro[r] + d];
  const T xk = X[own];
  if (PRELOAD) __builtin_amdgcn_sched_barrier(0);
  T self = T(0), part = T(0);
#pragma unroll
  for (int m = 0; m < P; ++m) {
    T rm[3], ra[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const T(&v)[5] = win[m][r];
      const T e = v[0] + v[4], d = v[1] + v[3], c = v[2];  // the x factors are symmetric
      rm[r] = fma(s1d[0], e, fma(s1d[1], d, s1d[2] * c));
      ra[r] = fma(s1d[5], e, fma(s1d[6], d, s1d[7] * c));
    }
    const T* my = s1d + 10;
    const T* ay = s1d + 15;
    T p0 = my[0] * rm[1], p1 = ay[0] * rm[1];
    p0 = fma(my[1], rm[2], p0);
    p1 = fma(ay[1], rm[2], fma(my[0], ra[1], p1));
    p1 = fma(my[1], ra[2], p1);
    T q0 = my[0] * rm[0], q1 = ay[0] * rm[0];
    q0 = fma(my[1], rm[1], fma(my[2], rm[2], q0));
    q1 = fma(ay[1], rm[1], fma(ay[2], rm[2], q1));
    T qa = my[0] * ra[0];
    qa = fma(my[1], ra[1], fma(my[2], ra[2], qa));
    q0 += dpp_lane<DPP_XOR2>(p0);
    q1 = (q1 + qa) + dpp_lane<DPP_XOR2>(p1);
    self = fma(w.own0[m], q0, fma(w.own1[m], q1, self));
    part = fma(w.oth0[m], q0, fma(w.oth1[m], q1, part));
  }
  T ax = self + dpp_lane<DPP_XOR3>(dpp_lane<DPP_XOR7>(part));
  if (SPLIT == 4) ax = sum_rows(ax);
  const T res = bk - ax;
  const T mir = dpp_lane<DPP_XOR7>(res);  // lane ^ 7
  T v0 = xk, v1 = noise;
  v0 = fma(w.F[0], res, v0);
  v1 = fma(w.F[7], mir, v1);
  v0 = fma(w.F[1], dpp_lane<DPP_XOR1>(res), v0);
  v1 = fma(w.F[6], dpp_lane<DPP_XOR1>(mir), v1);
  v0 = fma(w.F[2], dpp_lane<DPP_XOR2>(res), v0);
  v1 = fma(w.F[5], dpp_lane<DPP_XOR2>(mir), v1);
  v0 = fma(w.F[3], dpp_lane<DPP_XOR3>(res), v0);
  v1 = fma(w.F[4], dpp_lane<DPP_XOR3>(mir), v1);
  return v0 + v1;
}

// The same in index order (FP32).  Here each lane needs its cell's five plane sums themselves, and
// the block's eight residuals by cell: more moves and selects than above.
template <typename T>
__device__ __forceinline__ T lane_z_partner(T v) {  // lane ^ 4
  return dpp_lane<DPP_XOR3>(dpp_lane<DPP_XOR7>(v));
}
template <int CTRL>
__device__ __forceinline__ float quad_value(float v) {
  return dpp_lane<CTRL>(v);
}
template <typename T, int SPLIT, bool PRELOAD>
__device__ __forceinline__ T block_update(const T* X, const int (&ro)[3], const T* s1d,
                                        const BlockWeights<T, SPLIT, true>& w, int own, T bk,
                                        T noise) {
  constexpr int P = BlockWeights<T, SPLIT, true>::P;
  const bool kz = threadIdx.x & 4;
  T win[P][3][5];
#pragma unroll
  for (int m = 0; m < P; ++m)
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int d = 0; d < 5; ++d) win[m][r][d] = X[w.po[m] + ro[r] + d];
  const T xk = X[own];
  if (PRELOAD) __builtin_amdgcn_sched_barrier(0);
  T q0[3], q1[3];
#pragma unroll
  for (int m = 0; m < P; ++m) {
    T rm[3], ra[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      T sm = T(0), sa = T(0);
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        sm = fma(s1d[d], win[m][r][d], sm);
        sa = fma(s1d[5 + d], win[m][r][d], sa);
      }
      rm[r] = sm;
      ra[r] = sa;
    }
    const T* my = s1d + 10;
    const T* ay = s1d + 15;
    T o0 = T(0), o1 = T(0);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      o0 = fma(my[r], rm[r], o0);
      o1 = fma(ay[r], rm[r], o1);
      o1 = fma(my[r], ra[r], o1);
    }
    T p0 = my[0] * rm[1];
    p0 = fma(my[1], rm[2], p0);
    T p1 = ay[0] * rm[1];
    p1 = fma(ay[1], rm[2], p1);
    p1 = fma(my[0], ra[1], p1);
    p1 = fma(my[1], ra[2], p1);
    q0[m] = o0 + dpp_lane<DPP_XOR2>(p0);
    q1[m] = o1 + dpp_lane<DPP_XOR2>(p1);
  }
  if constexpr (SPLIT == 4) {
    // planes m = 0, 1, 2 from the lanes of the four rows of sixteen
    auto gather = [](T (&q)[3]) {
      unsigned a, b, c, d;
      a = lane_pairs16(__float_as_uint(q[0]), b);
      a = lane_pairs32(a, c);
      b = lane_pairs32(b, d);
      q[0] = __uint_as_float(a);
      q[1] = __uint_as_float(b);
      q[2] = __uint_as_float(c);
    };
    gather(q0);
    gather(q1);
  }
  // planes kz .. kz + 4: the partner's two nearest come from it
  auto planes = [&](const T (&q)[3], const T (&z)[5]) {
    const T oa = lane_z_partner(kz ? q[0] : q[1]), ob = lane_z_partner(kz ? q[1] : q[2]);
    T acc = T(0);
    acc = fma(z[0], kz ? oa : q[0], acc);
    acc = fma(z[1], kz ? ob : q[1], acc);
    acc = fma(z[2], kz ? q[0] : q[2], acc);
    acc = fma(z[3], kz ? q[1] : oa, acc);
    return fma(z[4], kz ? q[2] : ob, acc);
  };
  const T ax = planes(q0, w.z0) + planes(q1, w.z1);
  const T res = bk - ax;
  const T mir = dpp_lane<DPP_XOR7>(res);  // lane ^ 7
  // residuals by cell: the own quad's in order, the other's reversed
  const T b0 = quad_value<0x00>(res), b1 = quad_value<0x55>(res), b2 = quad_value<0xAA>(res),
          b3 = quad_value<0xFF>(res);
  const T c0 = quad_value<0xFF>(mir), c1 = quad_value<0xAA>(mir), c2 = quad_value<0x55>(mir),
          c3 = quad_value<0x00>(mir);
  T v0 = xk, v1 = noise;
  v0 = fma(w.F[0], kz ? c0 : b0, v0);
  v1 = fma(w.F[1], kz ? c1 : b1, v1);
  v0 = fma(w.F[2], kz ? c2 : b2, v0);
  v1 = fma(w.F[3], kz ? c3 : b3, v1);
  v0 = fma(w.F[4], kz ? b0 : c0, v0);
  v1 = fma(w.F[5], kz ? b1 : c1, v1);
  v0 = fma(w.F[6], kz ? b2 : c2, v0);
  v1 = fma(w.F[7], kz ? b3 : c3, v1);
  return v0 + v1;
}

// The level's 1D stencils in scalar registers: the table is read-only while kernels run, and only
// loads from the constant space are taken as such past a kernel's stores.
template <typename T>
struct Stencils {
  T v[20];
};
template <typename T>
__device__ __forceinline__ Stencils<T> load_stencils(const T* s1d) {
  typedef const __attribute__((address_space(4))) T* cptr;
  Stencils<T> r;
#pragma unroll
  for (int q = 0; q < 20; ++q) r.v[q] = ((cptr)s1d)[q];
  return r;
}

// Plane stride of an LDS tile of rows of 2 mod 4 elements: padded so that the lanes served together
// fall on different banks (32 of four bytes).  FP64 reads are served sixteen lanes at a time (two
// neighbouring blocks: x steps 0, 1, 4, 5; the y-partners an odd number of rows apart, the
// z-partners three planes), which need distinct elements mod 16: planes of 8 mod 16.  FP32 reads
// are served 32 lanes at a time: planes of 16 mod 32.  (Bottom launches of a 16^3 level, half a
// cycle: FP64 34.9 us, with 16 mod 32, where its z-partners share a bank, 40.9; FP32 32.1, with 8
// mod 16 34.8.)
__host__ __device__ constexpr int block_plane_stride(int plane, size_t elem) {
  return elem == 8 ? plane + (24 - plane % 16) % 16 : plane + (48 - plane % 32) % 32;
}

}  // namespace smg
