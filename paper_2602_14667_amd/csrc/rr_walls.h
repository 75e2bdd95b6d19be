// rr_walls.h -- the pull of one node on any 2D grid, periodic or walled, and
// the workgroup orders of the step kernels.
#pragma once
#include "rr_kernels.h"
#include "rr_node.h"

namespace rr {

// ---------------------------------------------------------------------------
// Pull addressing (task 6).  For a node (x, y) the population i comes from
// (x - c_ix, y - c_iy), periodic in x, periodic or walled in y.  With walls,
// a population whose source lies beyond a wall is the node's own
// post-collision population in the opposite direction (half-way
// bounce-back); for the magnetic populations the anti-bounce-back adds the
// wall term: g_j = -g*_opp(j) + 2 psi_j b_wall.
// ---------------------------------------------------------------------------
struct Rows {
  int xm, xp;                // x - 1, x + 1 (periodic)
  int64_t rm, r0, rp;        // element offsets of the rows y - 1, y, y + 1
  bool lo, hi;       // wall below (y == 0) / above (y == ny - 1)
};

template <bool WALLS>
__device__ __forceinline__ Rows rows_of(const Domain &D, int x, int y) {
  Rows R;
  R.xm = x == 0 ? D.nx - 1 : x - 1;
  R.xp = x == D.nx - 1 ? 0 : x + 1;
  const int ym = y == 0 ? D.ny - 1 : y - 1;
  const int yp = y == D.ny - 1 ? 0 : y + 1;
  R.rm = (int64_t)ym * D.row;
  R.r0 = (int64_t)y * D.row;
  R.rp = (int64_t)yp * D.row;
  R.lo = WALLS && y == 0;
  R.hi = WALLS && y == D.ny - 1;
  return R;
}

// Load population i (decoded, f - w) of node x through the pull.
template <class C, bool WALLS, int I>
__device__ __forceinline__ float pull_f(const Domain &D,
                                        const typename C::T *__restrict__ s,
                                        const Rows &R, int x) {
  constexpr int CX = cx(I), CY = cy(I);
  const int sx = CX == 0 ? x : (CX > 0 ? R.xm : R.xp);
  int64_t off = (CY == 0 ? R.r0 : (CY > 0 ? R.rm : R.rp)) + sx;
  int plane = I;
  if constexpr (WALLS && CY != 0) {
    const bool wall = CY > 0 ? R.lo : R.hi;
    if (wall) {
      plane = opp_f(I);
      off = R.r0 + x;
    }
  }
  return C::dec(s[(int64_t)plane * D.plane + off], D.inv_s);
}

template <class C, bool WALLS, int J>
__device__ __forceinline__ void pull_g(const Domain &D,
                                       const typename C::T *__restrict__ s,
                                       const Rows &R, int x, float &gx,
                                       float &gy) {
  constexpr int EX = ex(J), EY = ey(J);
  const int sx = EX == 0 ? x : (EX > 0 ? R.xm : R.xp);
  int64_t off = (EY == 0 ? R.r0 : (EY > 0 ? R.rm : R.rp)) + sx;
  int j = J;
  bool wall = false;
  if constexpr (WALLS && EY != 0) {
    wall = EY > 0 ? R.lo : R.hi;
    if (wall) {
      j = opp_g(J);
      off = R.r0 + x;
    }
  }
  gx = C::dec(s[(int64_t)gplane(j, 0) * D.plane + off], D.inv_s);
  gy = C::dec(s[(int64_t)gplane(j, 1) * D.plane + off], D.inv_s);
  if constexpr (WALLS && EY != 0) {
    if (wall) {
      gx = D.bw2x - gx;
      gy = D.bw2y - gy;
    }
  }
}

template <class C, bool WALLS>
__device__ __forceinline__ void pull_node(const Domain &D,
                                          const typename C::T *__restrict__ s,
                                          int x, int y, float (&d)[kQ],
                                          float (&g)[2 * kQm]) {
  const Rows R = rows_of<WALLS>(D, x, y);
  d[0] = pull_f<C, WALLS, 0>(D, s, R, x);
  d[1] = pull_f<C, WALLS, 1>(D, s, R, x);
  d[2] = pull_f<C, WALLS, 2>(D, s, R, x);
  d[3] = pull_f<C, WALLS, 3>(D, s, R, x);
  d[4] = pull_f<C, WALLS, 4>(D, s, R, x);
  d[5] = pull_f<C, WALLS, 5>(D, s, R, x);
  d[6] = pull_f<C, WALLS, 6>(D, s, R, x);
  d[7] = pull_f<C, WALLS, 7>(D, s, R, x);
  d[8] = pull_f<C, WALLS, 8>(D, s, R, x);
  pull_g<C, WALLS, 0>(D, s, R, x, g[0], g[1]);
  pull_g<C, WALLS, 1>(D, s, R, x, g[2], g[3]);
  pull_g<C, WALLS, 2>(D, s, R, x, g[4], g[5]);
  pull_g<C, WALLS, 3>(D, s, R, x, g[6], g[7]);
  pull_g<C, WALLS, 4>(D, s, R, x, g[8], g[9]);
}

// Block order: hardware hands consecutive workgroups to the eight XCDs in
// turn.  Renumbering so that each XCD receives a contiguous run of tiles
// keeps the cache lines shared by neighbouring tiles (the +-1 pull offsets)
// inside one L2.
__device__ __forceinline__ int xcd_remap(int L, int n) {
  const int q = n >> 3, r = n & 7, k = L & 7, m = L >> 3;
  return k < r ? k * (q + 1) + m : r * (q + 1) + (k - r) * q + m;
}

// Local variant: within each run of 64 consecutive workgroups, XCD k
// (workgroups L with L % 8 == k) takes 8 neighbouring tiles, so 7 of every 8
// tile boundaries stay inside one L2 while all XCDs still sweep the same
// region of memory together.
__device__ __forceinline__ int xcd_local(int L, int n) {
  const int g = L >> 6, j = L & 63;
  if ((g + 1) * 64 > n) return L;
  return (g << 6) + ((j & 7) << 3) + (j >> 3);
}

}  // namespace rr
