// rr_multi.h -- several time steps per pass over memory (unforced, periodic
// grids; the tile form also walls and a body force).
//
// One step per launch streams all 19 planes through HBM (or, on small grids,
// waits for a launch) every step.  Both forms here take T steps from one read
// and one write of the state and repeat the one-step kernel's per-node
// arithmetic exactly (the storage rounding between steps included), so the
// state after T steps is bit for bit that of T single steps.
//
//  * march_strip: a wavefront owns a window of 64 neighbouring nodes and
//    marches down a strip of rows.  Stage s of the march holds step s of one
//    row; stage s + 1 works one row behind it.  Streaming in x is a one-lane
//    DPP shift, streaming in y a register delay: the planes with c_y = 0 wait
//    one row, those with c_y = +1 two, those with c_y = -1 none (19 registers
//    per stage boundary).  No LDS; each step loses one node per side of the
//    window (T = 4: 56 of 64 lanes store) and two rows per strip end.
//  * tile_steps: a workgroup owns a BX x BY tile held one node per thread;
//    between steps the populations that move are exchanged through LDS.  Each
//    step after the first loses a one-node ring.  For grids too small to fill
//    the chip with marching strips.
#pragma once
#include <utility>

#include "rr_node.h"
#include "rr_pull.h"
#include "rr_walls.h"

namespace rr {

__host__ __device__ constexpr int plane_cx(int p) { return p < kQ ? cx(p) : ex((p - kQ) / 2); }
__host__ __device__ constexpr int plane_cy(int p) { return p < kQ ? cy(p) : ey((p - kQ) / 2); }
__host__ __device__ constexpr int plane_opp(int p) {
  return p < kQ ? opp_f(p) : gplane(opp_g((p - kQ) / 2), (p - kQ) & 1);
}
// Number of planes q < p with c_y = cyv: the plane's place in a delay line.
__host__ __device__ constexpr int delay_slot(int p, int cyv) {
  int n = 0;
  for (int q = 0; q < p; ++q) n += plane_cy(q) == cyv;
  return n;
}
constexpr int kDelayZero = delay_slot(kPlanes, 0), kDelayPlus = delay_slot(kPlanes, 1);

// The value a step stores and the next one reads back (seed, plane: the random
// bits of the stochastic-rounding codec).
template <class C>
__device__ __forceinline__ float through_storage(float v, float s, float inv_s, uint32_t seed = 0,
                                                 int plane = 0) {
  if constexpr (std::is_same_v<C, CodecF32>)
    return v;
  else if constexpr (codec_sr<C>::value)
    return C::dec(C::enc_sr(v, s, sr_plane(seed, plane)), inv_s);
  else
    return C::dec(C::enc(v, s), inv_s);
}

// ---- marching strips -----------------------------------------------------------
// Nodes of a window lost to the halo on each side (one per step, four at most),
// and those stored.
constexpr int kMarchHalo = 4, kMarchOut = 64 - 2 * kMarchHalo;

// Lane i takes the value of lane i - 1 (c_x = +1) or i + 1 (c_x = -1).  The
// window's end lanes get zero (written by the shift itself, so no register is
// cleared for it): their values are lost to the halo anyway.
template <int CX>
__device__ __forceinline__ float lane_shift(float v) {
  if constexpr (CX == 0) return v;
  constexpr int ctrl = CX > 0 ? 0x138 : 0x130;  // wave_shr:1 / wave_shl:1
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xf, 0xf, true));
}

// Collide one row of the window: v holds the 19 post-collision planes of the
// previous step at the rows they are pulled from, unshifted in x.
template <class C, int... P>
__device__ __forceinline__ void march_shift(float (&v)[kPlanes], std::integer_sequence<int, P...>) {
  ((v[P] = lane_shift<plane_cx(P)>(v[P])), ...);
}
template <class C>
__device__ __forceinline__ void march_stage(float (&v)[kPlanes], const CollideParams &P) {
  march_shift<C>(v, std::make_integer_sequence<int, kPlanes>{});
  float(&d)[kQ] = *reinterpret_cast<float(*)[kQ]>(v);
  float(&g)[2 * kQm] = *reinterpret_cast<float(*)[2 * kQm]>(v + kQ);
  collide<false>(d, g, P);
}

template <class C, int... P>
__device__ __forceinline__ void march_load(const PlaneGeom &G, const typename C::T *rm,
                                           const typename C::T *rz, const typename C::T *rp,
                                           uint32_t xo, float (&v)[kPlanes],
                                           std::integer_sequence<int, P...>) {
  using T = typename C::T;
  ((v[P] = C::dec(
        ld_at<T, false>(
            plane_ptr(plane_cy(P) == 0 ? rz : (plane_cy(P) > 0 ? rm : rp), P, G.plane), xo),
        G.inv_s)),
   ...);
}
template <class C, int... P>
__device__ __forceinline__ void march_store(const PlaneGeom &G, typename C::T *row, uint32_t xo,
                                            const float (&v)[kPlanes],
                                            std::integer_sequence<int, P...>) {
  using T = typename C::T;
  ((st_at<T, false>(row + (int64_t)P * G.plane, xo, C::enc(v[P], G.s))), ...);
}

// T steps on the rows ys .. ys + rows - 1 of the calling wavefront's window:
// lane 0 stands at node x0 (any sign; positions wrap), and the lanes with
// `live` set store.  Every wavefront of a workgroup calls it with the same
// `rows` (it holds barriers); rows at or past ny are not stored.  The barrier
// per row keeps the workgroup's windows side by side, so the cache lines that
// neighbouring windows both write are complete in L2 before they are evicted
// (8192^2 FP32: 1.7 x slower without); the stores are plain for that reason.
template <class C, int T>
__device__ __forceinline__ void march_strip(const PlaneGeom &G, const CollideParams &P,
                                            const typename C::T *__restrict__ src,
                                            typename C::T *__restrict__ dst, int x0, bool live,
                                            int ys, int rows) {
  using TT = typename C::T;
  constexpr auto planes = std::make_integer_sequence<int, kPlanes>{};
  int x = x0 % G.nx;
  x += x < 0 ? G.nx : 0;
  uint32_t xo = (uint32_t)x * (uint32_t)sizeof(TT);
  float z[T - 1][kDelayZero], p1[T - 1][kDelayPlus], p2[T - 1][kDelayPlus];
#pragma unroll
  for (int s = 0; s < T - 1; ++s) {
#pragma unroll
    for (int i = 0; i < kDelayZero; ++i) z[s][i] = 0.0f;
#pragma unroll
    for (int i = 0; i < kDelayPlus; ++i) p1[s][i] = p2[s][i] = 0.0f;
  }
  // rows y - 1, y, y + 1 of the first stage, y from ys - (T - 1)
  auto wrap = [&](int v) {
    v %= G.ny;
    return v < 0 ? v + G.ny : v;
  };
  int ym = wrap(ys - T), yz = wrap(ys - T + 1), yp = wrap(ys - T + 2);
  const int last = rows + 2 * (T - 1);
  for (int i = 0; i < last; ++i) {
    asm("" : "+v"(xo));  // keeps the 32-bit offset beside its use (scalar-base addressing)
    float v[kPlanes];
    march_load<C>(G, src + (int64_t)ym * G.row, src + (int64_t)yz * G.row,
                  src + (int64_t)yp * G.row, xo, v, planes);
    ym = yz;
    yz = yp;
    yp = yp == G.ny - 1 ? 0 : yp + 1;
    // the later stages; false while the delay lines still fill.  A row that is
    // not stored leaves here, so that no value is copied to be kept for the
    // store (with the shifts above, pass of four steps: 4096^2 FP16 624 -> 591 us,
    // 2000^2 FP32 202 -> 191, 8192^2 FP32 2328 -> 2289).
    auto stages = [&]() {
      march_stage<C>(v, P);
#pragma unroll
      for (int s = 0; s < T - 1; ++s) {
        // keeps the collision whole above the branch (sunk into the branches
        // it held 143 registers)
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) asm volatile("" ::"v"(v[p]));
        if (i < 2 * s) return false;  // stage s has no valid row yet
        float c[kPlanes];
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) {
          const float w = through_storage<C>(v[p], G.s, G.inv_s);
          const int q = delay_slot(p, plane_cy(p));
          if (plane_cy(p) < 0) {
            c[p] = w;
          } else if (plane_cy(p) == 0) {
            c[p] = z[s][q];
            z[s][q] = w;
          } else {
            c[p] = p2[s][q];
            p2[s][q] = p1[s][q];
            p1[s][q] = w;
          }
        }
        if (i < 2 * (s + 1)) return false;
        march_stage<C>(c, P);
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) v[p] = c[p];
      }
      return true;
    };
    if (!stages()) {
      __builtin_amdgcn_s_barrier();
      continue;
    }
    __builtin_amdgcn_s_barrier();
    const int yo = ys + i - 2 * (T - 1);
    if (live && yo < G.ny) march_store<C>(G, dst + (int64_t)yo * G.row, xo, v, planes);
  }
}

// ---- tiles with LDS exchange -----------------------------------------------------
// Populations that move, i.e. all but f_0 and g_0: 16 planes.
__host__ __device__ constexpr bool plane_moves(int p) { return plane_cx(p) || plane_cy(p); }
__host__ __device__ constexpr int moving_slot(int p) {
  int n = 0;
  for (int q = 0; q < p; ++q) n += plane_moves(q);
  return n;
}
constexpr int kMoving = moving_slot(kPlanes);

// A B x B tile of the grid D, one node per thread, through T steps: the first
// pulls from memory, the later ones from the neighbours through LDS (two
// buffers, so one barrier per step).  After T steps the inner B - 2 (T - 1)
// square is valid and stored; tile (tx, ty) stores the square at (tx, ty) times
// that side.  With walls the tiles cover [0, ny) in y, threads beyond a wall
// idle, and bounce-back reads the node's own values as the one-step kernel does.
template <class C, int B, bool WALLS, bool FORCED>
__device__ __forceinline__ void tile_steps(const Domain &D, float (&ex)[2][kMoving][B * B], int tx,
                                           int ty, int T, const typename C::T *__restrict__ src,
                                           typename C::T *__restrict__ dst) {
  constexpr int N = B * B;
  const int halo = T - 1, out = B - 2 * halo;
  const int t = threadIdx.x, ly = t / B, lx = t - ly * B;
  const int xr = tx * out - halo + lx, yr = ty * out - halo + ly;
  int x = xr % D.nx;
  x += x < 0 ? D.nx : 0;
  int y = yr;
  bool inside = true;
  if constexpr (WALLS) {
    inside = yr >= 0 && yr < D.ny;
    y = inside ? yr : 0;
  } else {
    y %= D.ny;
    y += y < 0 ? D.ny : 0;
  }
  const bool lo = WALLS && y == 0, hi = WALLS && y == D.ny - 1;
  const CollideParams P{D.om_c, D.omm_c, D.Gx, D.Gy, D.src_c};
  PlaneGeom G{D.plane, D.nx, D.ny, D.s, D.inv_s, 0u, D.row};
  if constexpr (codec_sr<C>::value) G.sr_key = sr_step_key(D.sr_key);
  float v[kPlanes];
  float(&d)[kQ] = *reinterpret_cast<float(*)[kQ]>(v);
  float(&g)[2 * kQm] = *reinterpret_cast<float(*)[2 * kQm]>(v + kQ);
  if constexpr (WALLS)
    pull_node<C, true>(D, src, x, y, d, g);
  else
    pull_node_per<C, false>(G, row_addr<RM_LANE>(G, src, y), x, d, g);
#pragma unroll 1
  for (int s = 1;; ++s) {
    collide<FORCED>(d, g, P);
    if (s == T) break;
    float(&b)[kMoving][N] = ex[s & 1];
    const uint32_t seed = node_seed<C>(G, x, y);
    if constexpr (codec_sr<C>::value) G.sr_key = sr_step_key(D.sr_key + s);  // of the next step
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) {
      v[p] = through_storage<C>(v[p], D.s, D.inv_s, seed, p);
      if (plane_moves(p)) b[moving_slot(p)][t] = v[p];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) {
      if (!plane_moves(p)) continue;
      // the upstream neighbour; cells past the tile's edge (whose values the
      // halo discards) stay in bounds
      const int o = t - plane_cx(p) - plane_cy(p) * B;
      float w = b[moving_slot(p)][min(max(o, 0), N - 1)];
      if constexpr (WALLS) {
        if (plane_cy(p) != 0 && (plane_cy(p) > 0 ? lo : hi)) {
          w = b[moving_slot(plane_opp(p))][t];
          if (p >= kQ) w = ((p - kQ) & 1 ? D.bw2y : D.bw2x) - w;
        }
      }
      v[p] = w;
    }
  }
  if (inside && lx >= halo && lx < B - halo && ly >= halo && ly < B - halo && xr < D.nx &&
      yr < D.ny)
    store_node<C, false, RM_LANE>(G, dst, x, y, d, g);
}

// ---- what a pass costs (launch rules) -----------------------------------------------
constexpr int kCUs = 256;

// Estimated time (us) of one pass of four marching steps with w workgroups per
// CU and strips of `rows` rows: per row each wavefront on a SIMD issues four
// collisions (1.8 us), each strip adds its halo rows, plus the launch.  Fits
// the measured passes of 20 grids from 320^2 to 5000^2, 1 to 16 workgroups
// per CU, to 4 % on average.
inline double march_us(double w, int rows) {
  return 6.0 + (1.1 + 1.75 * (w > 1.0 ? w : 1.0)) * (rows + 2.5);
}
// The same for a pass of T steps in 32 x 32 tiles, one workgroup per CU at a
// time (131 KB of LDS), q tiles per CU.
inline double tile32_us(int T, double q) { return T == 5 ? 1.5 + 13.0 * q : 2.0 + 11.5 * q; }
// One step of the one-step kernels, `bytes` of state: a launch, and the state
// read and written at `rate` bytes per us (through HBM).
inline double single_us(double bytes, double rate = 5.4e6) { return 3.0 + 2.0 * bytes / rate; }

// Windows of equal width covering a row of nx nodes, in multiples of 8.
struct MarchWindows {
  int n, out;
};
inline MarchWindows march_windows(int nx) {
  const int w = (nx + kMarchOut - 1) / kMarchOut;
  int out = ((nx + w - 1) / w + 7) / 8 * 8;
  if (out > kMarchOut) out = kMarchOut;
  return MarchWindows{(nx + out - 1) / out, out};
}

}  // namespace rr
