// rr_multi.hip -- kernels and launch rules of the multi-step forms
// (rr_multi.h): T time steps from one read and one write of the state.
#include <hip/hip_runtime.h>

#include "rr_kernels.h"
#include "rr_multi.h"
#include "rr_node.h"
#include "rr_pull.h"
#include "rr_walls.h"

namespace rr {

// ---- marching strips -------------------------------------------------------------
// A workgroup is four wavefronts: wx neighbouring windows of `out` stored
// nodes each, times 4 / wx strips of `rows` rows (wx = 4 unless the grid is
// narrower than that).  Eight neighbouring workgroups of every 64 share an XCD.
//
// Bound by the vector ALU, and at sizes far past the caches by HBM as well:
// 8192^2 FP32, 4 steps per pass, 558 us per step over 10,000 steps (120 GLUPS;
// ~260 VALU instructions per node and step with 56 of 64 lanes storing take 510
// at 39.3 T lane instructions/s, and 11.5 GB per pass are 5.1 TB/s, what a copy
// reaches) against 1652 us one step at a time; 4096^2 FP16 (~290) 133 us against
// 222.  Counters at 8192^2: VALU busy 88 %, reads 1.25 x
// the state (a workgroup of four windows reads nine lines for the seven it stores).
// Four steps and not more: 2 / 3 / 4 / 6 steps measured, when four took 586, 1076 / 725 / 586 /
// 625 us per step (six lose 12 of 64 lanes to the halo); two nodes per lane
// need twice the delay registers and measured 694 us at three steps.  Four
// neighbouring windows of 56 nodes are 7 x 128 B lines in FP32.

template <class C, int T>
__global__ __launch_bounds__(256) void k_march(PlaneGeom G, CollideParams P, int groups_x, int wx,
                                               int out, int rows,
                                               const typename C::T *__restrict__ src,
                                               typename C::T *__restrict__ dst) {
  static_assert(T <= kMarchHalo, "each step loses one node per side");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int L = xcd_local(blockIdx.x, gridDim.x);
  const int gy = L / groups_x, gx = L - gy * groups_x;
  const int wy = wave / wx;
  const int x0 = (gx * wx + (wave - wy * wx)) * out - kMarchHalo + lane;
  const bool live = lane >= kMarchHalo && lane < kMarchHalo + out && x0 < G.nx;
  march_strip<C, T>(G, P, src, dst, x0, live, (gy * (4 / wx) + wy) * rows, rows);
}

// ---- tiles with LDS exchange ---------------------------------------------------
template <class C, int B, bool WALLS, bool FORCED>
__global__ __launch_bounds__(B *B) void k_tile_steps(Domain D, int tiles_x, int T,
                                                     const typename C::T *__restrict__ src,
                                                     typename C::T *__restrict__ dst) {
  __shared__ float ex[2][kMoving][B * B];
  const int ty = blockIdx.x / tiles_x, tx = blockIdx.x - ty * tiles_x;
  tile_steps<C, B, WALLS, FORCED>(D, ex, tx, ty, T, src, dst);
}

// ---- launch rules ------------------------------------------------------------------
template <class C>
static void march_t(const MultiPlan &M, const Domain &D, const void *src, void *dst,
                    hipStream_t st) {
  using T = typename C::T;
  const PlaneGeom G{D.plane, D.nx, D.ny, D.s, D.inv_s, 0u, D.row};
  const CollideParams P{D.om_c, D.omm_c, 0.0f, 0.0f, 0.0f};
  const int strips = 4 / M.wx;
  const int groups_y = (D.ny + M.rows * strips - 1) / (M.rows * strips);
  const dim3 grid(M.groups_x * groups_y), block(256);
  auto s = (const T *)src;
  auto d = (T *)dst;
  if (M.steps == 4)
    hipLaunchKernelGGL((k_march<C, 4>), grid, block, 0, st, G, P, M.groups_x, M.wx, M.out, M.rows, s, d);
  else if (M.steps == 3)
    hipLaunchKernelGGL((k_march<C, 3>), grid, block, 0, st, G, P, M.groups_x, M.wx, M.out, M.rows, s, d);
  else
    hipLaunchKernelGGL((k_march<C, 2>), grid, block, 0, st, G, P, M.groups_x, M.wx, M.out, M.rows, s, d);
}

template <class C, int B>
static void tile_b(const MultiPlan &M, const Domain &D, const void *src, void *dst,
                   hipStream_t st) {
  using T = typename C::T;
  const int out = B - 2 * (M.steps - 1);
  const int tiles_x = (D.nx + out - 1) / out, tiles_y = (D.ny + out - 1) / out;
  const dim3 grid(tiles_x * tiles_y), block(B * B);
  const bool forced = D.Gx != 0.0f || D.Gy != 0.0f;
  auto s = (const T *)src;
  auto d = (T *)dst;
  if (D.walls && forced)
    hipLaunchKernelGGL((k_tile_steps<C, B, true, true>), grid, block, 0, st, D, tiles_x, M.steps, s, d);
  else if (D.walls)
    hipLaunchKernelGGL((k_tile_steps<C, B, true, false>), grid, block, 0, st, D, tiles_x, M.steps, s, d);
  else if (forced)
    hipLaunchKernelGGL((k_tile_steps<C, B, false, true>), grid, block, 0, st, D, tiles_x, M.steps, s, d);
  else
    hipLaunchKernelGGL((k_tile_steps<C, B, false, false>), grid, block, 0, st, D, tiles_x, M.steps, s, d);
}

template <class C>
static void multi_t(const MultiPlan &M, const Domain &D, const void *src, void *dst,
                    hipStream_t st) {
  if (M.tile == 0)
    march_t<C>(M, D, src, dst, st);
  else if (M.tile == 16)
    tile_b<C, 16>(M, D, src, dst, st);
  else
    tile_b<C, 32>(M, D, src, dst, st);
}

// The estimate of single_us for this grid.  The rate (bytes per us) of a state
// that the caches hold is higher where a step is whole waves of one row, 64
// nodes (64 x 3000 and 64 x 5000: FP32 5.8 and 6.9 to 10.2 us per step, FP16 4.7
// and 6.2, walls as periodic), and in one buffer, half the footprint (512 x 500
// FP32 6.5 us against 9.8 in two, 64 x 5000 6.9 / 10.2, 127 x 4000 FP16 7.8 / 9.9).
// At the common rate passes were taken that lose to it: 64 x 5000 FP16 walls 7.0
// against 6.2, one buffer FP32 8.0 / 6.9, 127 x 4000 FP16 in one buffer 9.6 / 7.8.
static double single_us(const Domain &D, bool one_buffer) {
  const double bytes = (double)D.nx * D.ny * D.elem * kStatePlanes;
  const bool f32 = D.elem == 4;
  double rate = 5.4e6;
  if (one_buffer) rate = f32 ? 9.0e6 : 6.0e6;
  if (D.nx == 64 && bytes < 128e6) rate = one_buffer && f32 ? 12.0e6 : 8.0e6;
  return single_us(bytes, rate);
}

// Tiles per CU of a pass of T steps in B x B tiles.
static int64_t tiles_per_cu(const Domain &D, int B, int T) {
  const int64_t out = B - 2 * (T - 1);
  return ((D.nx + out - 1) / out * ((D.ny + out - 1) / out) + kCUs - 1) / kCUs;
}

// The form and the number of steps of the next pass with n steps to go.
//
// Where the workgroups are at most one per CU, a pass is one round of tiles,
// bound by latency: 16 x 16 tiles if they can take five steps or more (up to
// seven), else 32 x 32 (up to nine), with as many steps as still give one
// round (us per step, one at a time in brackets: 64^2 FP32 7 steps 1.17 (3.12),
// 5 steps 1.28; 96^2 6 steps 1.40 (3.20); 128^2 5 steps 1.64 (3.26); 192^2, 32 x
// 32, 9 steps 2.01 (3.50), 5 steps 2.41; 256^2 9 steps 2.26 (3.90), 5 steps 2.73;
// 320^2 7 steps 2.53 (4.35); FP16 within 15 % of these; tiles of 24 x 24 were
// between the two or level with them everywhere).  The steps to go are shared
// out evenly among the passes.  Above that the estimates decide between 32 x
// 32 tiles and marching strips (512^2 FP32 5.7 / 9.6 in tiles, 768^2 9.8 / 20.0,
// 1024^2 13.6 / 30.2, 2048^2 45 / 108, 8192^2 558 / 1652 marching; FP16 1024^2
// 14.4 / 19.3, 4096^2 133 / 222).  Short remainders stay one step at a time
// where the halo costs more than the launches saved, and grids so narrow or
// short that the estimate exceeds the one-step kernel's: two steps in tiles at
// 256^2 measured 5.0 us per step against 3.9, three 3.9.  Narrow FP16 grids: 33 x
// 6000 5.7 / 8.7 in tiles, 100 x 3000 6.9 / 8.4, one step at a time 64 x 3000
// 4.7 (level) and 127 x 8000 16.2 (tiles 18.3).
//
// Stochastic rounding draws its bits per step, node and plane, so a pass
// reproduces them, at about half the collision's instructions again: it takes
// the passes that are one round of tiles (64^2 1.51 us per step against 3.65,
// 256^2 3.22 against 4.05), where launches and not instructions are what costs.
//
// Walls and forces exist as tiles only.  FP32 takes them at any size (tiles /
// one step at a time, walls: 1000 x 600 13.2 / 17.6, 2048^2 73 / 124, 4001 x 2000
// 137 / 312; walls and force 14.9 / 17.3, 86 / 118, 165 / 305); with FP16, half
// the bytes, the one-step kernel is ahead beyond three tiles per CU (walls:
// 700 x 500 8.2 / 8.5, 1000 x 600 12.4 / 11.4, 2048^2 70 / 59), forced beyond two
// (700 x 500 9.8 / 9.9, 2048^2 86 / 76).  From nine tiles per CU on five steps
// beat four (1500 x 1000 28.0 / 29.0, 2048^2 73 / 82).
MultiPlan multi_plan(const Domain &D, int64_t n, bool one_buffer) {
  MultiPlan M{};
  if (n < 2 || D.feq || D.nx > (1 << 30) || D.ny > (1 << 30)) return M;
  const bool forced = D.Gx != 0.0f || D.Gy != 0.0f;
  auto tile = [&](int B, int T) {
    MultiPlan P{};
    P.tile = B;
    const int64_t passes = (n + T - 1) / T;
    P.steps = (int)((n + passes - 1) / passes);
    // an even share below what 32 x 32 tiles take would end in single steps:
    // full passes first then (512 x 500 FP32, run of six: 5 + 1 steps 5.6 us per
    // step, 3 + 1 + 1 + 1 8.5)
    if (B == 32 && n / passes < 4) P.steps = (int)(n < T ? n : T);
    return P;
  };
  for (int T = 7; T >= 5; --T)
    if (tiles_per_cu(D, 16, T) == 1) return tile(16, T);
  if (n >= 4)
    for (int T = 9; T >= 6; --T)
      if (tiles_per_cu(D, 32, T) == 1) return tile(32, T);
  if (D.sr) return M;
  int T = 5;
  int64_t q = tiles_per_cu(D, 32, 5);
  const int64_t q4 = tiles_per_cu(D, 32, 4);
  if (q <= 8 && tile32_us(4, q4) / 4 < tile32_us(5, q) / 5) {
    T = 4;
    q = q4;
  }
  const double single = single_us(D, one_buffer);
  const bool tiles = n >= 4 && (q == 1 || tile32_us(T, q) / T < 1.1 * single);
  if (D.walls || forced)
    return tiles && (D.elem == 4 || q <= (forced ? 2 : 3)) ? tile(32, T) : M;
  if (tiles && q == 1) return tile(32, T);
  if ((int64_t)D.nx * D.ny < (n >= 4 ? 200000 : 400000)) return tiles ? tile(32, T) : M;
  const MarchWindows mw = march_windows(D.nx);
  MultiPlan W{};
  W.out = mw.out;
  W.wx = mw.n >= 3 ? 4 : mw.n;
  W.groups_x = (mw.n + W.wx - 1) / W.wx;
  const int64_t strips = 4 / W.wx;  // strips per workgroup
  double best = 0.0;
  // five workgroups are resident per CU; up to about 12 M nodes one such round
  // with longer strips beats the estimate's choice (2500^2 FP32 62.6 against
  // 66.4 us per step, 3000^2 84.5 / 87.6, FP16 77.1 / 78.4), past that more and
  // shorter strips even out (8192^2 FP32 3 % faster than one round, FP16 7 %,
  // 4096^2 FP16 2 %)
  const int kmax = (int64_t)D.nx * D.ny < 12000000 ? 5 : 16;
  for (int k = 1; k <= kmax; ++k) {
    const int64_t groups_y = kCUs * k / W.groups_x > 0 ? kCUs * k / W.groups_x : 1;
    int rows = (int)((D.ny + groups_y * strips - 1) / (groups_y * strips));
    if (rows < 3) rows = 3;
    const int64_t wgs = W.groups_x * ((D.ny + rows * strips - 1) / (rows * strips));
    const double us = march_us((double)wgs / kCUs, rows);
    if (W.rows == 0 || us < best) {
      best = us;
      W.rows = rows;
    }
  }
  if (tiles && tile32_us(T, q) / T < best / 4) return tile(32, T);
  if (best / 4 > 1.1 * single) return M;
  W.steps = n < 4 ? (int)n : 4;
  return W;
}

hipError_t launch_multi(const MultiPlan &M, int storage, const Domain &D, const void *src,
                        void *dst, hipStream_t st) {
  if (storage == kF16 && D.sr && M.tile == 16)
    tile_b<CodecF16SR, 16>(M, D, src, dst, st);
  else if (storage == kF16 && D.sr)
    tile_b<CodecF16SR, 32>(M, D, src, dst, st);
  else if (storage != kF16)
    multi_t<CodecF32>(M, D, src, dst, st);
  else if (D.s == 1.0f)
    multi_t<CodecF16U>(M, D, src, dst, st);
  else
    multi_t<CodecF16>(M, D, src, dst, st);
  return hipGetLastError();
}

}  // namespace rr
