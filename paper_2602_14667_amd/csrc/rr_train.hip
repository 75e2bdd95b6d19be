// rr_train.hip -- training kernels of the closure network (FP32): data
// preparation from filtered fine-grid moments, forward and backward passes,
// deterministic gradient reduction, Adam.
//
// Training data (a-priori regression): the fine moments are box-filtered
// over factor x factor blocks; the coarse node's features are
// (rho_bar, u_bar, b_bar, a_CE) with u_bar = (rho u)_bar / rho_bar and the
// Chapman-Enskog estimate a_CE = -rho_bar c_s^2 tau_c (grad u_bar + grad
// u_bar^T) from the isotropic lattice gradient of the coarse grid; the target
// is tau_sgs / (tau_c - 1) with tau_sgs = (rho u u)_bar - rho_bar u_bar
// u_bar + M(b)_bar - M(b_bar), M = |b|^2 I / 2 - b b.  A constant correction
// D added to a_1^(2) every step settles at a = (tau - 1) D, so this target
// makes the added momentum flux equal the subgrid stress.
//
// One-step solver-in-the-loop objective: the coarse grid is restarted from
// the filtered fine fields at t (f = f_eq(rho_bar, u_bar, b_bar) +
// f_neq,reg(u_bar, a_CE), g = g_eq) and advanced one coarse step with the
// network's correction D(Y) added to a_1^(2) at every node Y; the loss is
// L = sum_X |j_c(X) - j_bar(X, t + fac)|^2 / sum_X |j_bar(t + fac) - j_bar(t)|^2.
// The post-collision populations of a node are affine in its own D:
// f*_i(Y) = f*_i(Y)|_{D=0} + (1 - 1/tau_c) w_i R_i(u(Y)) . D(Y), with
// R_i . D the regularised expansion (second order 9/2, recursive third order
// 27/2, fourth order 81/4) of the coefficient D, so after the pull
// j_c(X) = j_c(X)|_{D=0} + sum_i c_i (1 - 1/tau_c) w_i R_i(u(X - c_i)) . D(X - c_i),
// and dL/dD(Y) is the transpose stencil: (2/den) (1 - 1/tau_c) sum_i
// (c_i . r(Y + c_i)) w_i R_i(u(Y)).  The D = 0 part is prepared once per
// snapshot in FP64; the network-dependent part runs in FP32.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <new>

#include "../../include/rrmhd.h"
#include "rr_internal.h"
#include "rr_kernels.h"
#include "rr_mlp.h"
#include "rr_node.h"
#include "rr_pull.h"

namespace rr {

constexpr int kTB = 256;

// GELU in its tanh form and its derivative, as z s and s + 2 z s (1 - s) v'(z)
// with s = 1 / (1 + e), e = exp(-2 v), v = sqrt(2/pi) (z + 0.044715 z^3): the
// same functions as z/2 (1 + tanh v), without the cancellation of 1 + tanh v
// at negative z, at one v_exp_f32 and one v_rcp_f32.  The rounding of 1 + e is
// carried into the reciprocal's correction step; 1 - s is e s.  Largest and
// rms error over |z| <= 5 against FP64 (library tanhf form in brackets): 3.7e-7
// (4.3e-7) and 6.4e-8 (7.5e-8), derivative 1.4e-7 (5.6e-7) and 2.9e-8 (1.3e-7).
__device__ __forceinline__ void gelu_parts(float z, float &h, float &es, float &s) {
  constexpr double kL = 2.302208198144325;  // 2 sqrt(2 / pi) log2(e)
  constexpr float c1 = (float)kL, c1l = (float)(kL - (double)c1), c2 = (float)(kL * 0.044715);
  const float p = fmaf(z, c1, z * fmaf(c2, z * z, c1l));  // e = 2^-p
  const float e = __builtin_amdgcn_exp2f(fminf(-p, 126.0f));
  const float d = 1.0f + e, bb = d - 1.0f;
  const float err = (1.0f - (d - bb)) + (e - bb);  // 1 + e = d + err
  const float r0 = __builtin_amdgcn_rcpf(d);
  s = fmaf(fmaf(-err, r0, fmaf(-d, r0, 1.0f)), r0, r0);
  es = e * s;
  h = z * s;
}
__device__ __forceinline__ float gelu32(float z) {
  float h, es, s;
  gelu_parts(z, h, es, s);
  return h;
}
__device__ __forceinline__ void gelu_pair(float z, float &h, float &g) {
  float es, s;
  gelu_parts(z, h, es, s);
  // 2 v'(z): 6 sqrt(2/pi) 0.044715, 2 sqrt(2/pi).  It only counts while s (1 - s)
  // does; past |z| = 16, where that is below 2^-450, it stops growing, or z^3
  // would outrun the smallest s of gelu_parts (2^-126) from |z| = 1e12 on.
  const float zc = __builtin_amdgcn_fmed3f(z, -16.0f, 16.0f);
  const float w = fmaf(0.21406445f, zc * zc, 1.5957691f);
  g = fmaf(h * w, es, s);
}

// ---- data preparation -------------------------------------------------------
// Coarse box-filtered fields, FP64: out[c][Nc] with c = rho, (rho u)x,
// (rho u)y, bx, by, (rho u u)xx, xy, yy, M(b)xx, M(b)xy.
constexpr int kFilt = 10;

//
// One thread per coarse node, bound by the read of the five fine fields.  The
// common factors are compiled in: a thread's loads are 16 bytes wide and all of
// a row of the block are in flight before the first sum, in the same order of
// summation as the general form.  2048^2 to 512^2: 45 us (general form: 54).
// double2 loads need an even factor and 16-byte aligned fields.
template <int FAC>
__global__ __launch_bounds__(256) void k_box_filter(const double *__restrict__ rho,
                                                    const double *__restrict__ u,
                                                    const double *__restrict__ b, int nf,
                                                    int fac_arg, double *__restrict__ out) {
  const int fac = FAC ? FAC : fac_arg;
  const int nc = nf / fac;
  const int64_t Nc = (int64_t)nc * nc, Nf = (int64_t)nf * nf;
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= Nc) return;
  const int cy = (int)(c / nc), cx = (int)(c - (int64_t)cy * nc);
  double acc[kFilt] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  auto add = [&](double r, double ux, double uy, double bx, double by) {
    acc[0] += r;
    acc[1] += r * ux;
    acc[2] += r * uy;
    acc[3] += bx;
    acc[4] += by;
    acc[5] += r * ux * ux;
    acc[6] += r * ux * uy;
    acc[7] += r * uy * uy;
    acc[8] += 0.5 * (by * by - bx * bx);  // M_xx = -M_yy
    acc[9] += -bx * by;                   // M_xy
  };
  for (int j = 0; j < fac; ++j) {
    const int64_t f = (int64_t)(cy * fac + j) * nf + (int64_t)cx * fac;
    if constexpr (FAC > 0) {
      constexpr int H = FAC / 2;
      const double2 *src[5] = {(const double2 *)(rho + f), (const double2 *)(u + f),
                               (const double2 *)(u + Nf + f), (const double2 *)(b + f),
                               (const double2 *)(b + Nf + f)};
      double2 v[5][H];
#pragma unroll
      for (int i = 0; i < H; ++i)
#pragma unroll
        for (int k = 0; k < 5; ++k) v[k][i] = src[k][i];
#pragma unroll
      for (int i = 0; i < H; ++i) {
        add(v[0][i].x, v[1][i].x, v[2][i].x, v[3][i].x, v[4][i].x);
        add(v[0][i].y, v[1][i].y, v[2][i].y, v[3][i].y, v[4][i].y);
      }
    } else {
      for (int i = 0; i < fac; ++i)
        add(rho[f + i], u[f + i], u[Nf + f + i], b[f + i], b[Nf + f + i]);
    }
  }
  const double inv = 1.0 / (fac * fac);
  for (int k = 0; k < kFilt; ++k) out[(int64_t)k * Nc + c] = acc[k] * inv;
}

static void launch_box_filter(const double *rho, const double *u, const double *b, int nf,
                              int fac, double *out, hipStream_t st) {
  const int64_t Nc = (int64_t)(nf / fac) * (nf / fac);
  const dim3 grid((unsigned)((Nc + 255) / 256));
  const bool wide = (((uintptr_t)rho | (uintptr_t)u | (uintptr_t)b) & 15) == 0;
  auto k = k_box_filter<0>;
  if (wide && fac == 2) k = k_box_filter<2>;
  if (wide && fac == 4) k = k_box_filter<4>;
  if (wide && fac == 8) k = k_box_filter<8>;
  hipLaunchKernelGGL(k, grid, dim3(256), 0, st, rho, u, b, nf, fac, out);
}

// Coarse features (rho_bar, u_bar, b_bar, a_CE) of node (cx, cy), FP64, from
// the filtered fields.
__device__ void features_at(const double *__restrict__ flt, int nc, double tau_c, int cx,
                            int cy, double out[8]) {
  const int64_t Nc = (int64_t)nc * nc;
  auto F = [&](int k, int xx, int yy) {
    xx = (xx + nc) % nc;
    yy = (yy + nc) % nc;
    return flt[(int64_t)k * Nc + (int64_t)yy * nc + xx];
  };
  auto ubar = [&](int comp, int xx, int yy) { return F(1 + comp, xx, yy) / F(0, xx, yy); };
  // isotropic gradient d_a phi = 3 sum_i w_i phi(x + c_i) c_ia on D2Q9
  double g[2][2] = {{0, 0}, {0, 0}};  // g[a][b] = d_a u_b
  for (int i = 1; i < 9; ++i) {
    const double w = 1.0 / (double)wdiv(i);
    for (int comp = 0; comp < 2; ++comp) {
      const double v = ubar(comp, cx + rr::cx(i), cy + rr::cy(i));
      g[0][comp] += 3.0 * w * v * rr::cx(i);
      g[1][comp] += 3.0 * w * v * rr::cy(i);
    }
  }
  const double r = F(0, cx, cy);
  const double k = -r * tau_c / 3.0;
  out[0] = r;
  out[1] = ubar(0, cx, cy);
  out[2] = ubar(1, cx, cy);
  out[3] = F(3, cx, cy);
  out[4] = F(4, cx, cy);
  out[5] = k * 2.0 * g[0][0];
  out[6] = k * (g[0][1] + g[1][0]);
  out[7] = k * 2.0 * g[1][1];
}

// Features x[Nc][8] and raw targets t[Nc][3] (FP32) from the filtered fields.
__global__ void k_samples(const double *__restrict__ flt, int nc, double tau_c,
                          float *__restrict__ x, float *__restrict__ t) {
  const int64_t Nc = (int64_t)nc * nc;
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= Nc) return;
  const int cy = (int)(c / nc), cx = (int)(c - (int64_t)cy * nc);
  double ft[8];
  features_at(flt, nc, tau_c, cx, cy, ft);
  for (int k = 0; k < 8; ++k) x[c * 8 + k] = (float)ft[k];
  const double r = ft[0], ux = ft[1], uy = ft[2], bx = ft[3], by = ft[4];
  auto F = [&](int k) { return flt[(int64_t)k * Nc + c]; };
  const double mbxx = 0.5 * (by * by - bx * bx), mbxy = -bx * by;
  const double sxx = F(5) - r * ux * ux + F(8) - mbxx;
  const double sxy = F(6) - r * ux * uy + F(9) - mbxy;
  const double syy = F(7) - r * uy * uy - F(8) + mbxx;
  const double inv = 1.0 / (tau_c - 1.0);
  t[c * 3 + 0] = (float)(sxx * inv);
  t[c * 3 + 1] = (float)(sxy * inv);
  t[c * 3 + 2] = (float)(syy * inv);
}

// ---- one-step objective: data preparation (FP64) ----------------------------
// Regularised expansion R_i . a of a second-order coefficient (axx, axy,
// ayy) at velocity u, without the weight: 9/2 H2:a + 27/2 (H_xxy a_xxy +
// H_xyy a_xyy) + 81/4 H_xxyy a_xxyy with the recursive a_xxy = 2 u_x a_xy +
// u_y a_xx, a_xyy = 2 u_y a_xy + u_x a_yy, a_xxyy = u_x^2 a_yy + u_y^2 a_xx +
// 4 u_x u_y a_xy; written with X2 = 3 c_x^2 - 1 = 3 H_xx, Y2 = 3 c_y^2 - 1.
template <typename R>
__device__ __forceinline__ R reg_expand(int i, R ux, R uy, R axx, R axy, R ayy) {
  const R X2 = (R)(3 * rr::cx(i) * rr::cx(i) - 1), Y2 = (R)(3 * rr::cy(i) * rr::cy(i) - 1);
  const R CX = (R)rr::cx(i), CY = (R)rr::cy(i);
  const R a3x = 2 * ux * axy + uy * axx, a3y = 2 * uy * axy + ux * ayy;
  const R a4 = ux * ux * ayy + uy * uy * axx + 4 * ux * uy * axy;
  return (R)1.5 * (X2 * axx + Y2 * ayy) + (R)9 * CX * CY * axy +
         (R)4.5 * (CY * X2 * a3x + CX * Y2 * a3y) + (R)2.25 * X2 * Y2 * a4;
}

// Equilibrium population i (fourth-order Hermite with the Maxwell stress at
// second order), FP64.
__device__ __forceinline__ double feq64(int i, double rho, double ux, double uy, double bx,
                                        double by) {
  const double X2 = 3 * rr::cx(i) * rr::cx(i) - 1, Y2 = 3 * rr::cy(i) * rr::cy(i) - 1;
  const double CX = rr::cx(i), CY = rr::cy(i);
  const double Axx = rho * ux * ux + 0.5 * (by * by - bx * bx);
  const double Axy = rho * ux * uy - bx * by;
  const double Ayy = rho * uy * uy + 0.5 * (bx * bx - by * by);
  const double t2 = 1.5 * (X2 * Axx + Y2 * Ayy) + 9.0 * CX * CY * Axy;
  const double t3 = 4.5 * rho * (CY * X2 * ux * ux * uy + CX * Y2 * ux * uy * uy);
  const double t4 = 2.25 * rho * X2 * Y2 * ux * ux * uy * uy;
  return (rho + 3.0 * rho * (CX * ux + CY * uy) + t2 + t3 + t4) / (double)wdiv(i);
}

// FP64 features of every coarse node: feat[8][Nc].
__global__ void k_features64(const double *__restrict__ flt, int nc, double tau_c,
                             double *__restrict__ feat) {
  const int64_t Nc = (int64_t)nc * nc;
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= Nc) return;
  const int cy = (int)(c / nc), cx = (int)(c - (int64_t)cy * nc);
  double ft[8];
  features_at(flt, nc, tau_c, cx, cy, ft);
  for (int k = 0; k < 8; ++k) feat[(int64_t)k * Nc + c] = ft[k];
}

// Sum over a workgroup of 256 in a fixed tree; the result is thread 0's.
__device__ __forceinline__ double block_sum64(double a, double *red) {
  red[threadIdx.x] = a;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  return red[0];
}

// x[Nc][8] (FP32 features), r0[Nc][2] = j_c(X)|_{D=0} - j_bar(X, t + fac)
// (FP32 of FP64), and per workgroup of 256 nodes the FP64 sum dm of
// |j_bar(t + fac) - j_bar(t)|^2 in a fixed tree, so that the closing sum reads
// one value per workgroup instead of walking Nc values in a single one
// (512^2: 258 us of one workgroup's serial loads became 4.7, and 2 here).
__global__ __launch_bounds__(256) void k_onestep_prep(const double *__restrict__ flt0,
                                                      const double *__restrict__ flt1,
                                                      const double *__restrict__ feat, int nc,
                                                      double omega, float *__restrict__ x,
                                                      float *__restrict__ r0,
                                                      double *__restrict__ dm) {
  const int64_t Nc = (int64_t)nc * nc;
  const int64_t own = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t c = own < Nc ? own : Nc - 1;  // past the end: the last node again, not stored
  const int cy = (int)(c / nc), cx = (int)(c - (int64_t)cy * nc);
  if (own < Nc) {
#pragma unroll
    for (int k = 0; k < 8; ++k) x[c * 8 + k] = (float)feat[(int64_t)k * Nc + c];
  }
  double jx = 0.0, jy = 0.0;
  for (int i = 1; i < 9; ++i) {
    // f*_i of the upstream node Y = X - c_i arrives at X
    const int yx = (cx - rr::cx(i) + nc) % nc, yy = (cy - rr::cy(i) + nc) % nc;
    const int64_t q = (int64_t)yy * nc + yx;
    double v[8];
    for (int k = 0; k < 8; ++k) v[k] = feat[(int64_t)k * Nc + q];
    const double fs = feq64(i, v[0], v[1], v[2], v[3], v[4]) +
                      (1.0 - omega) * reg_expand<double>(i, v[1], v[2], v[5], v[6], v[7]) /
                          (double)wdiv(i);
    jx += rr::cx(i) * fs;
    jy += rr::cy(i) * fs;
  }
  const double j1x = flt1[1 * Nc + c], j1y = flt1[2 * Nc + c];
  const double dx = j1x - flt0[1 * Nc + c], dy = j1y - flt0[2 * Nc + c];
  if (own < Nc) {
    r0[2 * c + 0] = (float)(jx - j1x);
    r0[2 * c + 1] = (float)(jy - j1y);
  }
  __shared__ double red[256];
  const double sum = block_sum64(own < Nc ? dx * dx + dy * dy : 0.0, red);
  if (threadIdx.x == 0) dm[blockIdx.x] = sum;
}

// out[0] = sum of v[0..n) in a fixed order (one workgroup of 256).
__global__ __launch_bounds__(256) void k_sum64(const double *__restrict__ v, int64_t n,
                                               double *__restrict__ out) {
  __shared__ double red[256];
  double a = 0.0;
  for (int64_t k = threadIdx.x; k < n; k += 256) a += v[k];
  a = block_sum64(a, red);
  if (threadIdx.x == 0) out[0] = a;
}

// ---- the network in FP32 on matrix cores --------------------------------------
// A wavefront holds 16 samples as the columns of 16x16x4 FP32 MFMAs, written
// transposed (Z^T = W X^T): lane (column c, quarter q), register r of block b
// is hidden unit 16 b + 4 q + r.  A layer's activations feed the next product's
// B operand register by register: step r of block b takes the four units that
// register r holds in the four quarters, and the A operand is read from the
// weights in LDS in that order (one 16-byte read per block), so activations
// never leave their registers.  The gradient products contract over the
// samples, which need the other orientation: each wavefront turns its 64 x 16
// blocks through LDS, and the four wavefronts of a workgroup share out the
// products over their 64 samples (wavefront w keeps rows 16 w .. 16 w + 15 of
// dW2 and dW1 and columns 16 w .. of dW3).
//
// Activations are recomputed in the reverse pass, not stored: the former
// kernels kept 395 floats per sample in memory and reduced the weight gradients
// with one thread per parameter reading whole sample rows (4.4 ms per
// activation set at 262,144 samples).  A training step of the feedback form on
// 512^2 nodes: 9260 us before, 304 us now (k_net_grad 217, k_net_forward
// 92); its products take 130 us at the FP32 matrix rate (150 TFLOP/s measured).
// Of the same design with 32-sample wavefronts (32x32x2 MFMAs), one wavefront
// per SIMD holding all of dW2 took 360 us in k_net_grad, and eight in one workgroup
// 308 (in step with each other at every barrier, and out of registers).
struct alignas(16) NetLds {
  float w2[kNH][kNH + 4];       // W2, rows padded against bank conflicts
  float w1[kNH][kNIN + 4];      // W1
  float w1t[kNOUT][kNH];        // columns 5..7 of W1 (the a_1^(2) inputs)
  float w3[kNOUT][kNH];
  float b1[kNH], b2[kNH];
  float mu[kNIN], sigma[kNIN];
  float b3[kNOUT], so[kNOUT], pad_[2];
};
constexpr int kNetWaves = 4, kNetThreads = 64 * kNetWaves;
constexpr int kNetGroup = 16;  // samples of a wavefront's pass
typedef float floatx2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void net_to_lds(NetLds &W, const float *__restrict__ p,
                                           const float *__restrict__ norm) {
  const int t = threadIdx.x;
  for (int k = t; k < kNH * kNH; k += kNetThreads) W.w2[k / kNH][k % kNH] = p[kOffW2 + k];
  for (int k = t; k < kNH * kNIN; k += kNetThreads) {
    const float v = p[kOffW1 + k];
    W.w1[k / kNIN][k % kNIN] = v;
    if (k % kNIN >= 5) W.w1t[k % kNIN - 5][k / kNIN] = v;
  }
  for (int k = t; k < kNOUT * kNH; k += kNetThreads) W.w3[k / kNH][k % kNH] = p[kOffW3 + k];
  if (t < kNH) {
    W.b1[t] = p[kOffB1 + t];
    W.b2[t] = p[kOffB2 + t];
  }
  if (t < kNOUT) {
    W.b3[t] = p[kOffB3 + t];
    W.so[t] = norm[2 * kNIN + t];
  }
  if (t < kNIN) {
    W.mu[t] = norm[t];
    W.sigma[t] = norm[kNIN + t];
  }
  __syncthreads();
}

__device__ __forceinline__ floatx4 ld_f4(const float *p) {
  floatx4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}
// Keeps the weights in LDS (not hoisted into registers) and the phases of a
// pass apart.
__device__ __forceinline__ void net_phase() { asm volatile("" ::: "memory"); }

// The lane's share of a wavefront: column c (sample), quarter q.
struct NetLane {
  int c, q;
};
__device__ __forceinline__ NetLane net_lane() {
  return NetLane{(int)threadIdx.x & 15, ((int)threadIdx.x >> 4) & 3};
}

// Pre-activations of layer 1 from the lane's two normalised features (2 q and
// 2 q + 1 of its sample).
__device__ __forceinline__ void net_layer1(const NetLds &W, const float (&xh)[2], NetLane L,
                                           floatx4 (&z)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    z[m] = ld_f4(W.b1 + 16 * m + 4 * L.q);
    floatx2_t a;
    __builtin_memcpy(&a, &W.w1[16 * m + L.c][2 * L.q], 8);
    z[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], xh[0], z[m], 0, 0, 0);
    z[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], xh[1], z[m], 0, 0, 0);
  }
}
// z = b + W2 h (layer 2).
__device__ __forceinline__ void net_layer2(const NetLds &W, const floatx4 (&h)[4], NetLane L,
                                           floatx4 (&z)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) z[m] = ld_f4(W.b2 + 16 * m + 4 * L.q);
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const floatx4 a = ld_f4(&W.w2[16 * m + L.c][16 * b + 4 * L.q]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        z[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], h[b][r], z[m], 0, 0, 0);
    }
}
// d = W2^T z.
__device__ __forceinline__ void net_layer2_t(const NetLds &W, const floatx4 (&z)[4], NetLane L,
                                             floatx4 (&d)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) d[m] = floatx4{0};
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int m = 0; m < 4; ++m)
        d[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(W.w2[16 * b + 4 * L.q + r][16 * m + L.c],
                                                    z[b][r], d[m], 0, 0, 0);
}
// Rows `m` (3 x 64) times the activations, summed over the quarters.
__device__ __forceinline__ void net_rows3(const float (&m)[kNOUT][kNH], const floatx4 (&h)[4],
                                          NetLane L, float (&y)[kNOUT]) {
#pragma unroll
  for (int o = 0; o < kNOUT; ++o) {
    float a = 0.0f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const floatx4 w = ld_f4(&m[o][16 * b + 4 * L.q]);
#pragma unroll
      for (int r = 0; r < 4; ++r) a = fmaf(w[r], h[b][r], a);
    }
    a += __shfl_xor(a, 16, 64);
    y[o] = a + __shfl_xor(a, 32, 64);
  }
}

// The lane's two features of sample s, its a_1^(2) entries (features 5, 6, 7)
// shifted by qv, normalised.
__device__ __forceinline__ void net_features(const NetLds &W, const float *__restrict__ x,
                                             int64_t s, NetLane L, const float (&qv)[kNOUT],
                                             float (&xh)[2]) {
  floatx2_t f;
  __builtin_memcpy(&f, x + s * kNIN + 2 * L.q, 8);
  if (L.q == 2) f[1] += qv[0];
  if (L.q == 3) {
    f[0] += qv[1];
    f[1] += qv[2];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) xh[k] = (f[k] - W.mu[2 * L.q + k]) / W.sigma[2 * L.q + k];
}

// D = sigma_out y of every sample (SoA [3][n]).  FEEDBACK: a first pass gives
// q = (tau_c - 1) sigma_out y(x) (SoA, kept), the second runs on x with its
// a_1^(2) entries shifted by q, and D = sigma_out y + q.
template <bool FEEDBACK>
__global__ __launch_bounds__(kNetThreads) void k_net_forward(const float *__restrict__ p,
                                                             const float *__restrict__ norm,
                                                             const float *__restrict__ x, int n,
                                                             float tm1, float *__restrict__ q,
                                                             float *__restrict__ D) {
  __shared__ NetLds W;
  net_to_lds(W, p, norm);
  const NetLane L = net_lane();
  const int groups = (n + kNetGroup - 1) / kNetGroup;
  for (int g = blockIdx.x * kNetWaves + (threadIdx.x >> 6); g < groups;
       g += gridDim.x * kNetWaves) {
    const int64_t s = (int64_t)g * kNetGroup + L.c, sc = s < n ? s : n - 1;
    float xh[2], y[kNOUT], qv[kNOUT] = {0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int pass = FEEDBACK ? 0 : 1; pass < 2; ++pass) {
      net_phase();
      net_features(W, x, sc, L, qv, xh);
      floatx4 h[4], z[4];
      net_layer1(W, xh, L, h);
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) h[b][r] = gelu32(h[b][r]);
      net_layer2(W, h, L, z);
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) z[b][r] = gelu32(z[b][r]);
      net_rows3(W.w3, z, L, y);
#pragma unroll
      for (int o = 0; o < kNOUT; ++o) {
        y[o] = W.so[o] * (y[o] + W.b3[o]);
        if (FEEDBACK && pass == 0) qv[o] = tm1 * y[o];
      }
    }
    if (s < n && L.q < kNOUT) {  // quarter o writes output o
      const float d = L.q == 0 ? y[0] : (L.q == 1 ? y[1] : y[2]);
      const float v = L.q == 0 ? qv[0] : (L.q == 1 ? qv[1] : qv[2]);
      D[(int64_t)L.q * n + s] = FEEDBACK ? d + v : d;
      if (FEEDBACK) q[(int64_t)L.q * n + s] = v;
    }
  }
}

// Gradient accumulators of a wavefront: its rows of dW2 (four 16 x 16 blocks)
// and dW1 (unit, feature), its columns of dW3 (output, unit), the biases of its
// rows (this lane's quarter of the samples) and of the outputs (its sample).
struct NetGrad {
  floatx4 w2[4], w1, w3;
  float b1, b2, b3[kNOUT];
};
// A wavefront's turning buffers (64 units x 16 samples).
struct alignas(16) NetTurn {
  float a[kNH][kNetGroup + 4], b[kNH][kNetGroup + 4];
};
__device__ __forceinline__ void turn_in(float (*t)[kNetGroup + 4], const floatx4 (&v)[4],
                                        NetLane L) {
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) t[16 * b + 4 * L.q + r][L.c] = v[b][r];
}

// Forward again and reverse mode for the lane's sample; the whole workgroup
// calls it together.  dy: dL/dy, or (LOSS) formed here from the target t
// (already over sigma_out) and the squared residual added to `loss`; live =
// false adds nothing.  gx[3] (GX) = dL/d of the normalised a_1^(2) inputs.
template <bool LOSS, bool GX>
__device__ __forceinline__ void net_reverse(const NetLds &W, NetTurn *TT, NetGrad &G,
                                            const float (&xh)[2], float (&dy)[kNOUT],
                                            const float (&t)[kNOUT], float scale, bool live,
                                            float &loss, float (&gx)[kNOUT]) {
  const NetLane L = net_lane();
  const int wave = threadIdx.x >> 6;
  NetTurn &T = TT[wave];
  floatx4 h1[4], g1[4], z[4];
  net_layer1(W, xh, L, z);
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float h, g;
      gelu_pair(z[b][r], h, g);
      h1[b][r] = h;
      g1[b][r] = g;
    }
  net_layer2(W, h1, L, z);
  // h2 to the turning buffer (and, for the loss, through layer 3); z becomes
  // the derivative
  float y[kNOUT] = {0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float h, g;
      gelu_pair(z[b][r], h, g);
      const int u = 16 * b + 4 * L.q + r;
      T.b[u][L.c] = h;
      if (LOSS) {
#pragma unroll
        for (int o = 0; o < kNOUT; ++o) y[o] = fmaf(W.w3[o][u], h, y[o]);
      }
      z[b][r] = g;
    }
  if (LOSS) {
#pragma unroll
    for (int o = 0; o < kNOUT; ++o) {
      float a = y[o];
      a += __shfl_xor(a, 16, 64);
      a += __shfl_xor(a, 32, 64);
      const float r = (a + W.b3[o]) - t[o];
      if (live && L.q == 0) loss = fmaf(r, r, loss);
      dy[o] = live ? 2.0f * r * scale : 0.0f;
    }
  }
  if (L.q == 0) {
#pragma unroll
    for (int o = 0; o < kNOUT; ++o) {
      T.a[o][L.c] = dy[o];
      G.b3[o] += dy[o];
    }
  }
  __syncthreads();
  // dW3 (rows 3 .. 15 of the product are zero)
#pragma unroll
  for (int w = 0; w < kNetWaves; ++w) {
    floatx4 a = {0.0f, 0.0f, 0.0f, 0.0f};
    if (L.c < kNOUT) a = ld_f4(&TT[w].a[L.c][4 * L.q]);
    const floatx4 b = ld_f4(&TT[w].b[16 * wave + L.c][4 * L.q]);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      G.w3 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b[r], G.w3, 0, 0, 0);
  }
  // dz2 = (W3^T dy) gelu'(z2)
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    floatx4 d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int o = 0; o < kNOUT; ++o) {
      const floatx4 w = ld_f4(&W.w3[o][16 * b + 4 * L.q]);
#pragma unroll
      for (int r = 0; r < 4; ++r) d[r] = fmaf(w[r], dy[o], d[r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) z[b][r] *= d[r];
  }
  __syncthreads();
  // dW2 and db2
  turn_in(T.a, z, L);
  turn_in(T.b, h1, L);
  __syncthreads();
#pragma unroll 2
  for (int w = 0; w < kNetWaves; ++w) {
    const floatx4 a = ld_f4(&TT[w].a[16 * wave + L.c][4 * L.q]);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const floatx4 b = ld_f4(&TT[w].b[16 * nb + L.c][4 * L.q]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        G.w2[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b[r], G.w2[nb], 0, 0, 0);
    }
    G.b2 += (a[0] + a[1]) + (a[2] + a[3]);
  }
  // dz1 = (W2^T dz2) gelu'(z1); dW1 and db1
  net_layer2_t(W, z, L, h1);
#pragma unroll
  for (int b = 0; b < 4; ++b) h1[b] *= g1[b];
  __syncthreads();
  turn_in(T.a, h1, L);
  T.b[2 * L.q][L.c] = xh[0];
  T.b[2 * L.q + 1][L.c] = xh[1];
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kNetWaves; ++w) {
    const floatx4 a = ld_f4(&TT[w].a[16 * wave + L.c][4 * L.q]);
    floatx4 b = {0.0f, 0.0f, 0.0f, 0.0f};
    if (L.c < kNIN) b = ld_f4(&TT[w].b[L.c][4 * L.q]);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      G.w1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b[r], G.w1, 0, 0, 0);
    G.b1 += (a[0] + a[1]) + (a[2] + a[3]);
  }
  if (GX) net_rows3(W.w1t, h1, L, gx);
  __syncthreads();
}

// The workgroup's accumulators in `out` (the parameter vector's order); b3: the
// wavefronts' sums of dy.
__device__ __forceinline__ void net_grad_out(const NetGrad &G, float *out, float (*b3)[kNOUT]) {
  const NetLane L = net_lane();
  const int wave = threadIdx.x >> 6;
  float v1 = G.b1, v2 = G.b2;
  v1 += __shfl_xor(v1, 16, 64);
  v1 += __shfl_xor(v1, 32, 64);
  v2 += __shfl_xor(v2, 16, 64);
  v2 += __shfl_xor(v2, 32, 64);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * L.q + r;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
      out[kOffW2 + (16 * wave + row) * kNH + 16 * nb + L.c] = G.w2[nb][r];
    if (L.c < kNIN) out[kOffW1 + (16 * wave + row) * kNIN + L.c] = G.w1[r];
    if (row < kNOUT) out[kOffW3 + row * kNH + 16 * wave + L.c] = G.w3[r];
  }
  if (L.q == 0) {
    out[kOffB1 + 16 * wave + L.c] = v1;
    out[kOffB2 + 16 * wave + L.c] = v2;
  }
#pragma unroll
  for (int o = 0; o < kNOUT; ++o) {
    float v = G.b3[o];  // samples of quarter 0
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) b3[wave][o] = v;
  }
  __syncthreads();
  if (threadIdx.x < kNOUT) {
    const int o = threadIdx.x;
    out[kOffB3 + o] = (b3[0][o] + b3[1][o]) + (b3[2][o] + b3[3][o]);
  }
}

// Parameter gradient of a batch: part[block][4931], and (apriori) the block's
// sum of squared residuals.  NET_APRIORI: mean squared error against the
// target tg over sigma_out.  NET_ONESTEP: dL/dD per sample (gE, SoA) from the
// one-step stencil.  NET_FEEDBACK: the same through both network passes, the
// second on the features shifted by q, the first with dL/dq = gE + dL/dx1.
// Every sum has a fixed order: the samples of a workgroup's passes, then
// (k_net_final) the workgroups.
enum { NET_APRIORI = 0, NET_ONESTEP = 1, NET_FEEDBACK = 2 };
template <int MODE>
__global__ __launch_bounds__(kNetThreads, 2) void k_net_grad(
    const float *__restrict__ p, const float *__restrict__ norm, const float *__restrict__ x,
    const float *__restrict__ tg, const float *__restrict__ q, const float *__restrict__ gE, int n,
    float tm1, float *__restrict__ part, float *__restrict__ loss_part) {
  __shared__ NetLds W;
  __shared__ NetTurn T[kNetWaves];
  __shared__ float red[kNetWaves][kNOUT];
  net_to_lds(W, p, norm);
  const NetLane L = net_lane();
  const int wave = threadIdx.x >> 6;
  NetGrad G{};
  float loss = 0.0f;
  const float scale = 1.0f / (float)n;
  const int groups = (n + kNetGroup - 1) / kNetGroup;
  // the wavefronts of a workgroup stay together (barriers in net_reverse)
  for (int g0 = blockIdx.x * kNetWaves; g0 < groups; g0 += gridDim.x * kNetWaves) {
    const int64_t s = (int64_t)(g0 + wave) * kNetGroup + L.c;
    const bool live = s < n;
    const int64_t sc = live ? s : n - 1;
    float xh[2], dy[kNOUT] = {0.0f, 0.0f, 0.0f}, t[kNOUT] = {0.0f, 0.0f, 0.0f};
    float ge[kNOUT] = {0.0f, 0.0f, 0.0f}, gx[kNOUT];
    if (MODE == NET_APRIORI) {
#pragma unroll
      for (int o = 0; o < kNOUT; ++o) t[o] = tg[sc * kNOUT + o] / W.so[o];
    } else if (live) {
#pragma unroll
      for (int o = 0; o < kNOUT; ++o) ge[o] = gE[(int64_t)o * n + s];
    }
#pragma unroll 1
    for (int pass = MODE == NET_FEEDBACK ? 1 : 0; pass >= 0; --pass) {
      net_phase();
      float qv[kNOUT] = {0.0f, 0.0f, 0.0f};
      if (MODE == NET_FEEDBACK && pass == 1) {
#pragma unroll
        for (int o = 0; o < kNOUT; ++o) qv[o] = q[(int64_t)o * n + sc];
      }
      net_features(W, x, sc, L, qv, xh);
      if (!live) xh[0] = xh[1] = 0.0f;  // finite whatever the sample, without effect: dy = 0
      if (MODE != NET_APRIORI) {
#pragma unroll
        for (int o = 0; o < kNOUT; ++o)
          dy[o] = W.so[o] * (MODE == NET_FEEDBACK && pass == 0 ? tm1 * ge[o] : ge[o]);
      }
      net_reverse<MODE == NET_APRIORI, MODE == NET_FEEDBACK>(W, T, G, xh, dy, t, scale, live, loss,
                                                             gx);
      if (MODE == NET_FEEDBACK) {
#pragma unroll
        for (int o = 0; o < kNOUT; ++o) ge[o] = live ? ge[o] + gx[o] / W.sigma[5 + o] : 0.0f;
      }
    }
  }
  net_grad_out(G, part + (int64_t)blockIdx.x * kNParam, red);
  if (MODE == NET_APRIORI) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) loss += __shfl_xor(loss, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave][0] = loss;
    __syncthreads();
    if (threadIdx.x == 0) loss_part[blockIdx.x] = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
  }
}

// grad = sum of the blocks' partial gradients (16 parameters x 16 slices of the
// blocks per workgroup, FP64), loss = loss_scale * sum of loss_part (the last
// workgroup, FP64).
__global__ __launch_bounds__(256) void k_net_final(const float *__restrict__ part, int nparts,
                                                   const float *__restrict__ loss_part, int nlb,
                                                   double loss_scale, float *__restrict__ grad,
                                                   float *__restrict__ loss) {
  __shared__ double red[256];
  const int t = threadIdx.x, j = t & 15, slice = t >> 4;
  double a = 0.0;
  if (blockIdx.x + 1 < gridDim.x) {
    const int k = blockIdx.x * 16 + j;
    if (k < kNParam)
      for (int c = slice; c < nparts; c += 16) a += (double)part[(int64_t)c * kNParam + k];
    red[t] = a;
    __syncthreads();
    if (slice == 0 && k < kNParam) {
      for (int c = 1; c < 16; ++c) a += red[16 * c + j];
      grad[k] = (float)a;
    }
    return;
  }
  if (!loss) return;
  for (int c = t; c < nlb; c += 256) a += (double)loss_part[c];
  red[t] = a;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  if (t == 0) *loss = (float)(red[0] * loss_scale);
}

// One-step objective, network-dependent part (FP32).  Node s of the batch is
// node s % Nc of snapshot s / Nc (periodic nc x nc).  D (SoA [3][n]): the
// correction each node's collision relaxes.  res[2][n] = r0 + sum_i c_i (1 -
// omega) w_i R_i(u(X - c_i)) . D(X - c_i); loss_part = per-workgroup sums of
// |res|^2.
__global__ __launch_bounds__(kTB) void k_onestep_fwd(const float *__restrict__ x,
                                                     const float *__restrict__ r0, int nsnap,
                                                     int nc, float om1,
                                                     const float *__restrict__ D,
                                                     float *__restrict__ res,
                                                     float *__restrict__ loss_part) {
  __shared__ float red[kTB / 64];
  const int Nc = nc * nc, n = nsnap * Nc;
  const int s = blockIdx.x * kTB + threadIdx.x;
  float l = 0.0f;
  if (s < n) {
    const int sn = s / Nc, c = s - sn * Nc;
    const int cy = c / nc, cx = c - cy * nc;
    float jx = r0[2 * (int64_t)s], jy = r0[2 * (int64_t)s + 1];
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      const int yx = (cx - rr::cx(i) + nc) % nc, yy = (cy - rr::cy(i) + nc) % nc;
      const int qn = sn * Nc + yy * nc + yx;
      const float ux = x[(int64_t)qn * kNIN + 1], uy = x[(int64_t)qn * kNIN + 2];
      const float d = om1 *
                      reg_expand<float>(i, ux, uy, D[qn], D[(int64_t)n + qn],
                                        D[2 * (int64_t)n + qn]) /
                      wdiv(i);
      if (rr::cx(i)) jx = fmaf((float)rr::cx(i), d, jx);
      if (rr::cy(i)) jy = fmaf((float)rr::cy(i), d, jy);
    }
    res[s] = jx;
    res[(int64_t)n + s] = jy;
    l = fmaf(jx, jx, jy * jy);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) l += __shfl_xor(l, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = l;
  __syncthreads();
  if (threadIdx.x == 0) loss_part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Transpose stencil: dL/dD_k(Y) = scale om1 sum_i (c_i . res(Y + c_i)) w_i
// dR_i/dD_k(u(Y)), scale = 2 / den, SoA [3][n].
__global__ __launch_bounds__(kTB) void k_onestep_adj(const float *__restrict__ x, int nsnap,
                                                     int nc, float om1, float scale,
                                                     const float *__restrict__ res,
                                                     float *__restrict__ gE) {
  const int Nc = nc * nc, n = nsnap * Nc;
  const int s = blockIdx.x * kTB + threadIdx.x;
  if (s >= n) return;
  const int sn = s / Nc, c = s - sn * Nc;
  const int cy = c / nc, cx = c - cy * nc;
  const float ux = x[(int64_t)s * kNIN + 1], uy = x[(int64_t)s * kNIN + 2];
  float gxx = 0.0f, gxy = 0.0f, gyy = 0.0f;
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    const int xx = (cx + rr::cx(i) + nc) % nc, xy = (cy + rr::cy(i) + nc) % nc;
    const int q = sn * Nc + xy * nc + xx;
    const float m = ((float)rr::cx(i) * res[q] + (float)rr::cy(i) * res[(int64_t)n + q]) / wdiv(i);
    // columns of the linear map D -> R_i . D
    gxx = fmaf(m, reg_expand<float>(i, ux, uy, 1.0f, 0.0f, 0.0f), gxx);
    gxy = fmaf(m, reg_expand<float>(i, ux, uy, 0.0f, 1.0f, 0.0f), gxy);
    gyy = fmaf(m, reg_expand<float>(i, ux, uy, 0.0f, 0.0f, 1.0f), gyy);
  }
  const float k = scale * om1;
  gE[s] = k * gxx;
  gE[(int64_t)n + s] = k * gxy;
  gE[2 * (int64_t)n + s] = k * gyy;
}

__global__ void k_adam(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ g, int n, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const float gk = g[k];
  const float mk = fmaf(b1, m[k], (1.0f - b1) * gk);
  const float vk = fmaf(b2, v[k], (1.0f - b2) * gk * gk);
  m[k] = mk;
  v[k] = vk;
  p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

// ---- imposed fluid state (best-velocity bound of the closure protocol) ----
// Writes the fluid planes of a periodic two-buffer state so that the pulled
// populations of node X are f_eq(rho(X), j(X) / rho(X), b(X)), FP64
// evaluated, stored in the handle's codec: the slot of population i at node
// Y is pulled by Y + c_i, so it receives that node's equilibrium.  The
// magnetic planes are not touched.
template <class C>
__global__ void k_impose_fluid(PlaneGeom G, const double *__restrict__ rho,
                               const double *__restrict__ j, const double *__restrict__ b,
                               typename C::T *__restrict__ dst) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y;
  if (x >= G.nx) return;
  const int64_t N = (int64_t)G.nx * G.ny;
  const int64_t o = (int64_t)y * G.row + x;  // stored state
  for (int i = 0; i < 9; ++i) {
    int tx = x + rr::cx(i), ty = y + rr::cy(i);
    tx = tx < 0 ? tx + G.nx : (tx >= G.nx ? tx - G.nx : tx);
    ty = ty < 0 ? ty + G.ny : (ty >= G.ny ? ty - G.ny : ty);
    const int64_t q = (int64_t)ty * G.nx + tx;
    const double r = rho[q];
    const double f = feq64(i, r, j[q] / r, j[N + q] / r, b[q], b[N + q]);
    dst[(int64_t)i * G.plane + o] = C::enc((float)(f - 1.0 / (double)wdiv(i)), G.s);
  }
}

}  // namespace rr

// Launcher used by rrmhd_train_impose_fluid (rr_api.hip).
extern "C" RR_HIDDEN int rr_launch_impose_fluid(int storage, const rr::Domain *D, void *dst,
                                                const double *rho, const double *j,
                                                const double *b, hipStream_t st) {
  const dim3 block(64), grid((D->nx + 63) / 64, D->ny);
  const rr::PlaneGeom G{D->plane, D->nx, D->ny, D->s, D->inv_s, 0u, D->row};
  if (storage == rr::kF16)
    hipLaunchKernelGGL(rr::k_impose_fluid<rr::CodecF16>, grid, block, 0, st, G, rho, j, b,
                       (uint16_t *)dst);
  else
    hipLaunchKernelGGL(rr::k_impose_fluid<rr::CodecF32>, grid, block, 0, st, G, rho, j, b,
                       (float *)dst);
  return hipGetLastError() == hipSuccess ? RRMHD_OK : RRMHD_EDEVICE;
}

// ---------------------------------------------------------------------------
// C-ABI
// ---------------------------------------------------------------------------
// Workgroups of the network kernels, at most one per 64 samples: two per CU in
// the reverse pass (LDS), four in the forward one (registers).
static int net_blocks(int64_t n, int most = 512) {
  const int64_t per = rr::kNetWaves * rr::kNetGroup, b = (n + per - 1) / per;
  return (int)(b < most ? b : most);
}

struct rrmhd_trainer {
  int64_t cap = 0;
  hipStream_t st = nullptr;
  float *part = nullptr;       // [blocks][4931] partial gradients
  float *loss_part = nullptr;  // partial losses
  float *node = nullptr;       // per sample: D [3], q [3], residual [2], dL/dD [3] (SoA)
};

namespace {
thread_local char g_tdetail[256] = "";
int terr(hipError_t e, const char *w) {
  std::snprintf(g_tdetail, sizeof g_tdetail, "%s: %s", w, hipGetErrorString(e));
  return e == hipErrorOutOfMemory ? RRMHD_ENOMEM : RRMHD_EDEVICE;
}
#define THIP(expr)                                  \
  do {                                              \
    hipError_t e_ = (expr);                         \
    if (e_ != hipSuccess) return terr(e_, #expr);   \
  } while (0)
}  // namespace

extern "C" {

int rrmhd_train_destroy(rrmhd_trainer *t) {
  if (!t) return RRMHD_OK;
  (void)hipStreamSynchronize(t->st);
  if (t->part) (void)hipFree(t->part);
  if (t->loss_part) (void)hipFree(t->loss_part);
  if (t->node) (void)hipFree(t->node);
  delete t;
  return RRMHD_OK;
}

int rrmhd_train_create(int64_t max_batch, void *hip_stream, rrmhd_trainer **out) {
  if (!out) return RRMHD_EINVAL;
  *out = nullptr;
  if (max_batch < 1 || max_batch > (int64_t)1 << 26) return RRMHD_EINVAL;
  rrmhd_trainer *t = new (std::nothrow) rrmhd_trainer();
  if (!t) return RRMHD_ENOMEM;
  t->cap = max_batch;
  t->st = (hipStream_t)hip_stream;
  // partial losses: of the stencil's workgroups, or of the network's
  int64_t lblocks = (max_batch + rr::kTB - 1) / rr::kTB;
  if (lblocks < net_blocks(max_batch)) lblocks = net_blocks(max_batch);
  hipError_t e = hipMalloc((void **)&t->part,
                           sizeof(float) * (int64_t)net_blocks(max_batch) * rr::kNParam);
  if (e == hipSuccess) e = hipMalloc((void **)&t->loss_part, sizeof(float) * lblocks);
  if (e == hipSuccess) e = hipMalloc((void **)&t->node, sizeof(float) * 11 * max_batch);
  if (e != hipSuccess) {
    int rc = terr(e, "hipMalloc(trainer)");
    rrmhd_train_destroy(t);
    return rc;
  }
  *out = t;
  return RRMHD_OK;
}

}  // extern "C"

// The partial gradients summed, and the loss.
static int net_final(rrmhd_trainer *t, int nparts, int nlb, double loss_scale, float *grad,
                     float *loss) {
  hipLaunchKernelGGL(rr::k_net_final, dim3((rr::kNParam + 15) / 16 + 1), dim3(256), 0, t->st,
                     (const float *)t->part, nparts, (const float *)t->loss_part, nlb, loss_scale,
                     grad, loss);
  THIP(hipGetLastError());
  return RRMHD_OK;
}

extern "C" {

int rrmhd_train_loss_grad(rrmhd_trainer *t, const float *params, const float *norm,
                          const float *x, const float *target, int64_t n, float *grad,
                          float *loss) {
  if (!t || !params || !norm || !x || !target || !grad || n < 1 || n > t->cap)
    return RRMHD_EINVAL;
  const int nb = net_blocks(n);
  hipLaunchKernelGGL(rr::k_net_grad<rr::NET_APRIORI>, dim3(nb), dim3(rr::kNetThreads), 0, t->st,
                     params, norm, x, target, (const float *)nullptr, (const float *)nullptr,
                     (int)n, 0.0f, t->part, t->loss_part);
  THIP(hipGetLastError());
  return net_final(t, nb, nb, 1.0 / (double)n, grad, loss);
}

int rrmhd_train_onestep_loss_grad(rrmhd_trainer *t, const float *params, const float *norm,
                                  const float *x, const float *r0, int nsnap, int nc,
                                  double tau_c, double den, int feedback, float *grad,
                                  float *loss) {
  if (!t || !params || !norm || !x || !r0 || !grad || nsnap < 1 || nc < 1 ||
      !(tau_c > 0.5) || !(den > 0.0) || !std::isfinite(den) || (feedback != 0 && feedback != 1))
    return RRMHD_EINVAL;
  const int64_t n = (int64_t)nsnap * nc * nc;
  if (n > t->cap || n > INT32_MAX) return RRMHD_EINVAL;
  const int nb = (int)((n + rr::kTB - 1) / rr::kTB), ng = net_blocks(n);
  const int nf = net_blocks(n, 1024);
  const float om1 = (float)(1.0 - 1.0 / tau_c), tm1 = (float)(tau_c - 1.0);
  const dim3 net(rr::kNetThreads);
  float *D = t->node, *q = D + 3 * n, *res = q + 3 * n, *gE = res + 2 * n;
  if (feedback)
    hipLaunchKernelGGL(rr::k_net_forward<true>, dim3(nf), net, 0, t->st, params, norm, x, (int)n,
                       tm1, q, D);
  else
    hipLaunchKernelGGL(rr::k_net_forward<false>, dim3(nf), net, 0, t->st, params, norm, x, (int)n,
                       tm1, q, D);
  THIP(hipGetLastError());
  hipLaunchKernelGGL(rr::k_onestep_fwd, dim3(nb), dim3(rr::kTB), 0, t->st, x, r0, nsnap, nc, om1,
                     (const float *)D, res, t->loss_part);
  THIP(hipGetLastError());
  hipLaunchKernelGGL(rr::k_onestep_adj, dim3(nb), dim3(rr::kTB), 0, t->st, x, nsnap, nc, om1,
                     (float)(2.0 / den), (const float *)res, gE);
  THIP(hipGetLastError());
  if (feedback)
    hipLaunchKernelGGL(rr::k_net_grad<rr::NET_FEEDBACK>, dim3(ng), net, 0, t->st, params, norm, x,
                       (const float *)nullptr, (const float *)q, (const float *)gE, (int)n, tm1,
                       t->part, (float *)nullptr);
  else
    hipLaunchKernelGGL(rr::k_net_grad<rr::NET_ONESTEP>, dim3(ng), net, 0, t->st, params, norm, x,
                       (const float *)nullptr, (const float *)nullptr, (const float *)gE, (int)n,
                       tm1, t->part, (float *)nullptr);
  THIP(hipGetLastError());
  return net_final(t, ng, nb, 1.0 / den, grad, loss);
}

int rrmhd_train_adam(rrmhd_trainer *t, float *params, float *m, float *v, const float *grad,
                     float lr, float beta1, float beta2, float eps, int step) {
  if (!t || !params || !m || !v || !grad || step < 1) return RRMHD_EINVAL;
  const float c1 = (float)(1.0 - std::pow((double)beta1, step));
  const float c2 = (float)(1.0 - std::pow((double)beta2, step));
  hipLaunchKernelGGL(rr::k_adam, dim3((rr::kNParam + 255) / 256), dim3(256), 0, t->st, params, m,
                     v, grad, rr::kNParam, lr, beta1, beta2, eps, c1, c2);
  THIP(hipGetLastError());
  return RRMHD_OK;
}

int rrmhd_train_samples(const double *rho, const double *u, const double *b, int nf,
                        int factor, double tau_c, double *work, float *x, float *target,
                        void *hip_stream) {
  if (!rho || !u || !b || !work || !x || !target || factor < 1 || nf < factor ||
      nf % factor != 0 || !(tau_c > 0.5))
    return RRMHD_EINVAL;
  const hipStream_t st = (hipStream_t)hip_stream;
  const int nc = nf / factor;
  const int64_t Nc = (int64_t)nc * nc;
  const int blocks = (int)((Nc + 255) / 256);
  rr::launch_box_filter(rho, u, b, nf, factor, work, st);
  THIP(hipGetLastError());
  hipLaunchKernelGGL(rr::k_samples, dim3(blocks), dim3(256), 0, st, work, nc, tau_c, x, target);
  THIP(hipGetLastError());
  return RRMHD_OK;
}

int rrmhd_train_box_filter(const double *rho, const double *u, const double *b, int nf,
                           int factor, double *out, void *hip_stream) {
  if (!rho || !u || !b || !out || factor < 1 || nf < factor || nf % factor != 0)
    return RRMHD_EINVAL;
  rr::launch_box_filter(rho, u, b, nf, factor, out, (hipStream_t)hip_stream);
  THIP(hipGetLastError());
  return RRMHD_OK;
}

int rrmhd_train_onestep_samples(const double *rho0, const double *u0, const double *b0,
                                const double *rho1, const double *u1, const double *b1,
                                int nf, int factor, double tau_c, double *work, float *x,
                                float *r0, double *den, void *hip_stream) {
  if (!rho0 || !u0 || !b0 || !rho1 || !u1 || !b1 || !work || !x || !r0 || !den ||
      factor < 1 || nf < factor || nf % factor != 0 || !(tau_c > 0.5))
    return RRMHD_EINVAL;
  const hipStream_t st = (hipStream_t)hip_stream;
  const int nc = nf / factor;
  const int64_t Nc = (int64_t)nc * nc;
  const int blocks = (int)((Nc + 255) / 256);
  // work: filtered fields at t [10][Nc] and t + factor [10][Nc], FP64
  // features [8][Nc], per-workgroup sums of |j_bar(t + factor) - j_bar(t)|^2 [<= Nc]: 29 Nc
  double *flt0 = work, *flt1 = work + rr::kFilt * Nc, *feat = work + 2 * rr::kFilt * Nc;
  double *dm = feat + 8 * Nc;
  rr::launch_box_filter(rho0, u0, b0, nf, factor, flt0, st);
  THIP(hipGetLastError());
  rr::launch_box_filter(rho1, u1, b1, nf, factor, flt1, st);
  THIP(hipGetLastError());
  hipLaunchKernelGGL(rr::k_features64, dim3(blocks), dim3(256), 0, st, (const double *)flt0, nc,
                     tau_c, feat);
  THIP(hipGetLastError());
  hipLaunchKernelGGL(rr::k_onestep_prep, dim3(blocks), dim3(256), 0, st, (const double *)flt0,
                     (const double *)flt1, (const double *)feat, nc, 1.0 / tau_c, x, r0, dm);
  THIP(hipGetLastError());
  hipLaunchKernelGGL(rr::k_sum64, dim3(1), dim3(256), 0, st, (const double *)dm,
                     (int64_t)blocks, den);
  THIP(hipGetLastError());
  return RRMHD_OK;
}

const char *rrmhd_train_last_error_detail(void) { return g_tdetail; }

}  // extern "C"
