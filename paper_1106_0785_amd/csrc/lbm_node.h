// Per-node arithmetic of the D2V16 MRT finite-difference lattice Boltzmann
// step (Sec. II): moment transform f^ = M f, equilibria f^eq, and the
// back-transform M^-1, in the shell-factorised form generated into
// lbm_consts.h. Host and device; no memory access, no state.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "lbm_consts.h"

namespace lbm {

#define LBM_HD __host__ __device__ __forceinline__

// a b + c with one rounding. Sums of two products are written with it: left
// to contraction, which product is rounded depends on the kernel the code is
// inlined in, and the step kernels' results would agree to rounding only.
LBM_HD double mad(double a, double b, double c) { return fma(a, b, c); }

// Shell quantities (sigma, gx, gy, q) of the four shells of f (see lbm_consts.h).
template <class S>
LBM_HD void shell_quantities(const S* f, S* sig, S* gx, S* gy, S* q) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const S a = f[4 * s + 0], b = f[4 * s + 1], c = f[4 * s + 2], d = f[4 * s + 3];
    const S P = a + c, Q = b + d;
    sig[s] = P + Q;
    q[s] = P - Q;
    if (s == 0 || s == 2) {  // axis shell E, N, W, S
      gx[s] = a - c;
      gy[s] = b - d;
    } else {  // diagonal shell NE, NW, SW, SE
      const S R = a - c, W = b - d;
      gx[s] = R - W;
      gy[s] = R + W;
    }
  }
}

// All 16 moments f^_k = sum_i M_ki f_i (k = 1..16 stored at index k-1).
LBM_HD void moments_from_f(const double* f, double* m) {
  double sig[4], gx[4], gy[4], q[4];
  shell_quantities(f, sig, gx, gy, q);
  const int ks[4] = {0, 3, 10, 11};
  const int kx[4] = {1, 6, 8, 14};
  const int ky[4] = {2, 7, 9, 15};
  // the conserved ones summed as in density_momentum, so that a node's own
  // velocity and the one its neighbours see agree bit by bit
  m[0] = (sig[0] + sig[1]) + (sig[2] + sig[3]);
  m[1] = mad(2.0, gx[2] + gx[3], gx[0] + gx[1]);
  m[2] = mad(2.0, gy[2] + gy[3], gy[0] + gy[1]);
#pragma unroll
  for (int r = 1; r < 4; ++r) {
    // (sums start from their first term: adding to a zero is an operation)
    double a = A_SIG[r][0] * sig[0], b = A_GX[r][0] * gx[0], c = A_GY[r][0] * gy[0];
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      a = mad(A_SIG[r][s], sig[s], a);
      b = mad(A_GX[r][s], gx[s], b);
      c = mad(A_GY[r][s], gy[s], c);
    }
    m[ks[r]] = a;
    m[kx[r]] = b;
    m[ky[r]] = c;
  }
  m[4] = mad(A_QA[0][1], q[2], A_QA[0][0] * q[0]);
  m[12] = mad(A_QA[1][1], q[2], A_QA[1][0] * q[0]);
  m[5] = mad(A_QD[0][1], q[3], A_QD[0][0] * q[1]);
  m[13] = mad(A_QD[1][1], q[3], A_QD[1][0] * q[1]);
}

// rho, j_x, j_y only (the velocity of a neighbour node).
LBM_HD void density_momentum(const double* f, double& rho, double& jx, double& jy) {
  double sig[4], gx[4], gy[4], q[4];
  shell_quantities(f, sig, gx, gy, q);
  rho = (sig[0] + sig[1]) + (sig[2] + sig[3]);
  jx = mad(2.0, gx[2] + gx[3], gx[0] + gx[1]);
  jy = mad(2.0, gy[2] + gy[3], gy[0] + gy[1]);
}

// f = M^-1 m for a full moment vector m (index k-1 holds moment k). The
// weights 1/4 and 1/2 of a shell's reconstruction are folded into the block
// coefficients (powers of two: the same values, 16 operations fewer).
// CONSERVED false: moments 1..4 are zero and not read.
template <bool CONSERVED>
LBM_HD void reconstruct(const double* m, double* f) {
  const int ks[4] = {0, 3, 10, 11};
  const int kx[4] = {1, 6, 8, 14};
  const int ky[4] = {2, 7, 9, 15};
  constexpr int s0 = CONSERVED ? 0 : 2, g0 = CONSERVED ? 0 : 1;  // first moment of each family
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const double wg = (s == 0 || s == 2) ? 0.5 : 0.25;
    double h = (0.25 * AINV_SIG[s][s0]) * m[ks[s0]];
    double X = (wg * AINV_GX[s][g0]) * m[kx[g0]], Y = (wg * AINV_GY[s][g0]) * m[ky[g0]];
#pragma unroll
    for (int r = s0 + 1; r < 4; ++r) h = mad(0.25 * AINV_SIG[s][r], m[ks[r]], h);
#pragma unroll
    for (int r = g0 + 1; r < 4; ++r) {
      X = mad(wg * AINV_GX[s][r], m[kx[r]], X);
      Y = mad(wg * AINV_GY[s][r], m[ky[r]], Y);
    }
    double q;
    if (s == 0 || s == 2)
      q = mad(0.25 * AINV_QA[s / 2][1], m[12], (0.25 * AINV_QA[s / 2][0]) * m[4]);
    else
      q = mad(0.25 * AINV_QD[s / 2][1], m[13], (0.25 * AINV_QD[s / 2][0]) * m[5]);
    const double hp = h + q, hm = h - q;
    if (s == 0 || s == 2) {  // E, N, W, S
      f[4 * s + 0] = hp + X;
      f[4 * s + 1] = hm + Y;
      f[4 * s + 2] = hp - X;
      f[4 * s + 3] = hm - Y;
    } else {  // NE, NW, SW, SE
      const double U = X + Y, V = X - Y;
      f[4 * s + 0] = hp + U;
      f[4 * s + 1] = hm - V;
      f[4 * s + 2] = hp - U;
      f[4 * s + 3] = hm + V;
    }
  }
}

LBM_HD void f_from_moments(const double* m, double* f) { reconstruct<true>(m, f); }

// Transposed transforms, used by the adjoint.
//
// M^T nu: the transpose of moments_from_f. The block coefficients act on
// nu first (A^T), then each shell's four values are spread back to its
// points with the sign patterns of the shell quantities (S^T).
LBM_HD void mt_apply(const double* nu, double* out) {
  const int ks[4] = {0, 3, 10, 11};
  const int kx[4] = {1, 6, 8, 14};
  const int ky[4] = {2, 7, 9, 15};
  double sig[4], gx[4], gy[4], q[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    double a = A_SIG[0][s] * nu[ks[0]], b = A_GX[0][s] * nu[kx[0]], c = A_GY[0][s] * nu[ky[0]];
#pragma unroll
    for (int r = 1; r < 4; ++r) {
      a += A_SIG[r][s] * nu[ks[r]];
      b += A_GX[r][s] * nu[kx[r]];
      c += A_GY[r][s] * nu[ky[r]];
    }
    sig[s] = a;
    gx[s] = b;
    gy[s] = c;
  }
  q[0] = A_QA[0][0] * nu[4] + A_QA[1][0] * nu[12];
  q[2] = A_QA[0][1] * nu[4] + A_QA[1][1] * nu[12];
  q[1] = A_QD[0][0] * nu[5] + A_QD[1][0] * nu[13];
  q[3] = A_QD[0][1] * nu[5] + A_QD[1][1] * nu[13];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s == 0 || s == 2) {  // E, N, W, S
      out[4 * s + 0] = (sig[s] + q[s]) + gx[s];
      out[4 * s + 1] = (sig[s] - q[s]) + gy[s];
      out[4 * s + 2] = (sig[s] + q[s]) - gx[s];
      out[4 * s + 3] = (sig[s] - q[s]) - gy[s];
    } else {  // NE, NW, SW, SE
      out[4 * s + 0] = (sig[s] + q[s]) + (gx[s] + gy[s]);
      out[4 * s + 1] = (sig[s] - q[s]) - (gx[s] - gy[s]);
      out[4 * s + 2] = (sig[s] + q[s]) - (gx[s] + gy[s]);
      out[4 * s + 3] = (sig[s] - q[s]) + (gx[s] - gy[s]);
    }
  }
}

// M^-T lambda: the transpose of f_from_moments. The per-shell
// reconstruction is transposed first (shell quantities of lambda with the
// reconstruction's 1/4 and 1/2 weights), then the inverse blocks.
LBM_HD void minvt_apply(const double* lam, double* mu) {
  double sig[4], gx[4], gy[4], q[4];
  shell_quantities(lam, sig, gx, gy, q);
  // (the weights are folded into the block coefficients, as in reconstruct)
  const int ks[4] = {0, 3, 10, 11};
  const int kx[4] = {1, 6, 8, 14};
  const int ky[4] = {2, 7, 9, 15};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double a = (0.25 * AINV_SIG[0][r]) * sig[0], b = (0.5 * AINV_GX[0][r]) * gx[0], c = (0.5 * AINV_GY[0][r]) * gy[0];
#pragma unroll
    for (int s = 1; s < 4; ++s) {
      const double wg = s == 2 ? 0.5 : 0.25;
      a += (0.25 * AINV_SIG[s][r]) * sig[s];
      b += (wg * AINV_GX[s][r]) * gx[s];
      c += (wg * AINV_GY[s][r]) * gy[s];
    }
    mu[ks[r]] = a;
    mu[kx[r]] = b;
    mu[ky[r]] = c;
  }
  // inverse quadrupole blocks: q of shells 0, 2 from m5, m13; of shells 1, 3 from m6, m14
  mu[4] = (0.25 * AINV_QA[0][0]) * q[0] + (0.25 * AINV_QA[1][0]) * q[2];
  mu[12] = (0.25 * AINV_QA[0][1]) * q[0] + (0.25 * AINV_QA[1][1]) * q[2];
  mu[5] = (0.25 * AINV_QD[0][0]) * q[1] + (0.25 * AINV_QD[1][0]) * q[3];
  mu[13] = (0.25 * AINV_QD[0][1]) * q[1] + (0.25 * AINV_QD[1][1]) * q[3];
}

// Velocity-space image of a moment vector with only the non-conserved
// components k = 5..16 set: f = M^-1 (0, 0, 0, 0, c_5, ..., c_16).
LBM_HD void f_from_nonconserved(const double* c, double* f) { reconstruct<false>(c, f); }

// 1 / x. On the device the hardware estimate and two Newton steps in fused
// multiply-adds: the last step's residual is exact to the rounding of the
// estimate's error, so the result is the correctly rounded one but for near
// ties, like the division's, at 5 instead of 11 instructions. Of 200 000
// random x in each of 2^-1024..2^-1022, 2^-1022..2^-1000, 2^-60..2^60,
// 2^1000..2^1022 and 2^1022..2^1024 none differs from the division in a bit.
// Where 1 / x overflows (x below 2^-1024, zero) and for an infinite x it is NaN
// where the division gives infinity or zero; the step that meets such a density
// reports it either way.
LBM_HD double recip(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
#else
  return 1.0 / x;
#endif
}

LBM_HD double sexp(double x) { return ::exp(x); }

// Free equilibrium moments 12, 15, 16 of versions 2 (the printed
// polynomials) and 3 (moments of the Maxwellian sampled at the velocities).
template <int VER, class S>
LBM_HD void free_moments(S rho, S ux, S uy, S jx, S jy, S T, S* q) {
  if constexpr (VER == 2) {
    const S d = 5.0 * ux * ux - 5.0 * uy * uy;
    q[11] = 0.0;
    q[14] = jx * (-4.0 + 10.0 * T + d);
    q[15] = jy * (4.0 - 10.0 * T + d);
  } else {
    S fm[16];
    const S pre = rho / (2.0 * M_PI * T), i2T = 0.5 / T;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const S cx = (double)VX[i] - ux, cy = (double)VY[i] - uy;
      fm[i] = pre * sexp(-(cx * cx + cy * cy) * i2T);
    }
    S sig[4], gx[4], gy[4], qq[4];
    shell_quantities(fm, sig, gx, gy, qq);
    S a = 0.0, b = 0.0, c = 0.0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      a += A_SIG[3][s] * sig[s];
      b += A_GX[3][s] * gx[s];
      c += A_GY[3][s] * gy[s];
    }
    q[11] = a;
    q[14] = b;
    q[15] = c;
  }
}

// Equilibrium moments, Eqs. (14a)-(14i); moments 1..4 are the conserved ones;
// free moments 12, 15, 16 by version VER (1: zero; 2: printed polynomials;
// 3: moments of the Maxwellian sampled at the velocities). S is double, or a
// dual number when the adjoint differentiates this very code.
// `ir` is 1 / rho. With a = j_x u_x, b = j_y u_y, k = a + b = rho u^2 the
// polynomials need 24 products: rho T = e - k/2, q_7, q_8 = (e + rho T) u,
// q_9 = (a - 3b) u_x, q_10 = (3a - b) u_y, q_11 = (2 e^2 - k^2/4) / rho,
// (q_13, q_14) = (6e - 2k) (a - b, j_x u_y) / rho.
template <int VER, class S>
LBM_HD void equilibrium_moments(S rho, S ir, S jx, S jy, S e, S* q) {
  const S ux = jx * ir, uy = jy * ir;
  const S a = jx * ux, b = jy * uy, k = mad(jx, ux, b);
  const S d5 = mad(jx, ux, -b), d6 = jx * uy;
  q[0] = rho;
  q[1] = jx;
  q[2] = jy;
  q[3] = e;
  q[4] = d5;
  q[5] = d6;
  const S h = e + (e - 0.5 * k);  // e + rho R T, R = 1
  q[6] = h * ux;
  q[7] = h * uy;
  q[8] = mad(S(-3.0), b, a) * ux;
  q[9] = mad(S(3.0), a, -b) * uy;
  q[10] = mad(-0.25 * k, k, 2.0 * e * e) * ir;
  const S w = mad(S(-2.0), k, 6.0 * e) * ir;
  q[12] = w * d5;
  q[13] = w * d6;
  if constexpr (VER != 1) {
    const S T = (e - 0.5 * k) * ir;
    free_moments<VER, S>(rho, ux, uy, jx, jy, T, q);
  } else {
    q[11] = 0.0;
    q[14] = 0.0;
    q[15] = 0.0;
  }
}

template <int VER, class S>
LBM_HD void equilibrium_moments(S rho, S jx, S jy, S e, S* q) {
  const S ir = 1.0 / rho;
  equilibrium_moments<VER, S>(rho, ir, jx, jy, e, q);
}

// Equilibrium distribution f^eq = M^-1 f^eq(rho, u, T).
template <int VER>
LBM_HD void equilibrium_f(double rho, double ux, double uy, double T, double* f) {
  double q[16];
  const double jx = rho * ux, jy = rho * uy;
  const double e = rho * (T + 0.5 * (ux * ux + uy * uy));
  equilibrium_moments<VER, double>(rho, jx, jy, e, q);
  f_from_moments(q, f);
}

// Runtime-version form for set-up code.
LBM_HD void equilibrium_f(int version, double rho, double ux, double uy, double T, double* f) {
  if (version == 2)
    equilibrium_f<2>(rho, ux, uy, T, f);
  else if (version == 3)
    equilibrium_f<3>(rho, ux, uy, T, f);
  else
    equilibrium_f<1>(rho, ux, uy, T, f);
}

}  // namespace lbm
