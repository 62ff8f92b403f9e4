// Adjoint (reverse-mode) step of the MRT FD-LBM update, hand-written.
//
// One forward step is f^{n+1}(x) = f(x) + L(x) + M^-1 col(x), with the
// per-axis Lax-Wendroff increments L, col_k = -dt s_k (m_k - q_k(c)) for the
// non-conserved moments (c = rho, j_x, j_y, e) and the energy-flux
// modification g_7, g_8 added to col_7, col_8 (Sec. II); g depends on the
// node's c and on the central-difference velocity gradients A, B built from
// the four neighbours' velocities. Its amplification matrix G_ij (Sec. III)
// is this map's Jacobian in Fourier space. Given lambda = dL/df^{n+1}, the
// adjoint step returns dL/df^n:
//
//   lambda^n_i(x) = lambda_i(x) + sum_axes [ p_i (lambda_i(x-e) - lambda_i(x))
//                                          + m_i (lambda_i(x+e) - lambda_i(x)) ]
//                 + (M^T nu)_i + (M_{1..4}^T g_c)_i
//   mu  = M^-T lambda(x),   nu_k = -dt s_k mu_k  (k >= 5)
//   g_c = - J_q^T nu + mu_7 dg_7/dc + mu_8 dg_8/dc + (du/dc)^T g_u
//   g_u(x) = gathered from the neighbours' dL/dA, dL/dB (the modification's
//            coupling to the velocities of the four neighbours)
//
// and accumulates dL/ds_k = sum_n sum_x mu_k d col_k/d s_k. Ghost layers
// are transposed: a periodic ghost is the wrapped node, a mirror ghost
// returns the mirrored lambda and (dL/dA, -dL/dB), a zero-gradient ghost
// returns lambda with the Lax-Wendroff weights swapped and (-dL/dA, -dL/dB),
// a fixed-state ghost returns nothing.
#pragma once

#include "lbm_dual.h"
#include "lbm_kernels.h"

namespace lbm {

// Derivatives of the modification coefficients (Hot::cmod) w.r.t. the rates:
// d cm0/d s5, d cm0/d s7, d cm1/d s6, d cm1/d s7, d cm2/d s6, d cm2/d s8,
// d cm3/d s5, d cm3/d s8 (all 0 for the unmodified model).
struct AdjCoef {
  double dcm[8];
  double mdt;  // -dt: d col_k / d s_k = -dt (m_k - q_k)
};

// Per-node record written by the first pass: dL/dA, dL/dB and the velocity.
enum { REC_GA = 0, REC_GB = 1, REC_UX = 2, REC_UY = 3, NREC = 4 };

// Record of a node from its distributions f (the forward level the next
// adjoint step linearises about) and its lambda (that step's input).
LBM_HD void record_from(const Hot& c, const double* f, const double* l, double* r) {
  double m[16], mu[16];
  moments_from_f(f, m);
  minvt_apply(l, mu);
  const double ir = recip(m[0]);
  const double ux = m[1] * ir, uy = m[2] * ir;
  const double rT = m[3] - 0.5 * (m[1] * ux + m[2] * uy);  // rho T
  r[REC_GA] = mu[6] * c.cmod[0] * rT * ux + mu[7] * c.cmod[3] * rT * uy;
  r[REC_GB] = mu[6] * c.cmod[1] * rT * uy + mu[7] * c.cmod[2] * rT * ux;
  r[REC_UX] = ux;
  r[REC_UY] = uy;
}

LBM_HD void adj_record(const Field& F, const Hot& c, const double* __restrict__ lam, double* __restrict__ rec, int x,
                       int y) {
  const long long k = (long long)y * F.pitch + x;
  double f[16], l[16], r[NREC];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    f[i] = F.fin[k + i * F.plane];
    l[i] = lam[k + i * F.plane];
  }
  record_from(c, f, l, r);
#pragma unroll
  for (int j = 0; j < NREC; ++j) rec[k + j * F.plane] = r[j];
}

template <int VER>
__global__ __launch_bounds__(256) void k_adj_records(Field F, const double* __restrict__ lam,
                                                     double* __restrict__ rec, const Hot* __restrict__ hot) {
  __shared__ Hot hs;
  stage_hot(hot, &hs);
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  if (x >= F.nx || y >= F.ny) return;
  adj_record(F, hs, lam, rec, x, y);
}

// Record of stencil point (x + ox, y + oy) of node (x, y) as its ghost
// transposition requires; ux, uy are the velocity the forward step used.
template <class C>
LBM_HD void rec_point(const Field& F, const C& c, const Cold* __restrict__ cold,
                                          const double* __restrict__ rec, int x, int y, int ox, int oy, double& GA,
                                          double& GB, double& ux, double& uy) {
  const int xn = x + ox, yn = y + oy;
  const Src sx = resolve(xn, F.nx, c.bc[0], c.bc[1], 0);
  const Src sy = resolve(yn, F.ny, c.bc[2], c.bc[3], 2);
  // kind of ghost this stencil point is (periodic: a stored node, perhaps
  // after wrapping) and its side; selects only, as in resolve()
  const bool xg = xn < 0 || xn >= F.nx;
  const int kind = xg ? sx.kind : sy.kind, side = xg ? sx.side : sy.side;
  const bool fixed = kind == BC_DIRICHLET_EQ, mirror = kind == BC_SPECULAR, zero = kind == BC_ZERO_GRADIENT;
  const long long k = (long long)sy.idx * F.pitch + sx.idx;
  const double ga = rec[k + REC_GA * F.plane], gb = rec[k + REC_GB * F.plane];
  const double vx = rec[k + REC_UX * F.plane], vy = rec[k + REC_UY * F.plane];
  const double* gv = cold->gvel[max(side, 0)];
  const double gx = gv[0], gy = gv[1];
  GA = fixed ? 0.0 : zero ? -ga : ga;
  GB = fixed ? 0.0 : (zero || mirror) ? -gb : gb;
  ux = fixed ? gx : (mirror && side < 2) ? -vx : vx;
  uy = fixed ? gy : (mirror && side >= 2) ? -vy : vy;
}

// Lambda at a neighbour along one axis as the transposed convection takes it:
// the stored node's address, the distance between a plane and the one it is
// taken from in units of MIRROR[I] - I (the plane distance at a mirror ghost,
// else 0), and whether it is a fixed-state ghost, which returns nothing. (A
// zero-gradient ghost gives the node's own lambda and the caller corrects the
// weights.)
struct LamSrc {
  const double* at;
  long long d;
  bool none;
};

template <class C>
LBM_HD LamSrc lam_src(const Field& F, const C& c, const double* __restrict__ lam, int x, int y, int ox, int oy) {
  const Src sx = resolve(x + ox, F.nx, c.bc[0], c.bc[1], 0);
  const Src sy = resolve(y + oy, F.ny, c.bc[2], c.bc[3], 2);
  LamSrc r;
  r.at = lam + ((long long)sy.idx * F.pitch + sx.idx);
  r.d = (sx.mode == 1 || sy.mode == 1) ? F.plane : 0;
  r.none = sx.mode == 2 || sy.mode == 2;
  return r;
}

// The planes that move along the axis (0: x, 1: y) from the neighbour s.
template <int AXIS, int I = 0>
LBM_HD void lam_planes(const Field& F, const LamSrc& s, double* l) {
  if constexpr ((AXIS == 0 ? VX[I] : VY[I]) != 0) {
    constexpr int k = (AXIS == 0 ? MIRROR_X[I] : MIRROR_Y[I]) - I;
    const double v = (s.at + k * s.d)[I * F.plane];
    l[I] = s.none ? 0.0 : v;
  }
  if constexpr (I < 15) lam_planes<AXIS, I + 1>(F, s, l);
}

// Transposed Lax-Wendroff increment of velocity component V along one axis,
// added to r; lc as in Hot::lx, of which the forward step applies p to
// (f(x+e) - f) and m to (f(x-e) - f). The node is the + neighbour of x-e
// (weight p) and the - neighbour of x+e (weight m). cz corrects for
// zero-gradient ghosts, which the node itself stands for: (m - p) of speeds 1
// and 2 where the low neighbour is one, (p - m) where the high one is, else 0.
template <int V>
LBM_HD double conv_t_axis(double r, const double* lc, const double* cz, double lo, double hi, double lam) {
  constexpr int a = V < 0 ? -V : V, p = 2 * (a - 1) + (V > 0 ? 0 : 1), m = 2 * (a - 1) + (V > 0 ? 1 : 0);
  r = mad(lc[p], lo - lam, r);
  r = mad(lc[m], hi - lam, r);
  return mad(V > 0 ? cz[a - 1] : -cz[a - 1], lam, r);
}

// cz of one axis (zl, zh: the node's low / high neighbour is a zero-gradient
// ghost).
LBM_HD void zero_gradient_t(const double* lc, bool zl, bool zh, double* cz) {
  const double s = (zl ? 1.0 : 0.0) - (zh ? 1.0 : 0.0);
  cz[0] = s * (lc[1] - lc[0]);
  cz[1] = s * (lc[3] - lc[2]);
}

// Transposed convection of all velocities along one axis, added to out, from
// lambda at the node (l) and at its two neighbours.
template <int AXIS, int I = 0>
LBM_HD void convect_t(const Hot& c, const double* cz, const double* l, const double* hi, const double* lo,
                      double* out) {
  constexpr int v = AXIS == 0 ? VX[I] : VY[I];
  if constexpr (v != 0) out[I] = conv_t_axis<v>(out[I], AXIS == 0 ? c.lx : c.ly, cz, lo[I], hi[I], l[I]);
  if constexpr (I < 15) convect_t<AXIS, I + 1>(c, cz, l, hi, lo, out);
}

// Adjoint of the collision at one node: from the moments m, the velocity
// gradients A and B, mu = M^-T lambda and the neighbours' velocity terms
// (gux, guy), the 16 moments nu whose M^T is the collision's part of the new
// lambda: nu_k = -dt s_k mu_k for k >= 5 and, in the first four, dL/d(rho,
// j_x, j_y, e) of the equilibria, the modification and the velocity. Adds the
// node's dL/ds_5..16 to sg. The derivatives of the equilibria are taken in
// reverse, one sweep over the forward intermediates (about 60 operations;
// four forward-mode sweeps, one per conserved moment, took about 300).
template <int VER>
LBM_HD void collision_adjoint(const Hot& c, const AdjCoef* __restrict__ adj, const double* m, double A, double B,
                              const double* mu, double gux, double guy, double* nu, double* sg) {
  const double rho = m[0], jx = m[1], jy = m[2], e = m[3], ir = recip(rho);
  const double ux = jx * ir, uy = jy * ir;
  double q[16];
  equilibrium_moments<VER, double>(rho, ir, jx, jy, e, q);
  const double a = jx * ux, b = jy * uy, k = a + b;
  const double rT = e - 0.5 * k;
  // dL/ds: d col_k/d s_k = -dt (m_k - q_k), plus the modification's
  // coefficients (their s-derivatives already carry the factor dt)
#pragma unroll
  for (int i = 4; i < 16; ++i) sg[i - 4] += mu[i] * adj->mdt * (m[i] - q[i]);
  const double tx = rT * ux, ty = rT * uy;
  const double a7 = tx * A, b7 = ty * B, b8 = tx * B, a8 = ty * A;
  sg[0] += mu[6] * adj->dcm[0] * a7 + mu[7] * adj->dcm[6] * a8;  // s5
  sg[1] += mu[6] * adj->dcm[2] * b7 + mu[7] * adj->dcm[4] * b8;  // s6
  sg[2] += mu[6] * (adj->dcm[1] * a7 + adj->dcm[3] * b7);        // s7
  sg[3] += mu[7] * (adj->dcm[5] * b8 + adj->dcm[7] * a8);        // s8
  double n[16];  // dL/dq_k = -nu_k
#pragma unroll
  for (int i = 4; i < 16; ++i) {
    nu[i] = c.cq[i - 4] * mu[i];
    n[i] = -nu[i];
  }
  // the intermediates of equilibrium_moments in reverse (g*: dL/d*)
  const double ctx = mu[6] * c.cmod[0] * A + mu[7] * c.cmod[2] * B;  // dL/d(rho T u_x)
  const double cty = mu[6] * c.cmod[1] * B + mu[7] * c.cmod[3] * A;
  const double W = 6.0 * e - 2.0 * k;
  const double gw = n[12] * q[4] + n[13] * q[5], gW = gw * ir;
  const double gE = n[10] * ir;
  double gir = n[10] * (2.0 * e * e - 0.25 * k * k) + gw * W;
  const double g5 = n[4] + n[12] * (W * ir), g6 = n[5] + n[13] * (W * ir);
  const double gh = n[6] * ux + n[7] * uy, h = e + rT;
  const double h8 = n[8] * ux, h9 = n[9] * uy;
  double gvx = gux + n[6] * h + n[8] * (a - 3.0 * b) + ctx * rT;
  double gvy = guy + n[7] * h + n[9] * (3.0 * a - b) + cty * rT;
  double grT = ctx * ux + cty * uy, grho = 0.0, gjx = 0.0, gjy = 0.0;
  if constexpr (VER == 2) {
    const double T = rT * ir, d = 5.0 * ux * ux - 5.0 * uy * uy;
    gjx = n[14] * (-4.0 + 10.0 * T + d);
    gjy = n[15] * (4.0 - 10.0 * T + d);
    const double p = n[14] * jx, r = n[15] * jy;
    const double gT = 10.0 * (p - r), gd = 10.0 * (p + r);
    gvx += gd * ux;
    gvy -= gd * uy;
    grT += gT * ir;
    gir += gT * rT;
  } else if constexpr (VER == 3) {
    // Maxwellian values fm_i weighted by M^T of the three moments taken of
    // them: d fm / fm = drho/rho + c.du/T + (|c|^2/(2 T) - 1) dT/T, c = v - u
    const double T = rT * ir, iT = 1.0 / T, pre = rho / (2.0 * M_PI * T), i2T = 0.5 / T;
    double G0 = 0.0, Gx = 0.0, Gy = 0.0, G2 = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int s = i / 4, p = i % 4;
      const double sg3 = A_SIG[3][s] * n[11], gx3 = A_GX[3][s] * n[14], gy3 = A_GY[3][s] * n[15];
      double w;
      if (s == 0 || s == 2)
        w = p == 0 ? sg3 + gx3 : p == 1 ? sg3 + gy3 : p == 2 ? sg3 - gx3 : sg3 - gy3;
      else
        w = p == 0 ? sg3 + (gx3 + gy3) : p == 1 ? sg3 - (gx3 - gy3) : p == 2 ? sg3 - (gx3 + gy3) : sg3 + (gx3 - gy3);
      const double cx = (double)VX[i] - ux, cy = (double)VY[i] - uy, c2 = cx * cx + cy * cy;
      const double v = w * (pre * sexp(-c2 * i2T));
      G0 += v;
      Gx += v * cx;
      Gy += v * cy;
      G2 += v * c2;
    }
    gvx += Gx * iT;
    gvy += Gy * iT;
    grho = G0 * ir;
    const double gT = (G2 * i2T - G0) * iT;
    grT += gT * ir;
    gir += gT * rT;
  }
  const double gk = -0.5 * (gh + grT) - 2.0 * gW - 0.5 * k * gE;
  const double ga = gk + g5 + h8 + 3.0 * h9, gb = gk - g5 - 3.0 * h8 - h9;
  gvx += ga * jx;
  gvy += gb * jy + g6 * jx;
  gir += gvx * jx + gvy * jy;
  nu[0] = grho - (gir * ir) * ir;
  nu[1] = gjx + ga * ux + g6 * uy + gvx * ir;
  nu[2] = gjy + gb * uy + gvy * ir;
  nu[3] = 2.0 * gh + grT + 6.0 * gW + 4.0 * e * gE;
}

// Value of lane l (uniform) of a wave.
__device__ __forceinline__ double read_lane(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Sum over the 64 lanes of a wave in a fixed order (rows of 16 by DPP, then
// the four row sums), so the result does not depend on timing.
__device__ __forceinline__ double wave_sum(double v) {
  v = row16_sum(v);
  return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// New adjoint lambda^n of every node into lam_out, and the step's dL/ds_5..16
// (index k - 5), one partial sum per block. With f_prev (the forward level of
// the next adjoint step, same layout as F.fin) also writes that step's
// records into rec_out. Launched with 64 x 4 threads per block.
//
// Bound by the latency of ~110 loads per node where a SIMD has one wave
// (grids of up to 1024 waves), so they are issued as early as their addresses
// are known: the node's own before the constants arrive, the neighbours'
// before the collision, f_prev's without a branch, and all of them before the
// first store (a wait for a later load would also wait for the stores before
// it). WIDE (grids of more than 2048 blocks, versions 1 and 2): two blocks per
// CU, whose waves hide each other's latency; the neighbours' planes are then
// loaded after the collision, which keeps its registers free. 11.9-12.2 us at 512 x 128 (12.9 with each plane's loads
// behind the previous plane's store, 12.6 with four forward-mode sweeps of
// the collision).
template <int VER, bool WIDE>
__global__ __launch_bounds__(256, WIDE ? 2 : 1) void k_adj_step(Field F, const double* __restrict__ lam_in,
                                                  double* __restrict__ lam_out, const double* __restrict__ rec,
                                                  const Hot* __restrict__ hot, const Cold* __restrict__ cold,
                                                  const AdjCoef* __restrict__ adj, double* __restrict__ partials,
                                                  const double* __restrict__ f_prev, double* __restrict__ rec_out) {
  __shared__ Hot hs;
  __shared__ double red[12][4];
  const int t = threadIdx.y * blockDim.x + threadIdx.x;
  const int xt = blockIdx.x * blockDim.x + threadIdx.x, yt = blockIdx.y * blockDim.y + threadIdx.y;
  const bool inside = xt < F.nx && yt < F.ny;
  const int x = min(xt, F.nx - 1), y = min(yt, F.ny - 1);  // threads outside repeat an edge node
  const long long k0 = (long long)y * F.pitch + x;
  double f[16], l[16], fp[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) f[i] = F.fin[k0 + i * F.plane];
#pragma unroll
  for (int i = 0; i < 16; ++i) l[i] = lam_in[k0 + i * F.plane];
  const double* fpp = f_prev ? f_prev : F.fin;
  auto load_prev = [&]() {
#pragma unroll
    for (int i = 0; i < 16; ++i) fp[i] = fpp[k0 + i * F.plane];
  };
  if (!WIDE) load_prev();
  // the block's running sum, added to at the end
  const long long slot = (long long)blockIdx.y * gridDim.x + blockIdx.x;
  const double psum = t < 12 ? partials[slot * 12 + t] : 0.0;
  // the neighbours' addresses need the boundary kinds only, by scalar loads
  struct {
    int bc[4];
  } side;
#pragma unroll
  for (int k = 0; k < 4; ++k) side.bc[k] = __builtin_amdgcn_readfirstlane(hot->bc[k]);
  const LamSrc sxp = lam_src(F, side, lam_in, x, y, +1, 0), sxm = lam_src(F, side, lam_in, x, y, -1, 0);
  const LamSrc syp = lam_src(F, side, lam_in, x, y, 0, +1), sym = lam_src(F, side, lam_in, x, y, 0, -1);
  double xp[16], xm[16], yp[16], ym[16];
  auto load_x = [&]() {
    lam_planes<0>(F, sxp, xp);
    lam_planes<0>(F, sxm, xm);
  };
  auto load_y = [&]() {
    lam_planes<1>(F, syp, yp);
    lam_planes<1>(F, sym, ym);
  };
  if (!WIDE) {
    load_x();
    load_y();
  }
  // neighbour records: velocities for A, B and dL/dA, dL/dB
  double GAxp, GBxp, uxxp, uyxp, GAxm, GBxm, uxxm, uyxm, GAyp, GByp, uxyp, uyyp, GAym, GBym, uxym, uyym;
  rec_point(F, side, cold, rec, x, y, +1, 0, GAxp, GBxp, uxxp, uyxp);
  rec_point(F, side, cold, rec, x, y, -1, 0, GAxm, GBxm, uxxm, uyxm);
  rec_point(F, side, cold, rec, x, y, 0, +1, GAyp, GByp, uxyp, uyyp);
  rec_point(F, side, cold, rec, x, y, 0, -1, GAym, GBym, uxym, uyym);
  if (!WIDE) __builtin_amdgcn_sched_barrier(0);  // all issued by here, not one by one where they are used
  stage_hot(hot, &hs);
  const Hot& c = hs;
  const double A = (uxxp - uxxm) * c.inv2dx - (uyyp - uyym) * c.inv2dy;
  const double B = (uyxp - uyxm) * c.inv2dx + (uxyp - uxym) * c.inv2dy;
  const double gux = (GAxm - GAxp) * c.inv2dx + (GBym - GByp) * c.inv2dy;
  const double guy = (GBxm - GBxp) * c.inv2dx - (GAym - GAyp) * c.inv2dy;
  double sg[12], m[16], mu[16], nu[16], out[16];
#pragma unroll
  for (int k = 0; k < 12; ++k) sg[k] = 0.0;
  moments_from_f(f, m);
  minvt_apply(l, mu);
  if (WIDE) __builtin_amdgcn_sched_barrier(0);
  collision_adjoint<VER>(c, adj, m, A, B, mu, gux, guy, nu, sg);
  mt_apply(nu, out);
  const bool zxl = x == 0 && side.bc[0] == BC_ZERO_GRADIENT, zxh = x == F.nx - 1 && side.bc[1] == BC_ZERO_GRADIENT;
  const bool zyl = y == 0 && side.bc[2] == BC_ZERO_GRADIENT, zyh = y == F.ny - 1 && side.bc[3] == BC_ZERO_GRADIENT;
  double zx[2], zy[2];
  zero_gradient_t(c.lx, zxl, zxh, zx);
  zero_gradient_t(c.ly, zyl, zyh, zy);
  if (WIDE) {
    __builtin_amdgcn_sched_barrier(0);
    load_x();
  }
  convect_t<0>(c, zx, l, xp, xm, out);
  if (WIDE) {
    __builtin_amdgcn_sched_barrier(0);
    load_y();
  }
  convect_t<1>(c, zy, l, yp, ym, out);
#pragma unroll
  for (int i = 0; i < 16; ++i) out[i] += l[i];
  if (WIDE) {
    __builtin_amdgcn_sched_barrier(0);
    load_prev();
  }
  double r[NREC];
  record_from(c, fp, out, r);
  // threads outside store the edge node's values again, the same bits (under a
  // branch the loads would move into it, behind each other's waits)
#pragma unroll
  for (int i = 0; i < 16; ++i) lam_out[k0 + i * F.plane] = out[i];
  if (f_prev) {
#pragma unroll
    for (int j = 0; j < NREC; ++j) rec_out[k0 + j * F.plane] = r[j];
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) sg[k] = inside ? sg[k] : 0.0;
  // deterministic block reduction, one slot per block, accumulated over steps
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const double w = wave_sum(sg[k]);
    if ((t & 63) == 0) red[k][t >> 6] = w;
  }
  __syncthreads();
  if (t < 12) partials[slot * 12 + t] = psum + ((red[t][0] + red[t][1]) + (red[t][2] + red[t][3]));
}

}  // namespace lbm

namespace lbm {

// Transpose of a non-equilibrium extrapolation wall (Sec. IV.A): the step
// writes f_w = f^eq(rho_n, u_w, T_w) + f_n - f^eq(rho_n, u_n, T_n) from the
// fluid neighbour's new distributions f_n, so lambda_n += (d f_w / d f_n)^T
// lambda_w. With mu = M^-T lambda_w (f^eq = M^-1 q): the fixed-state
// equilibrium depends on f_n through rho only (d rho / d f_i = 1), the
// neighbour's through (rho, j, e) = the first four moments (M^T of their
// derivatives), both by dual numbers through the step's own equilibria.
template <int VER>
LBM_HD void wall_t_apply(const double* wall, const double* fn, const double* lw, double* ln) {
  double mu[16], m[16];
  minvt_apply(lw, mu);
  moments_from_f(fn, m);
  const double uwx = wall[1], uwy = wall[2], ew = wall[3] + 0.5 * (uwx * uwx + uwy * uwy);
  double g1 = 0.0;
  {
    const Dual r(m[0], 1.0);
    Dual q[16];
    equilibrium_moments<VER, Dual>(r, r * uwx, r * uwy, r * ew, q);
#pragma unroll
    for (int k = 0; k < 16; ++k) g1 += mu[k] * q[k].d;
  }
  double nu[16];
#pragma unroll
  for (int k = 4; k < 16; ++k) nu[k] = 0.0;
#pragma unroll 1
  for (int a = 0; a < 4; ++a) {
    Dual cc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) cc[b] = Dual(m[b], a == b ? 1.0 : 0.0);
    Dual q[16];
    equilibrium_moments<VER, Dual>(cc[0], cc[1], cc[2], cc[3], q);
    double g = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) g += mu[k] * q[k].d;
#pragma unroll
    for (int b = 0; b < 4; ++b) nu[b] = (a == b) ? g : nu[b];
  }
  double t[16];
  mt_apply(nu, t);
#pragma unroll
  for (int i = 0; i < 16; ++i) ln[i] += lw[i] + g1 - t[i];
}

// Wall transposes of one adjoint step, applied to lambda^{n+1} before the
// step's transpose; F.fin = f^{n+1}. One thread per node along the walled
// sides (walls on one axis only); the wall node's own lambda is then 0 (the
// step overwrites it). With two walls 3 nodes apart both act on the same
// fluid node, in turn, in the same thread.
template <int VER>
__global__ __launch_bounds__(64) void k_adj_walls(Field F, double* __restrict__ lam, const Hot* __restrict__ hot,
                                                  const Cold* __restrict__ cold) {
  const bool ywalls = hot->bc[2] == BC_NEQ_WALL || hot->bc[3] == BC_NEQ_WALL;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (ywalls ? F.nx : F.ny)) return;
  const int across = ywalls ? F.ny : F.nx;
  for (int side = 0; side < 2; ++side) {
    const int sd = (ywalls ? 2 : 0) + side;
    if (hot->bc[sd] != BC_NEQ_WALL) continue;
    const int wpos = side == 0 ? 0 : across - 1, npos = side == 0 ? 1 : across - 2;
    const long long kw = ywalls ? (long long)wpos * F.pitch + i : (long long)i * F.pitch + wpos;
    const long long kn = ywalls ? (long long)npos * F.pitch + i : (long long)i * F.pitch + npos;
    double lw[16], fn[16], ln[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      lw[j] = lam[kw + j * F.plane];
      fn[j] = F.fin[kn + j * F.plane];
      ln[j] = lam[kn + j * F.plane];
    }
    wall_t_apply<VER>(cold->wall[sd], fn, lw, ln);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      lam[kn + j * F.plane] = ln[j];
      lam[kw + j * F.plane] = 0.0;
    }
  }
}

// lambda at the final level from dL/d(rho, u_x, u_y, T) of the final fields
// (any gradient pointer may be NULL); the fields are rho = m1, u = (m2, m3)/m1,
// T = m4/m1 - |u|^2/2 (R = 1).
LBM_HD void adj_final_node(const Field& F, const double* __restrict__ g_rho, const double* __restrict__ g_ux,
                           const double* __restrict__ g_uy, const double* __restrict__ g_T, double* __restrict__ lam,
                           int x, int y) {
  const long long k = (long long)y * F.pitch + x;
  const long long d = (long long)y * F.nx + x;
  double f[16], m[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) f[i] = F.fin[k + i * F.plane];
  moments_from_f(f, m);
  const double r = m[0], ir = 1.0 / r;
  const double gr = g_rho ? g_rho[d] : 0.0, gu = g_ux ? g_ux[d] : 0.0, gv = g_uy ? g_uy[d] : 0.0,
               gt = g_T ? g_T[d] : 0.0;
  double nu[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) nu[i] = 0.0;
  const double ux = m[1] * ir, uy = m[2] * ir;
  nu[0] = gr - (gu * ux + gv * uy) * ir + gt * (-m[3] * ir * ir + (ux * ux + uy * uy) * ir);
  nu[1] = gu * ir - gt * ux * ir;
  nu[2] = gv * ir - gt * uy * ir;
  nu[3] = gt * ir;
  double l[16];
  mt_apply(nu, l);
#pragma unroll
  for (int i = 0; i < 16; ++i) lam[k + i * F.plane] = l[i];
}

template <int U>
__global__ void k_adj_final(Field F, const double* __restrict__ g_rho, const double* __restrict__ g_ux,
                            const double* __restrict__ g_uy, const double* __restrict__ g_T, double* __restrict__ lam) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= F.nx) return;
  adj_final_node(F, g_rho, g_ux, g_uy, g_T, lam, x, y);
}

// dL/d(rho0, u0, T0) from lambda^0: f^0 = M^-1 q(rho, rho u, rho (T + u^2/2)).
template <int VER>
LBM_HD void adj_init_node(const Field& F, const double* __restrict__ lam, const double* __restrict__ rho,
                          const double* __restrict__ ux, const double* __restrict__ uy, const double* __restrict__ T,
                          double* g_rho, double* g_ux, double* g_uy, double* g_T, int x, int y) {
  const long long k = (long long)y * F.pitch + x;
  const long long d = (long long)y * F.nx + x;
  double l[16], mu[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) l[i] = lam[k + i * F.plane];
  minvt_apply(l, mu);
  const double p0[4] = {rho[d], ux[d], uy[d], T[d]};
  double g[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    Dual pv[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) pv[b] = Dual(p0[b], a == b ? 1.0 : 0.0);
    const Dual jx = pv[0] * pv[1], jy = pv[0] * pv[2];
    const Dual e = pv[0] * (pv[3] + 0.5 * (pv[1] * pv[1] + pv[2] * pv[2]));
    Dual q[16];
    equilibrium_moments<VER, Dual>(pv[0], jx, jy, e, q);
    double s = 0.0;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) s += mu[kk] * q[kk].d;
    g[a] = s;
  }
  if (g_rho) g_rho[d] = g[0];
  if (g_ux) g_ux[d] = g[1];
  if (g_uy) g_uy[d] = g[2];
  if (g_T) g_T[d] = g[3];
}

template <int VER>
__global__ void k_adj_init(Field F, const double* __restrict__ lam, const double* __restrict__ rho,
                           const double* __restrict__ ux, const double* __restrict__ uy, const double* __restrict__ T,
                           double* g_rho, double* g_ux, double* g_uy, double* g_T) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= F.nx) return;
  adj_init_node<VER>(F, lam, rho, ux, uy, T, g_rho, g_ux, g_uy, g_T, x, y);
}

// One pass of the fixed-order reduction of per-block partials [nrows][12]:
// out row r = sum of input rows r*CHUNK .. r*CHUNK + CHUNK - 1 (in order).
constexpr int ADJ_CHUNK = 64;
template <int U>
__global__ void k_adj_reduce(const double* __restrict__ in, int nrows, double* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long nout = ((long long)nrows + ADJ_CHUNK - 1) / ADJ_CHUNK;
  if (i >= nout * 12) return;
  const long long r = i / 12;
  const int comp = (int)(i % 12);
  const long long b0 = r * ADJ_CHUNK, b1 = min(b0 + ADJ_CHUNK, (long long)nrows);
  double s = 0.0;
  for (long long b = b0; b < b1; ++b) s += in[b * 12 + comp];
  out[i] = s;
}

// dL/ds_1..16 from the last reduction row (s_1..s_4 have no effect).
template <int U>
__global__ void k_adj_grad(const double* __restrict__ row, double* __restrict__ grad_s) {
  const int k = threadIdx.x;
  if (k < 16) grad_s[k] = (k >= 4) ? row[k - 4] : 0.0;
}

template <int U>
__global__ void k_raise_flag(int* flag) {
  if (threadIdx.x == 0) flag[0] = 1;
}

template <int U>
__global__ void k_zero(double* p, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

}  // namespace lbm
