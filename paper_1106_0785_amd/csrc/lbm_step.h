// Device-side description of one time step and the node update shared by
// every step kernel (plain, fused, batched). The update follows Eq. (3) with
// the scheme of Sec. III: explicit collision at the old level plus per-axis
// central Lax-Wendroff convection, and the energy-flux modification (Sec. II).
#pragma once

#include "lbm_node.h"

namespace lbm {

enum { BC_PERIODIC = 0, BC_ZERO_GRADIENT = 1, BC_SPECULAR = 2, BC_NEQ_WALL = 3, BC_DIRICHLET_EQ = 4 };

// Per-problem coefficients read in the inner loop (kept small: they live in
// scalar registers).
struct Hot {
  double cq[12];   // -dt s_k for k = 5..16 (index k-5)
  double cmod[4];  // -dt (s7/s5-1), -dt (s7/s6-1), -dt (s8/s6-1), -dt sgn (s8/s5-1); 0 if unmodified
  double inv2dx, inv2dy;
  // Lax-Wendroff along one axis for a velocity component v = +1 / +2 with
  // c = v dt/dx: coefficient of f(x+1) is p = (c^2 - c)/2 and of f(x-1) is
  // m = (c^2 + c)/2; for v = -1 / -2 the two swap. Stored as p1, m1, p2, m2.
  double lx[4], ly[4];
  // Flux-limited scheme (scheme 1) along one axis: for speeds 1 and 2,
  // a = |v| dt/dx and k = a (1 - a)/2. Stored as a1, k1, a2, k2.
  double tx[4], ty[4];
  int bc[4];
  int version;
  int modified;
  int scheme;  // 0 Lax-Wendroff (Sec. III); 1 its minmod flux-limited form
};

// Rarely read per-problem data.
struct Cold {
  double ghost[4][16];  // equilibrium ghosts of DIRICHLET_EQ sides
  double wall[4][4];    // (rho, ux, uy, T) per side for NEQ walls
  double gvel[4][2];    // velocities of the ghosts
};

// Coefficients read through the scalar cache: a reference whose loads the
// compiler makes scalar (constant address space, wave-uniform pointer) and,
// because the pointer is new at each call, repeats where it is taken instead
// of keeping 50 scalar registers alive across a kernel's loop. Beside reads
// from LDS, where one 16-byte broadcast to a wave takes the pipe eight cycles,
// the reads cost the vector units nothing.
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) Hot ScalarHot;
__device__ __forceinline__ ScalarHot& scalar_hot(const Hot* p) {
  ScalarHot* q = (ScalarHot*)(unsigned long long)p;
  asm volatile("" : "+s"(q));
  return *q;
}
#else
typedef const Hot ScalarHot;
LBM_HD ScalarHot& scalar_hot(const Hot* p) { return *p; }
#endif

// Neighbour velocities the modification needs.
struct NbrVel {
  double ux_xp, uy_xp, ux_xm, uy_xm;  // at x+1, x-1
  double ux_yp, uy_yp, ux_ym, uy_ym;  // at y+1, y-1
};

LBM_HD void velocity_of(const double* f, double& ux, double& uy) {
  double rho, jx, jy;
  density_momentum(f, rho, jx, jy);
  const double ir = recip(rho);
  ux = jx * ir;
  uy = jy * ir;
}

// Adds to v the Lax-Wendroff convection increment of velocity I (Sec. III,
// G_ij): sum over axes of p (f(+1) - f) + m (f(-1) - f), with p = (c^2 - c)/2
// and m = (c^2 + c)/2 for c = v dt/dx. Written with differences so that a
// uniform state is reproduced exactly and the grid totals of rho, j, e are
// conserved to rounding (a centre coefficient 1 - c^2 would scale every
// distribution by a rounding bias each step). Starting from the collision's
// increment leaves two differences and two fused multiply-adds per axis.
template <int I>
LBM_HD double convect(const Hot& c, double v, double f, double fxp, double fxm, double fyp, double fym) {
  constexpr int ax = VX[I] < 0 ? -VX[I] : VX[I], ay = VY[I] < 0 ? -VY[I] : VY[I];
  if constexpr (ax != 0) {
    v = mad(c.lx[2 * (ax - 1) + (VX[I] > 0 ? 0 : 1)], fxp - f, v);
    v = mad(c.lx[2 * (ax - 1) + (VX[I] > 0 ? 1 : 0)], fxm - f, v);
  }
  if constexpr (ay != 0) {
    v = mad(c.ly[2 * (ay - 1) + (VY[I] > 0 ? 0 : 1)], fyp - f, v);
    v = mad(c.ly[2 * (ay - 1) + (VY[I] > 0 ? 1 : 0)], fym - f, v);
  }
  return v;
}

// minmod(a, b): the argument of smaller magnitude when both have the same
// sign, else 0.
LBM_HD double minmod(double a, double b) { return (a * b > 0.0) ? (fabs(a) < fabs(b) ? a : b) : 0.0; }

// Flux-limited convection increment along one axis (scheme 1): the
// Lax-Wendroff update of Sec. III whose anti-diffusive flux k (f(+1) - f) is
// limited by minmod of the two differences around it; POS: velocity
// component > 0; (a, k) from Hot::tx / Hot::ty for this speed; f2m .. f2p the
// values at -2 .. +2 along the axis. With minmod(d1, d2) replaced by d1 it is
// exactly convect() below.
template <bool POS>
LBM_HD double limited_axis(double a, double k, double f2m, double f1m, double f0, double f1p, double f2p) {
  const double dm = f0 - f1m, dp = f1p - f0;
  if (POS) return -a * dm - k * (minmod(dp, dm) - minmod(dm, f1m - f2m));
  return a * dp - k * (minmod(dp, f2p - f1p) - minmod(dm, dp));
}

// Both axes of velocity I with the flux-limited scheme.
template <int I>
LBM_HD double convect_limited(const Hot& c, double f, double x2m, double x1m, double x1p, double x2p, double y2m,
                              double y1m, double y1p, double y2p) {
  double v = 0.0;
  constexpr int ax = VX[I] < 0 ? -VX[I] : VX[I], ay = VY[I] < 0 ? -VY[I] : VY[I];
  if constexpr (ax != 0)
    v += limited_axis<(VX[I] > 0)>(c.tx[2 * (ax - 1)], c.tx[2 * (ax - 1) + 1], x2m, x1m, f, x1p, x2p);
  if constexpr (ay != 0)
    v += limited_axis<(VY[I] > 0)>(c.ty[2 * (ay - 1)], c.ty[2 * (ay - 1) + 1], y2m, y1m, f, y1p, y2p);
  return v;
}

// convect_limited<I> for a run-time velocity index (unrolled loops only).
LBM_HD double convect_limited_i(const Hot& c, int i, double f, double x2m, double x1m, double x1p, double x2p,
                                double y2m, double y1m, double y1p, double y2p) {
  double v = 0.0;
#define LBM_CASE(I) \
  case I: v = convect_limited<I>(c, f, x2m, x1m, x1p, x2p, y2m, y1m, y1p, y2p); break;
  switch (i) {
    LBM_CASE(0) LBM_CASE(1) LBM_CASE(2) LBM_CASE(3) LBM_CASE(4) LBM_CASE(5) LBM_CASE(6) LBM_CASE(7)
    LBM_CASE(8) LBM_CASE(9) LBM_CASE(10) LBM_CASE(11) LBM_CASE(12) LBM_CASE(13) LBM_CASE(14) LBM_CASE(15)
  }
#undef LBM_CASE
  return v;
}

template <int I>
struct ConvAll {
  LBM_HD static void run(const Hot& c, const double* f, const double* fxp, const double* fxm, const double* fyp,
                         const double* fym, double* acc) {
    acc[I] = convect<I>(c, acc[I], f[I], fxp[I], fxm[I], fyp[I], fym[I]);
    ConvAll<I + 1>::run(c, f, fxp, fxm, fyp, fym, acc);
  }
};
template <>
struct ConvAll<16> {
  LBM_HD static void run(const Hot&, const double*, const double*, const double*, const double*, const double*,
                         double*) {}
};

// The same along one axis only (AXIS 0: x, 1: y), for a node whose
// neighbours along the other axis are itself (a one-dimensional problem:
// those terms are exact zeros, left out).
template <int I, int AXIS, class C>
LBM_HD double convect_axis(C& c, double v, double f, double fp, double fm) {
  constexpr int vel = AXIS == 0 ? VX[I] : VY[I], k = vel < 0 ? -vel : vel;
  auto* l = AXIS == 0 ? c.lx : c.ly;
  if constexpr (k != 0) {
    v = mad(l[2 * (k - 1) + (vel > 0 ? 0 : 1)], fp - f, v);
    v = mad(l[2 * (k - 1) + (vel > 0 ? 1 : 0)], fm - f, v);
  }
  return v;
}

// Collision of one node in velocity space, -dt M^-1 Q (Sec. II), into df,
// from the node's moments m = M f and ir = 1 / m[0]; A = d_x u_x - d_y u_y
// and B = d_x u_y + d_y u_x. Returns false when rho <= 0, T <= 0 or a NaN
// appears.
template <int VER, class C>
LBM_HD bool collide_from_moments(C& c, const double* m, double ir, double A, double B, double* df) {
  const double rho = m[0], jx = m[1], jy = m[2], e = m[3];
  double q[16];
  equilibrium_moments<VER, double>(rho, ir, jx, jy, e, q);
  double col[16];
#pragma unroll
  for (int k = 4; k < 16; ++k) col[k] = c.cq[k - 4] * (m[k] - q[k]);
  const double ux = jx * ir, uy = jy * ir;
  const double rT = e - 0.5 * mad(jx, ux, jy * uy);  // rho T
  // energy-flux modification; its coefficients are exactly 0 for the
  // unmodified model, so the terms then add exactly 0 (no branch)
  const double tx = rT * ux, ty = rT * uy;
  const double xA = tx * A, xB = tx * B, yA = ty * A, yB = ty * B;
  col[6] = mad(c.cmod[1], yB, mad(c.cmod[0], xA, col[6]));
  col[7] = mad(c.cmod[3], yA, mad(c.cmod[2], xB, col[7]));
  f_from_nonconserved(col, df);
  return (rho > 0.0) && (rT > 0.0);
}

// The same from the distributions f and the neighbours' velocities.
template <int VER>
LBM_HD bool collide_delta(const Hot& c, const double* f, const NbrVel& nv, double* df) {
  double m[16];
  moments_from_f(f, m);
  const double A = mad(nv.ux_xp - nv.ux_xm, c.inv2dx, -((nv.uy_yp - nv.uy_ym) * c.inv2dy));
  const double B = mad(nv.uy_xp - nv.uy_xm, c.inv2dx, (nv.ux_yp - nv.ux_ym) * c.inv2dy);
  return collide_from_moments<VER>(c, m, recip(m[0]), A, B, df);
}

// New distributions at one interior node.
template <int VER>
LBM_HD bool node_update(const Hot& c, const double* f, const double* fxp, const double* fxm, const double* fyp,
                        const double* fym, const NbrVel& nv, double* out) {
  const bool ok = collide_delta<VER>(c, f, nv, out);
  ConvAll<0>::run(c, f, fxp, fxm, fyp, fym, out);
#pragma unroll
  for (int i = 0; i < 16; ++i) out[i] += f[i];
  return ok;
}

// Non-equilibrium extrapolation wall node from its fluid neighbour's new
// distributions fn (Sec. IV.A): f_w = f^eq(rho_n, u_w, T_w) + (f_n - f^eq(rho_n, u_n, T_n)).
template <int VER>
LBM_HD void neq_wall(const double* wall, const double* fn, double* fw) {
  double m[16];
  moments_from_f(fn, m);
  const double rho = m[0], ir = recip(rho);
  const double uwx = wall[1], uwy = wall[2], ew = wall[3] + 0.5 * (uwx * uwx + uwy * uwy);
  // the two equilibria differ in their moments only, so one back-transform
  // serves both
  double qw[16], qn[16];
  equilibrium_moments<VER, double>(rho, ir, rho * uwx, rho * uwy, rho * ew, qw);
  equilibrium_moments<VER, double>(rho, ir, m[1], m[2], m[3], qn);
#pragma unroll
  for (int k = 0; k < 16; ++k) qw[k] -= qn[k];
  reconstruct<true>(qw, fw);
#pragma unroll
  for (int i = 0; i < 16; ++i) fw[i] += fn[i];
}

}  // namespace lbm
