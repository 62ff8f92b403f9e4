// Multi-step kernel for grids that one launch per step leaves bound by
// launch cost or latency: overlapping LDS windows, several steps per launch
// (a small grid is one window, the whole of it). The plain kernel's stencil,
// ghost rules and node arithmetic.
#pragma once

#include "lbm_kernels.h"

namespace lbm {

constexpr int SMALL_NODES = 512;  // most nodes one workgroup holds, one thread each

// ---------------------------------------------------------------------------
// Windowed multi-step kernel: each workgroup holds a window of wc columns by
// wr rows in LDS (one thread per node) and advances it up to h steps per
// launch (temporal blocking). Along an axis that one window covers whole,
// neighbours follow the ghost rules as in the other kernels. Along an axis
// cut into windows, windows overlap by h nodes on each side cut from a
// neighbouring window; after k steps a node is exact if it lies at least k
// nodes from every cut side, so the middle (w - 2 h) nodes are written back
// and those parts tile the axis. On a periodic cut axis the window holds the
// periodic images of the stored nodes (the update is translation invariant);
// on other cut axes windows are clipped to the domain and the ghost rules
// apply at the domain edge. Narrow grids (few rows) use one window row.
// Each node's arithmetic is the plain kernel's.
// ---------------------------------------------------------------------------
struct WinAxis {
  int w;      // window extent (nodes held); the whole axis when nwin == 1 and whole
  int v;      // nodes written per window (w - 2 halo on a cut axis)
  int nwin;   // windows along the axis
  int whole;  // 1: one window holds the whole axis (no cuts)
  int halo;   // overlap per cut side: h, or h + 1 on an axis with NEQ walls
              // (a wall node takes its fluid neighbour's value of the same
              // step, so it is exact one step less long than its distance
              // from a cut side)
};

struct WinGeom {
  WinAxis x, y;
  int h;  // most steps per launch
};

// One axis of one window: held nodes [s, e) (virtual on a periodic cut
// axis), the nodes it writes [o, o + v), and which sides are cuts.
struct WinSpan {
  int s, n, o, v;
  bool lo_cut, hi_cut;
};

__device__ __forceinline__ WinSpan win_span(const WinAxis& a, int win, int len, bool per) {
  WinSpan r;
  if (a.whole) {
    r.s = 0;
    r.n = len;
    r.o = 0;
    r.v = len;
    r.lo_cut = r.hi_cut = false;
    return r;
  }
  r.o = win * a.v;
  r.v = a.v;
  int s = r.o - a.halo, e = r.o + a.v + a.halo;
  if (!per) {
    s = max(s, 0);
    e = min(e, len);
  }
  r.s = s;
  r.n = e - s;
  r.lo_cut = per || s > 0;
  r.hi_cut = per || e < len;
  return r;
}

// Neighbour (offset d = +-1) of local node w along one axis of a window:
// local index and ghost treatment. At a cut side the node's own index is
// returned: the node is outside the exact region from the first step on.
__device__ __forceinline__ Src win_nbr(const WinSpan& sp, int w, int g, int d, int len, int bc_lo, int bc_hi,
                                       int side, int& local) {
  const int w2 = w + d;
  if (w2 >= 0 && w2 < sp.n) {
    local = w2;
    return Src{w2, 0, -1};
  }
  if ((d < 0 && sp.lo_cut) || (d > 0 && sp.hi_cut)) {
    local = w;
    return Src{w, 0, -1};
  }
  const Src sg = resolve(g + d, len, bc_lo, bc_hi, side);
  local = sg.idx - sp.s;
  return sg;
}

// Convection of all 16 velocities of a windowed node added to acc, and acc to
// the node's distributions f; the neighbour values are read from the window as
// they are used (entries kxp .. kym; a ghost without a mirror is an entry too).
// MIR: some lane's neighbour is a mirror ghost, its own entry with the planes
// mirrored (flags bit 0 x+1, 1 x-1, 2 y+1, 3 y-1).
template <int I, bool MIR, int W>
__device__ __forceinline__ void window_convect(const Hot& c, const double (*buf)[W], int kxp, int kxm, int kyp,
                                               int kym, int flags, double* f, const double* acc) {
  auto at = [&](int k, int bit, int mirror) {
    if constexpr (MIR) return buf[(flags & bit) ? mirror : I][k];
    return buf[I][k];
  };
  f[I] += convect<I>(c, acc[I], f[I], VX[I] ? at(kxp, 1, MIRROR_X[I]) : 0.0, VX[I] ? at(kxm, 2, MIRROR_X[I]) : 0.0,
                     VY[I] ? at(kyp, 4, MIRROR_Y[I]) : 0.0, VY[I] ? at(kym, 8, MIRROR_Y[I]) : 0.0);
  if constexpr (I < 15) window_convect<I + 1, MIR, W>(c, buf, kxp, kxm, kyp, kym, flags, f, acc);
}

// NODES: most nodes a window holds. The window is held once and updated in
// place (every node computed into registers, then written over the old one
// after a barrier), and a thread keeps its node's distributions and moments
// in registers, so a step reads the 48 neighbour values only. One LDS copy and
// at most 168 registers (up to 384 nodes) let three waves share a SIMD where
// two copies left one or two. Bound by the latency of the node update at one
// wave per SIMD and by FP64 issue at three. Per step, against two copies and
// the moments formed again from LDS (same shapes): 3.5 against 3.9 us at
// 60 x 40 with walls, 6.6 against 8.8 at 512 x 128 (both 16 x 16 nodes, 4
// steps), 9.2 against 11.9 at 400 x 300 (16 x 16, 3 steps), 2.1 against 2.6
// at 2000 x 4 (64 x 4, 8 steps).
// LEVELS: every step's state is stored, that of step s at fout + (s - 1) 16
// planes (the adjoint keeps them).
template <int VER, bool WALLS, int NODES, bool LEVELS = false>
__global__ __launch_bounds__(NODES, NODES <= 384 ? 3 : 2) void k_step_window(Field F, const Hot* __restrict__ hot,
                                                      const Cold* __restrict__ cold, WinGeom wg, int nsteps,
                                                      int* flag) {
  // 16 distributions and the velocity of every held node, and the ghosts of
  // the four sides' fixed states
  constexpr int W = NODES + 4;
  __shared__ double buf[NV][W];
  __shared__ Hot hs;
  stage_hot(hot, &hs);
  const Hot& c = hs;
  const bool xper = c.bc[0] == BC_PERIODIC, yper = c.bc[2] == BC_PERIODIC;
  const WinSpan sx = win_span(wg.x, blockIdx.x % wg.x.nwin, F.nx, xper);
  const WinSpan sy = win_span(wg.y, blockIdx.x / wg.x.nwin, F.ny, yper);
  const int t = threadIdx.x;
  const bool active = t < sx.n * sy.n;
  const int xw = active ? t % sx.n : 0, yw = active ? t / sx.n : 0;
  const int xv = sx.s + xw, yv = sy.s + yw;  // virtual on a periodic cut axis
  const int xg = xper ? ((xv % F.nx) + F.nx) % F.nx : xv;
  const int yg = yper ? ((yv % F.ny) + F.ny) % F.ny : yv;
  const long long at = (long long)yg * F.pitch + xg;
  auto put = [&](const double* f, double ux, double uy) {
#pragma unroll
    for (int i = 0; i < 16; ++i) buf[i][t] = f[i];
    buf[16][t] = ux;
    buf[17][t] = uy;
  };
  double f[16], m[16], ir = 0.0;
  if (active) {
#pragma unroll
    for (int i = 0; i < 16; ++i) f[i] = F.fin[at + i * F.plane];
    moments_from_f(f, m);
    ir = recip(m[0]);
    put(f, m[1] * ir, m[2] * ir);
  }
  // A wall node's thread is a twin of its fluid neighbour: it updates the
  // neighbour's state itself and takes the wall's from that, so walls need no
  // phase of their own after the others' (one barrier and a pass through LDS
  // less per step). (xu, yu): the node the thread updates, in the window.
  const bool wall = WALLS && active && is_wall_node(c, xg, yg, F.nx, F.ny);
  int xu = xw, yu = yw, wside = 0;
  if (WALLS) {
    const bool ylo = wall && c.bc[2] == BC_NEQ_WALL && yg == 0, yhi = wall && c.bc[3] == BC_NEQ_WALL && yg == F.ny - 1;
    const bool xlo = wall && !ylo && !yhi && c.bc[0] == BC_NEQ_WALL && xg == 0, xhi = wall && !ylo && !yhi && !xlo;
    wside = ylo ? 2 : yhi ? 3 : xlo ? 0 : 1;
    yu += ylo ? 1 : yhi ? -1 : 0;
    xu += xlo ? 1 : xhi ? -1 : 0;
    if (active) {
      const long long au = at + (long long)(yu - yw) * F.pitch + (xu - xw);
#pragma unroll
      for (int i = 0; i < 16; ++i) f[i] = F.fin[au + i * F.plane];
      moments_from_f(f, m);
      ir = recip(m[0]);
    }
  }
  const int xgu = xg + (xu - xw), ygu = yg + (yu - yw);
  for (int k = t; k < 4 * NV; k += blockDim.x) {
    const int side = k / NV, i = k % NV;
    if (c.bc[side] == BC_DIRICHLET_EQ) buf[i][NODES + side] = i < 16 ? cold->ghost[side][i] : cold->gvel[side][i - 16];
  }
  int lxp, lxm, lyp, lym;
  const Src nxp = win_nbr(sx, xu, xgu, 1, F.nx, c.bc[0], c.bc[1], 0, lxp);
  const Src nxm = win_nbr(sx, xu, xgu, -1, F.nx, c.bc[0], c.bc[1], 0, lxm);
  const Src nyp = win_nbr(sy, yu, ygu, 1, F.ny, c.bc[2], c.bc[3], 2, lyp);
  const Src nym = win_nbr(sy, yu, ygu, -1, F.ny, c.bc[2], c.bc[3], 2, lym);
  const int kxp = nxp.mode == 2 ? NODES + nxp.side : yu * sx.n + lxp;
  const int kxm = nxm.mode == 2 ? NODES + nxm.side : yu * sx.n + lxm;
  const int kyp = nyp.mode == 2 ? NODES + nyp.side : lyp * sx.n + xu;
  const int kym = nym.mode == 2 ? NODES + nym.side : lym * sx.n + xu;
  const int flags = (nxp.mode == 1 ? 1 : 0) | (nxm.mode == 1 ? 2 : 0) | (nyp.mode == 1 ? 4 : 0) | (nym.mode == 1 ? 8 : 0);
  const bool mirrors = __any(flags != 0);  // wave-uniform
  // steps after which this node is no longer exact (its distance from the
  // nearest cut side): it is left alone from then on
  int far = nsteps;
  if (sx.lo_cut) far = min(far, xu);
  if (sx.hi_cut) far = min(far, sx.n - 1 - xu);
  if (sy.lo_cut) far = min(far, yu);
  if (sy.hi_cut) far = min(far, sy.n - 1 - yu);
  __syncthreads();
  auto writes = [&]() {
    return active && xv >= sx.o && xv < sx.o + sx.v && xv >= 0 && xv < F.nx && yv >= sy.o && yv < sy.o + sy.v &&
           yv >= 0 && yv < F.ny;
  };
  bool ok = true;
  for (int s = 1;; ++s) {
    const bool update = active && s <= far;
    if (update) {
      double uxp = buf[16][kxp], vxp = buf[17][kxp], uxm = buf[16][kxm], vxm = buf[17][kxm];
      double uyp = buf[16][kyp], vyp = buf[17][kyp], uym = buf[16][kym], vym = buf[17][kym];
      if (mirrors) {
        uxp = (flags & 1) ? -uxp : uxp;
        uxm = (flags & 2) ? -uxm : uxm;
        vyp = (flags & 4) ? -vyp : vyp;
        vym = (flags & 8) ? -vym : vym;
      }
      const double A = mad(uxp - uxm, c.inv2dx, -((vyp - vym) * c.inv2dy));
      const double B = mad(vxp - vxm, c.inv2dx, (uyp - uym) * c.inv2dy);
      double df[16];
      ok &= collide_from_moments<VER>(c, m, ir, A, B, df);
      if (mirrors)
        window_convect<0, true, W>(c, buf, kxp, kxm, kyp, kym, flags, f, df);
      else
        window_convect<0, false, W>(c, buf, kxp, kxm, kyp, kym, flags, f, df);
      moments_from_f(f, m);
      ir = recip(m[0]);
    }
    if (s == nsteps) break;  // nothing is read from the window any more
    __syncthreads();  // every node of this step has been read
    if (update && !wall) put(f, m[1] * ir, m[2] * ir);
    if (WALLS && update && wall) {
      double fw[16], ux, uy;
      neq_wall<VER>(cold->wall[wside], f, fw);
      velocity_of(fw, ux, uy);
      put(fw, ux, uy);
    }
    if (LEVELS && writes()) {  // (a wall node's state is in its own entry only)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        F.fout[(s - 1) * 16 * F.plane + at + i * F.plane] = (WALLS && wall) ? buf[i][t] : f[i];
    }
    __syncthreads();
  }
  if (writes()) {
    if (WALLS && wall) {
      double fw[16];
      neq_wall<VER>(cold->wall[wside], f, fw);
#pragma unroll
      for (int i = 0; i < 16; ++i) f[i] = fw[i];
    }
    double* out = F.fout + (LEVELS ? (nsteps - 1) * 16 * F.plane : 0) + at;
#pragma unroll
    for (int i = 0; i < 16; ++i) out[i * F.plane] = f[i];
  }
  if (!ok) flag[0] = 1;
}

}  // namespace lbm
