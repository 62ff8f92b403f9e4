// Adjoint step staged through an LDS ring (the layout of the fused forward
// kernel, lbm_kernels.h): a workgroup of W wavefronts owns a tile of 62
// columns x `rows` rows and marches up it W rows at a time, one lane per
// column, the two outer lanes for the neighbours' columns. Each ring entry
// holds what the transposed step reads at a stencil point: the 16 planes of
// lambda^{n+1} and the point's record (dL/dA, dL/dB and its velocity), with
// the ghost rules of the transposed step already applied (mirror: mirrored
// planes and record; zero gradient: the record's dL/dA, dL/dB negated;
// fixed state: lambda 0, dL/dA = dL/dB = 0 and the state's velocity). A record
// follows from lambda and f^n at its point, both there when the row enters
// the ring, so none is kept in memory, and f^n stays with the wave that
// updates the node (versions 1 and 2). The arithmetic is
// k_adj_step's, in the same order.
// Bound by memory at large grids: 384 bytes per node and step, against 576
// with the records of the next step formed from f^{n-1} and stored;
// 202 us at 2048 x 1024 (231 so; 217 with f^n read again at the update).
#pragma once

#include "lbm_adjoint_kernels.h"

namespace lbm {

constexpr int NA = 20;  // ring entry: 16 lambda planes + GA, GB, ux, uy
constexpr int RA = 64;         // columns of a ring row: the tile's ACOLS and one on each side
constexpr int ACOLS = RA - 2;

// Ghost values of a ring entry read from stored node (sx, sy) (resolve):
// lambda as lam_src / lam_planes transform it, the record as rec_point does.
__device__ __forceinline__ void fix_ghost_adj(const Hot& c, const Cold* __restrict__ cold, const Src& sx,
                                              const Src& sy, double* l, double* r) {
  if (__builtin_expect(sx.side < 0 && sy.side < 0, 1)) return;
  const int side = sx.side >= 0 ? sx.side : sy.side;
  const int kind = c.bc[side];
  if (sx.mode == 2 || sy.mode == 2) {
#pragma unroll
    for (int i = 0; i < 16; ++i) l[i] = 0.0;
  } else if (sx.mode == 1 || sy.mode == 1) {
    double t[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) t[i] = l[i];
    if (sx.mode == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i) l[i] = t[MIRROR_X[i]];
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) l[i] = t[MIRROR_Y[i]];
    }
  }
  if (kind == BC_DIRICHLET_EQ) {
    r[REC_GA] = r[REC_GB] = 0.0;
    velocity_of(cold->ghost[side], r[REC_UX], r[REC_UY]);
  } else if (kind == BC_SPECULAR) {
    r[REC_GB] = -r[REC_GB];
    if (side < 2)
      r[REC_UX] = -r[REC_UX];
    else
      r[REC_UY] = -r[REC_UY];
  } else if (kind == BC_ZERO_GRADIENT) {
    r[REC_GA] = -r[REC_GA];
    r[REC_GB] = -r[REC_GB];
  }
}

// Transposed convection and identity for velocity I at ring column c0, the
// new lambda stored at once (convect_t with ring reads).
template <int I>
struct AdjOutRing {
  __device__ __forceinline__ static void run(const Hot& c, const double* r0, const double* rp, const double* rm,
                                             const double* zx, const double* zy, double* __restrict__ lo,
                                             long long plane, double* out) {
    const double l = r0[I * RA];
    double v = out[I];
    if constexpr (VX[I] != 0) v = conv_t_axis<VX[I]>(v, c.lx, zx, r0[I * RA - 1], r0[I * RA + 1], l);
    if constexpr (VY[I] != 0) v = conv_t_axis<VY[I]>(v, c.ly, zy, rm[I * RA], rp[I * RA], l);
    out[I] = l + v;
    lo[I * plane] = out[I];
    AdjOutRing<I + 1>::run(c, r0, rp, rm, zx, zy, lo, plane, out);
  }
};
template <>
struct AdjOutRing<16> {
  __device__ __forceinline__ static void run(const Hot&, const double*, const double*, const double*, const double*,
                                             const double*, double* __restrict__, long long, double*) {}
};

// k_adj_step's node with lambda and the records of the node and its four
// neighbours from ring rows r0 (the node's), rp (y+1), rm (y-1), each at the
// node's column; f is the node's f^n. Writes lambda^n through lo (the node's
// address in lam_out).
template <int VER>
__device__ __forceinline__ void adj_node_ring(const Hot& c, const AdjCoef* __restrict__ adj, const double* r0,
                                              const double* rp, const double* rm, const double* f, const double* zx,
                                              const double* zy, double* __restrict__ lo, long long plane, double* sg) {
  double m[16];
  moments_from_f(f, m);
  const double GAxp = r0[(16 + REC_GA) * RA + 1], GBxp = r0[(16 + REC_GB) * RA + 1];
  const double uxxp = r0[(16 + REC_UX) * RA + 1], uyxp = r0[(16 + REC_UY) * RA + 1];
  const double GAxm = r0[(16 + REC_GA) * RA - 1], GBxm = r0[(16 + REC_GB) * RA - 1];
  const double uxxm = r0[(16 + REC_UX) * RA - 1], uyxm = r0[(16 + REC_UY) * RA - 1];
  const double GAyp = rp[(16 + REC_GA) * RA], GByp = rp[(16 + REC_GB) * RA];
  const double uxyp = rp[(16 + REC_UX) * RA], uyyp = rp[(16 + REC_UY) * RA];
  const double GAym = rm[(16 + REC_GA) * RA], GBym = rm[(16 + REC_GB) * RA];
  const double uxym = rm[(16 + REC_UX) * RA], uyym = rm[(16 + REC_UY) * RA];
  const double A = (uxxp - uxxm) * c.inv2dx - (uyyp - uyym) * c.inv2dy;
  const double B = (uyxp - uyxm) * c.inv2dx + (uxyp - uxym) * c.inv2dy;
  const double gux = (GAxm - GAxp) * c.inv2dx + (GBym - GByp) * c.inv2dy;
  const double guy = (GBxm - GBxp) * c.inv2dx - (GAym - GAyp) * c.inv2dy;
  double mu[16], nu[16];
  {
    double l[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) l[i] = r0[i * RA];
    minvt_apply(l, mu);
  }
  collision_adjoint<VER>(c, adj, m, A, B, mu, gux, guy, nu, sg);
  double out[16];
  mt_apply(nu, out);
  __builtin_amdgcn_sched_barrier(0);  // no ring reads before: they would take the collision's registers
  AdjOutRing<0>::run(c, r0, rp, rm, zx, zy, lo, plane, out);
}

// One tile of the adjoint step. F.fin = f^n; lam_in = lambda^{n+1}; lam_out =
// lambda^n. The tile's dL/ds contribution is added to partials[tile * 12 ..]
// (one slot per tile, fixed order).
template <int VER, int W>
__device__ __forceinline__ void adj_tile(Field F, const double* __restrict__ lam_in, double* __restrict__ lam_out,
                                         const Hot* __restrict__ hot, const Cold* __restrict__ cold,
                                         const AdjCoef* __restrict__ adj, double* __restrict__ partials, MarchGeom g,
                                         int tile) {
  constexpr int RING = W + 2;
  __shared__ double ring[RING][NA][RA];
  __shared__ Hot hs;
  __shared__ double red[12][W];
  __shared__ double held[16][RA];
  stage_hot(hot, &hs);
  const Hot& c = hs;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int strip = tile % g.nstrips, seg = tile / g.nstrips;
  const int nx = F.nx, ny = F.ny;
  const int x = strip * ACOLS - 1 + lane;
  const bool inside = lane >= 1 && lane <= ACOLS && x < nx;  // the columns the tile writes
  const int y0 = seg * g.rows;
  const int y1 = min(y0 + g.rows, ny);
  const int ylast = y1;  // last ring row the tile reads
  const int base = y0 - 1;
  const Src sx = (x < nx + 1) ? resolve(x, nx, c.bc[0], c.bc[1], 0) : Src{nx - 1, 0, -1};
  const int c0 = lane;
  const int bylo = __builtin_amdgcn_readfirstlane(hot->bc[2]);
  const int byhi = __builtin_amdgcn_readfirstlane(hot->bc[3]);
  auto ysrc = [&](int yr) -> Src {
    if (yr < 0 || yr >= ny) return resolve(yr, ny, bylo, byhi, 2);
    return Src{yr, 0, -1};
  };
  auto load_row = [&](int yr, double* l, double* f) {
    const int yi = ysrc(min(yr, ylast)).idx;
    const long long k = (long long)yi * F.pitch + sx.idx;
#pragma unroll
    for (int i = 0; i < 16; ++i) l[i] = lam_in[k + i * F.plane];
#pragma unroll
    for (int i = 0; i < 16; ++i) f[i] = F.fin[k + i * F.plane];
  };
  auto enter_row = [&](int yr, double* l, const double* f) {
    double r[NREC];
    record_from(c, f, l, r);
    fix_ghost_adj(c, cold, sx, ysrc(yr), l, r);
    const int slot = (unsigned)(yr - base) % RING;
#pragma unroll
    for (int i = 0; i < 16; ++i) ring[slot][i][c0] = l[i];
#pragma unroll
    for (int j = 0; j < NREC; ++j) ring[slot][16 + j][c0] = r[j];
  };
  // the node's column of plane 0 in a ring row, its planes at constant offsets
  // (opaque, or an address per plane is computed and kept for each)
  auto at = [&](int slot) -> const double* {
    int k = slot * (NA * RA) + c0;
    asm volatile("" : "+v"(k));
    return &ring[0][0][0] + k;
  };

  // prologue: ring rows y0-1 .. y0+W (wave w fills slots w and w + W < RING)
  {
    double la[16], fa[16], lb[16], fb[16];
    const bool two = w < RING - W;
    load_row(base + w, la, fa);
    if (two) load_row(base + w + W, lb, fb);
    if (base + w <= ylast) enter_row(base + w, la, fa);
    if (two && base + w + W <= ylast) enter_row(base + w + W, lb, fb);
  }
  double sg[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) sg[k] = 0.0;
  const bool zxl = x == 0 && c.bc[0] == BC_ZERO_GRADIENT, zxh = x == nx - 1 && c.bc[1] == BC_ZERO_GRADIENT;
  double zx[2];
  zero_gradient_t(c.lx, zxl, zxh, zx);
  // f^n of the row the wave updates next. Of the rows that enter the ring, a
  // wave takes the one it updates in the next iteration (wave 0 the one after
  // that, so it holds one row back), so f^n is read once. Version 3's update
  // leaves no registers for that, nor for the row to be in flight during it:
  // it reads f^n again.
  constexpr bool KEEP = VER != 3;
  double f[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) f[i] = F.fin[(long long)min(y0 + w, ny - 1) * F.pitch + sx.idx + i * F.plane];
  if (KEEP && w == 0) {
#pragma unroll
    for (int i = 0; i < 16; ++i) held[i][lane] = F.fin[(long long)min(y0 + W, ny - 1) * F.pitch + sx.idx + i * F.plane];
  }
  for (int Y = y0; Y < y1; Y += W) {
    const int y = Y + w;
    const long long k0 = (long long)min(y, ny - 1) * F.pitch + min(max(x, 0), nx - 1);
    const int yn = w == 0 ? Y + 2 * W : Y + W + w;
    double ln[16], fn[16];
    if constexpr (KEEP) {
      load_row(yn, ln, fn);  // in flight across the barrier
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) f[i] = F.fin[k0 + i * F.plane];
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    if (y < y1 && inside) {
      const int s0 = (unsigned)(y - base) % RING, sp = (unsigned)(y + 1 - base) % RING,
                sm = (unsigned)(y - 1 - base) % RING;
      const bool zyl = y == 0 && c.bc[2] == BC_ZERO_GRADIENT, zyh = y == ny - 1 && c.bc[3] == BC_ZERO_GRADIENT;
      double zy[2];
      zero_gradient_t(c.ly, zyl, zyh, zy);
      adj_node_ring<VER>(c, adj, at(s0), at(sp), at(sm), f, zx, zy, lam_out + k0, F.plane, sg);
    }
    if constexpr (!KEEP) {
      __builtin_amdgcn_sched_barrier(0);
      load_row(yn, ln, fn);
    }
    __syncthreads();
    if (yn <= ylast) enter_row(yn, ln, fn);
    if (!KEEP) continue;
    if (w == 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        f[i] = held[i][lane];
        held[i][lane] = fn[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) f[i] = fn[i];
    }
  }
  // deterministic tile sum: DPP/readlane within each wave, then the waves
  // in order; one slot per tile, accumulated over the steps
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const double s = wave_sum(sg[k]);
    if (lane == 0) red[k][w] = s;
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < W; ++v) s += red[threadIdx.x][v];
    partials[(long long)tile * 12 + threadIdx.x] += s;
  }
}

template <int VER, int W>
__global__ __launch_bounds__(64 * W, 2) void k_adj_fused(Field F, const double* __restrict__ lam_in,
                                                        double* __restrict__ lam_out, const Hot* __restrict__ hot,
                                                        const Cold* __restrict__ cold,
                                                        const AdjCoef* __restrict__ adj,
                                                        double* __restrict__ partials, MarchGeom g) {
  const int tile = xcd_tile(blockIdx.x, g);
  if (tile >= g.ntiles) return;  // whole workgroup leaves together
  adj_tile<VER, W>(F, lam_in, lam_out, hot, cold, adj, partials, g, tile);
}

}  // namespace lbm
