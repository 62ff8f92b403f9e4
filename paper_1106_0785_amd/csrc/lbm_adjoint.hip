// Checkpointed forward sweep and reverse (adjoint) sweep; contracts in
// include/lbm_adjoint.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

#include "../../include/lbm_adjoint.h"
#include "lbm_adjoint_fused.h"
#include "lbm_internal.h"

using namespace lbm;

namespace {

size_t a256(size_t x) { return (x + 255) / 256 * 256; }

constexpr int HEALTH_WORDS = 64;  // int32 words of the flag block

struct AdjLayout {
  int C, K;               // checkpoint interval, segments
  long long pitch, plane;  // distribution layout
  int gx, gy;             // adjoint launch grid
  long long slots;        // partial dL/ds sums: one per block or tile
  size_t consts, adj, ckpt, seg, lam, rec, partials, red, red_bytes, flag, total;
};

lbm_status adj_layout(const lbm_params* p, int64_t nsteps, int32_t ckpt, AdjLayout* L) {
  lbm_status st = validate(p);
  if (st != LBM_OK) return st;
  if (p->scheme != 0) return fail(LBM_EINVAL, "the adjoint form supports scheme 0 (Lax-Wendroff) only");
  if (nsteps < 1) return fail(LBM_EINVAL, "nsteps must be >= 1");
  if (ckpt < 0) return fail(LBM_EINVAL, "checkpoint interval must be >= 0");
  L->C = ckpt > 0 ? ckpt : std::max(1, (int)std::lround(std::sqrt((double)nsteps)));
  L->C = (int)std::min<int64_t>(L->C, nsteps);
  L->K = (int)((nsteps + L->C - 1) / L->C);
  L->pitch = row_pitch(p->nx);
  L->plane = L->pitch * p->ny;
  L->gx = (p->nx + 63) / 64;
  L->gy = (p->ny + 3) / 4;
  // tiles have at least 4 rows
  L->slots = std::max<long long>((long long)L->gx * L->gy, (long long)((p->nx + ACOLS - 1) / ACOLS) * L->gy);
  const size_t state = (size_t)16 * L->plane * sizeof(double);
  size_t off = 0;
  L->consts = off;
  off += a256(sizeof(Consts));
  L->adj = off;
  off += a256(sizeof(AdjCoef));
  L->ckpt = off;
  off += (size_t)(L->K + 1) * state;
  L->seg = off;
  off += (size_t)std::max(L->C, 2) * state;
  L->lam = off;
  off += 2 * state;
  L->rec = off;
  off += 2 * a256((size_t)NREC * L->plane * sizeof(double));
  L->partials = off;
  off += a256((size_t)L->slots * 12 * sizeof(double));
  // two ping-pong buffers for the chunked reduction of the partials
  L->red = off;
  L->red_bytes = a256((size_t)((L->slots + ADJ_CHUNK - 1) / ADJ_CHUNK) * 12 * sizeof(double));
  off += 2 * L->red_bytes;
  L->flag = off;
  off += HEALTH_WORDS * sizeof(int);
  L->total = off;
  return LBM_OK;
}

}  // namespace

struct lbm_adjoint {
  lbm_params p;
  AdjLayout L;
  int64_t nsteps;
  hipStream_t stream;
  char* base;
  Consts host;
  AdjCoef adj;
  bool forward_done;
  // Segment whose levels the segment store holds, -1 if none. Not kept once a
  // call was captured into a graph: its replays overwrite the store unseen.
  int held = -1;
  bool captured = false;
  // Health words (int32 in the flag block): word 0 of every other step, words
  // 1..63 of the segments whose levels are stored, one after the other, so
  // that a sweep that finds its levels held reports what recomputing them
  // would. held_bad: the segment now held was found bad by a check.
  int word = 0;
  bool held_bad = false;
  int variant;  // adjoint step: 0 LDS-staged tiles, 1 one thread per node, global gathers
  double* state(size_t off, int i) { return (double*)(base + off) + (size_t)i * 16 * L.plane; }
  double* ckpt(int k) { return state(L.ckpt, k); }
  double* seg(int j) { return state(L.seg, j); }
  double* lam(int j) { return state(L.lam, j); }
  const Hot* dhot() { return &((Consts*)(base + L.consts))->hot; }
  const Cold* dcold() { return &((Consts*)(base + L.consts))->cold; }
  const AdjCoef* dadj() { return (const AdjCoef*)(base + L.adj); }
  double* rec(int j) {
    return (double*)(base + L.rec + (size_t)j * a256((size_t)NREC * L.plane * sizeof(double)));
  }
  double* partials() { return (double*)(base + L.partials); }
  double* red(int j) { return (double*)(base + L.red + (size_t)j * L.red_bytes); }
  int* flag() { return (int*)(base + L.flag); }
  Field field(const double* fin, double* fout) {
    Field F;
    F.fin = fin;
    F.fout = fout;
    F.nx = p.nx;
    F.ny = p.ny;
    F.pitch = L.pitch;
    F.plane = L.plane;
    return F;
  }
};

// Notes a stream capture; returns true when this handle has seen one.
static bool capture_seen(lbm_adjoint* a) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(a->stream, &st) != hipSuccess) {
    (void)hipGetLastError();  // not this call's error
    a->captured = true;
  }
  if (st != hipStreamCaptureStatusNone) a->captured = true;
  return a->captured;
}

static hipError_t step_into(lbm_adjoint* a, const double* fin, double* fout, int* flag) {
  return launch_step(a->field(fin, fout), a->dhot(), a->dcold(), a->p.eq_version, has_walls(&a->p), 0, 0,
                     default_tile(a->p.nx, a->p.ny), flag, a->stream);
}

// The segment store is about to be filled anew: the health word of its steps.
static void new_levels(lbm_adjoint* a) {
  a->held = -1;
  a->held_bad = false;
  a->word = a->word % (HEALTH_WORDS - 1) + 1;
}

// Steps from f^n (fin) into the levels of the segment store from `level` on,
// at most `left`; sets how many. Many per launch in windows where each window
// has a CU of its own, else one (whole runs of 90 steps forward and backward,
// windows against single steps: 1854 against 2106 us at 300 x 100, 1587
// against 1900 at 200 x 32; with three windows per CU, 60 steps at 512 x 128,
// 1686 against 1676, and 1540 against 1473 for 40 of version 3).
static hipError_t levels_into(lbm_adjoint* a, const double* fin, int level, int64_t left, int* taken) {
  const int variant = default_variant(&a->p), ver = a->p.eq_version;
  double* fout = a->seg(level);
  int* flag = a->flag() + a->word;
  *taken = 1;
  if (variant != 2 && variant != 3) return step_into(a, fin, fout, flag);
  WinGeom g;
  if (variant == 2) {
    g.x = win_axis(a->p.nx, a->p.nx, 0, false);
    g.y = win_axis(a->p.ny, a->p.ny, 0, false);
    g.h = (int)std::min<int64_t>(1 << 16, left);
  } else {
    g = default_window(&a->p);
    if ((long long)g.x.nwin * g.y.nwin > 256) return step_into(a, fin, fout, flag);
  }
  *taken = (int)std::min<int64_t>(g.h, left);
  const int threads = (g.x.w * g.y.w + 63) / 64 * 64;
  decltype(&k_step_window<1, false, 256, true>) k;
#define LBM_LEVELS(WALLS, NODES)                                                                                \
  k = ver == 2 ? k_step_window<2, WALLS, NODES, true> : ver == 3 ? k_step_window<3, WALLS, NODES, true>        \
                                                                 : k_step_window<1, WALLS, NODES, true>
  if (threads <= 256 && variant == 3) {
    if (has_walls(&a->p)) LBM_LEVELS(true, 256); else LBM_LEVELS(false, 256);
  } else {
    if (has_walls(&a->p)) LBM_LEVELS(true, SMALL_NODES); else LBM_LEVELS(false, SMALL_NODES);
  }
#undef LBM_LEVELS
  hipLaunchKernelGGL(k, dim3(g.x.nwin * g.y.nwin), dim3(threads), 0, a->stream, a->field(fin, fout), a->dhot(),
                     a->dcold(), g, *taken, flag);
  return hipGetLastError();
}

// Tiles of the LDS-staged adjoint step: 512 run at a time (two workgroups per
// CU), so the height (a multiple of 4, at most 64) of the fewest rounds times
// rows and start-up, as for the two-step kernel.
static MarchGeom adjoint_geom(int nx, int ny) {
  const long long strips = (nx + ACOLS - 1) / ACOLS;
  int rows = WAVES;
  long long cost = -1;
  for (int r = WAVES; r <= 64; r += WAVES) {
    const long long t = (strips * ((ny + r - 1) / r) + 511) / 512 * (r + 6);
    if (cost < 0 || t < cost) cost = t, rows = r;
  }
  MarchGeom g = march_geom(nx, ny, TileShape{rows, WAVES, 1});
  g.nstrips = (int)strips;
  g.ntiles = g.nstrips * g.nsegs;
  g.per_xcd = (g.ntiles + 7) / 8;
  return g;
}

// (Times per step of a backward pass over stored levels, launch gaps and
// records passes included; the kernels alone take less, k_adj_step 12.2 us at
// 512 x 128.) The gather step where its blocks have a CU each (13.8 us at
// 512 x 128, the LDS-staged one 17.8), or two on half of them and the staged
// step's tiles would be 8 rows tall (26.4 against 28.7 at 1000 x 128); the
// staged step otherwise (18.1 against 21.9 at 400 x 200 with 4-row tiles, 27.4
// against 34.9 at 700 x 220, 59 against 89 at 900 x 600, 230 against 336 at
// 2048 x 1024).
static bool staged_step(int nx, int ny) {
  const long long blocks = (long long)((nx + 63) / 64) * ((ny + 3) / 4);
  return blocks > 512 || (blocks > 256 && adjoint_geom(nx, ny).rows == WAVES);
}

extern "C" {

size_t lbm_adjoint_workspace_bytes(const lbm_params* p, int64_t nsteps, int32_t ckpt_interval) {
  AdjLayout L;
  if (adj_layout(p, nsteps, ckpt_interval, &L) != LBM_OK) return 0;
  return L.total;
}

lbm_status lbm_adjoint_create(const lbm_params* p, int64_t nsteps, int32_t ckpt_interval, void* d_workspace,
                              size_t ws_bytes, void* hip_stream, lbm_adjoint** out) {
  if (!out) return fail(LBM_EINVAL, "out is NULL");
  *out = nullptr;
  AdjLayout L;
  lbm_status st = adj_layout(p, nsteps, ckpt_interval, &L);
  if (st != LBM_OK) return st;
  if (!d_workspace || ((uintptr_t)d_workspace) % 256) return fail(LBM_EINVAL, "workspace must be 256-byte aligned");
  if (ws_bytes < L.total) return fail(LBM_ENOMEM, "workspace has %zu bytes, needs %zu", ws_bytes, L.total);
  lbm_adjoint* a = new (std::nothrow) lbm_adjoint;
  if (!a) return fail(LBM_ENOMEM, "host allocation failed");
  a->p = *p;
  a->L = L;
  a->nsteps = nsteps;
  a->stream = (hipStream_t)hip_stream;
  a->base = (char*)d_workspace;
  a->forward_done = false;
  a->variant = staged_step(p->nx, p->ny) ? 0 : 1;
  make_coef(p, &a->host.hot, &a->host.cold);
  std::memset(&a->adj, 0, sizeof(a->adj));
  const double dt = p->dt, s5 = p->s[4], s6 = p->s[5], s7 = p->s[6], s8 = p->s[7];
  a->adj.mdt = -dt;
  if (p->modified) {
    const double sgn = (p->modified == 2) ? 1.0 : -1.0;
    a->adj.dcm[0] = dt * s7 / (s5 * s5);  // d cm0 / d s5
    a->adj.dcm[1] = -dt / s5;             // d cm0 / d s7
    a->adj.dcm[2] = dt * s7 / (s6 * s6);  // d cm1 / d s6
    a->adj.dcm[3] = -dt / s6;             // d cm1 / d s7
    a->adj.dcm[4] = dt * s8 / (s6 * s6);  // d cm2 / d s6
    a->adj.dcm[5] = -dt / s6;             // d cm2 / d s8
    a->adj.dcm[6] = dt * sgn * s8 / (s5 * s5);  // d cm3 / d s5
    a->adj.dcm[7] = -dt * sgn / s5;             // d cm3 / d s8
  }
  hipError_t e = hipMemcpyAsync(a->base + L.consts, &a->host, sizeof(Consts), hipMemcpyHostToDevice, a->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(a->base + L.adj, &a->adj, sizeof(AdjCoef), hipMemcpyHostToDevice, a->stream);
  if (e == hipSuccess) e = hipMemsetAsync(a->flag(), 0, HEALTH_WORDS * sizeof(int), a->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(a->stream);
  if (e != hipSuccess) {
    delete a;
    return hip_fail(e, "uploading adjoint constants");
  }
  *out = a;
  clear_error();
  return LBM_OK;
}

lbm_status lbm_adjoint_forward(lbm_adjoint* a, const double* d_rho0, const double* d_ux0, const double* d_uy0,
                               const double* d_T0) {
  if (!a || !d_rho0 || !d_ux0 || !d_uy0 || !d_T0) return fail(LBM_EINVAL, "NULL argument");
  const int ver = a->p.eq_version;
  {
    Field F = a->field(nullptr, a->ckpt(0));
    dim3 grid((a->p.nx + 63) / 64, a->p.ny);
    auto k = ver == 2 ? k_init<2> : ver == 3 ? k_init<3> : k_init<1>;
    hipLaunchKernelGGL(k, grid, dim3(64), 0, a->stream, F, nullptr, d_rho0, d_ux0, d_uy0, d_T0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_init launch");
  }
  new_levels(a);
  const int C = a->L.C, K = a->L.K;
  // between checkpoints no intermediate state is kept, so steps go many per
  // launch with the kernel the problem takes by default (8.2 us per step one
  // by one at 512 x 128, 7.0 in windows); the last segment's levels go
  // straight to where the backward pass reads them, which then need not
  // recompute them
  const int variant = default_variant(&a->p);
  const bool walls = has_walls(&a->p);
  const TileShape t2 = default_tile2(a->p.nx, a->p.ny);
  const WinGeom win = default_window(&a->p);
  for (int k = 0; k < K; ++k) {
    const int64_t n0 = (int64_t)k * C, n1 = std::min<int64_t>(n0 + C, a->nsteps);
    const double* fin = a->ckpt(k);
    int j = 0;
    for (int64_t n = n0; n < n1;) {
      const int64_t left = n1 - n;
      int64_t take = 1;
      if (k < K - 1) {
        if (variant == 2) take = std::min<int64_t>(1 << 16, left);
        if (variant == 3) take = std::min<int64_t>(win.h, left);
        if (variant == 4 && left >= 2) take = 2;
      }
      hipError_t e;
      if (k == K - 1 && left > 1) {
        int taken = 0;
        const int level = (int)(n + 1 - n0);
        e = levels_into(a, fin, level, left - 1, &taken);
        if (e != hipSuccess) return hip_fail(e, "forward step launch");
        fin = a->seg(level + taken - 1);
        n += taken;
        continue;
      }
      double* fout = n + take == n1 ? a->ckpt(k + 1) : a->seg(j);
      const Field F = a->field(fin, fout);
      if (take == 1)
        e = step_into(a, fin, fout, a->flag());
      else if (variant == 2)
        e = launch_small(F, a->dhot(), a->dcold(), ver, walls, (int)take, a->flag(), a->stream);
      else if (variant == 3)
        e = launch_window(F, a->dhot(), a->dcold(), ver, walls, win, (int)take, a->flag(), a->stream);
      else
        e = launch_step2(F, a->dhot(), a->dcold(), ver, t2, a->flag(), a->stream);
      if (e != hipSuccess) return hip_fail(e, "forward step launch");
      fin = fout;
      j ^= 1;
      n += take;
    }
  }
  a->held = capture_seen(a) ? -1 : K - 1;
  a->forward_done = true;
  return LBM_OK;
}

lbm_status lbm_adjoint_final_moments(lbm_adjoint* a, double* d_rho, double* d_ux, double* d_uy, double* d_T,
                                     double* d_p) {
  if (!a) return fail(LBM_EINVAL, "adjoint handle is NULL");
  if (!a->forward_done) return fail(LBM_ESTATE, "run lbm_adjoint_forward first");
  Field F = a->field(a->ckpt(a->L.K), nullptr);
  dim3 grid((a->p.nx + 63) / 64, a->p.ny);
  hipLaunchKernelGGL(k_moments<0>, grid, dim3(64), 0, a->stream, F, d_rho, d_ux, d_uy, d_T, d_p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "k_moments launch");
  return LBM_OK;
}

lbm_status lbm_adjoint_backward(lbm_adjoint* a, const double* d_rho0, const double* d_ux0, const double* d_uy0,
                                const double* d_T0, const double* d_g_rho, const double* d_g_ux,
                                const double* d_g_uy, const double* d_g_T, double* d_grad_rho0,
                                double* d_grad_ux0, double* d_grad_uy0, double* d_grad_T0, double* d_grad_s) {
  if (!a || !d_rho0 || !d_ux0 || !d_uy0 || !d_T0) return fail(LBM_EINVAL, "NULL argument");
  if (!a->forward_done) return fail(LBM_ESTATE, "run lbm_adjoint_forward first");
  if (capture_seen(a)) a->held = -1;
  const int ver = a->p.eq_version;
  const AdjLayout& L = a->L;
  const dim3 grow((a->p.nx + 63) / 64, a->p.ny);
  const dim3 gblk(L.gx, L.gy), bblk(64, 4);
  int cur = 0, rc = 0;
  // lambda^T from the gradients of the final fields
  hipLaunchKernelGGL(k_adj_final<0>, grow, dim3(64), 0, a->stream, a->field(a->ckpt(L.K), nullptr), d_g_rho, d_g_ux,
                     d_g_uy, d_g_T, a->lam(cur));
  const long long np = L.slots * 12;
  hipLaunchKernelGGL(k_zero<0>, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, a->stream, a->partials(), np);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "adjoint set-up launch");
  auto krec = ver == 2 ? k_adj_records<2> : ver == 3 ? k_adj_records<3> : k_adj_records<1>;
  auto kwall = ver == 2 ? k_adj_walls<2> : ver == 3 ? k_adj_walls<3> : k_adj_walls<1>;
  const bool walls = has_walls(&a->p);
  // grids of more than 2048 blocks (8 per CU) take the two-blocks-per-CU form
  // of the gather step (only where lbm_adjoint_set_variant asks for the gather
  // step: by default they take the staged one): 90 against 114 us per step at
  // 900 x 600; not version 3, which spills 94 registers there (203 against 154)
  const bool wide = (long long)L.gx * L.gy > 2048;
  auto kstep = ver == 3 ? k_adj_step<3, false>
               : wide   ? (ver == 2 ? k_adj_step<2, true> : k_adj_step<1, true>)
                        : (ver == 2 ? k_adj_step<2, false> : k_adj_step<1, false>);
  auto kfused = ver == 2 ? k_adj_fused<2, 4> : ver == 3 ? k_adj_fused<3, 4> : k_adj_fused<1, 4>;
  const MarchGeom ag = adjoint_geom(a->p.nx, a->p.ny);
  const bool staged = a->variant == 0;
  for (int k = L.K - 1; k >= 0; --k) {
    const int64_t n0 = (int64_t)k * L.C, n1 = std::min<int64_t>(n0 + L.C, a->nsteps);
    // recompute f^{n0+1} .. f^{n1-1} into the segment store (f^{n0} is the
    // checkpoint) unless it holds them already
    if (a->held != k) {
      new_levels(a);
      for (int64_t n = n0 + 1; n < n1;) {
        const double* fin = (n - 1 == n0) ? a->ckpt(k) : a->seg((int)(n - 1 - n0));
        int taken = 0;
        e = levels_into(a, fin, (int)(n - n0), n1 - n, &taken);
        if (e != hipSuccess) return hip_fail(e, "recompute step launch");
        n += taken;
      }
      if (!a->captured) a->held = k;
    } else if (a->held_bad) {
      hipLaunchKernelGGL(k_raise_flag<0>, dim3(1), dim3(64), 0, a->stream, a->flag());
      e = hipGetLastError();
      if (e != hipSuccess) return hip_fail(e, "health flag launch");
    }
    // Each gather step n needs the records (dL/dA, dL/dB, velocity) of
    // every node at level n (the staged step forms them itself); step n writes those of step n - 1 as it
    // produces lambda^n, except across a segment boundary, where level
    // n - 1 is not recomputed yet and a records pass runs first.
    for (int64_t n = n1 - 1; n >= n0; --n) {
      const double* fn = (n == n0) ? a->ckpt(k) : a->seg((int)(n - n0));
      // with NEQ walls lambda^{n+1} first takes the walls' transpose, so the
      // records of every step come from a separate pass after it
      const double* fprev =
          (walls || n - 1 < n0) ? nullptr : (n - 1 == n0) ? a->ckpt(k) : a->seg((int)(n - 1 - n0));
      Field F = a->field(fn, nullptr);
      if (walls) {
        const double* fnext = (n + 1 == n1) ? a->ckpt(k + 1) : a->seg((int)(n + 1 - n0));
        const int along = (a->p.bc[2] == LBM_BC_NEQ_WALL || a->p.bc[3] == LBM_BC_NEQ_WALL) ? a->p.nx : a->p.ny;
        hipLaunchKernelGGL(kwall, dim3((along + 63) / 64), dim3(64), 0, a->stream, a->field(fnext, nullptr),
                           a->lam(cur), a->dhot(), a->dcold());
      }
      if (!staged && (walls || n == n1 - 1))
        hipLaunchKernelGGL(krec, gblk, bblk, 0, a->stream, F, a->lam(cur), a->rec(rc), a->dhot());
      if (staged)
        hipLaunchKernelGGL(kfused, dim3(8 * ag.per_xcd), dim3(256), 0, a->stream, F, a->lam(cur), a->lam(cur ^ 1),
                           a->dhot(), a->dcold(), a->dadj(), a->partials(), ag);
      else
        hipLaunchKernelGGL(kstep, gblk, bblk, 0, a->stream, F, a->lam(cur), a->lam(cur ^ 1), a->rec(rc), a->dhot(),
                           a->dcold(), a->dadj(), a->partials(), fprev, a->rec(rc ^ 1));
      e = hipGetLastError();
      if (e != hipSuccess) return hip_fail(e, "adjoint step launch");
      cur ^= 1;
      if (fprev) rc ^= 1;
    }
  }
  // initial-state adjoint and the s-gradient
  auto kinit = ver == 2 ? k_adj_init<2> : ver == 3 ? k_adj_init<3> : k_adj_init<1>;
  hipLaunchKernelGGL(kinit, grow, dim3(64), 0, a->stream, a->field(a->ckpt(0), nullptr), a->lam(cur), d_rho0, d_ux0,
                     d_uy0, d_T0, d_grad_rho0, d_grad_ux0, d_grad_uy0, d_grad_T0);
  if (d_grad_s) {
    // fixed-order reduction of the per-block partials: chunks of ADJ_CHUNK
    // rows, repeated until one row is left
    const double* in = a->partials();
    long long rows = L.slots;
    int j = 0;
    do {
      const long long nout = (rows + ADJ_CHUNK - 1) / ADJ_CHUNK;
      hipLaunchKernelGGL(k_adj_reduce<0>, dim3((unsigned)((nout * 12 + 255) / 256)), dim3(256), 0, a->stream, in,
                         (int)rows, a->red(j));
      in = a->red(j);
      j ^= 1;
      rows = nout;
    } while (rows > 1);
    hipLaunchKernelGGL(k_adj_grad<0>, dim3(1), dim3(64), 0, a->stream, in, d_grad_s);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "adjoint finish launch");
  return LBM_OK;
}

lbm_status lbm_adjoint_set_variant(lbm_adjoint* a, int32_t variant) {
  if (!a) return fail(LBM_EINVAL, "adjoint handle is NULL");
  if (variant != 0 && variant != 1) return fail(LBM_EINVAL, "adjoint variant must be 0 or 1");
  a->variant = variant;
  return LBM_OK;
}

lbm_status lbm_adjoint_check(lbm_adjoint* a) {
  if (!a) return fail(LBM_EINVAL, "adjoint handle is NULL");
  int words[HEALTH_WORDS] = {};
  hipError_t e = hipMemcpyAsync(words, a->flag(), sizeof(words), hipMemcpyDeviceToHost, a->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(a->stream);
  if (e != hipSuccess) return hip_fail(e, "reading the health flag");
  bool bad = false;
  for (int v : words) bad |= v != 0;
  if (bad) {
    if (words[a->word] != 0) a->held_bad = true;
    e = hipMemsetAsync(a->flag(), 0, sizeof(words), a->stream);
    if (e != hipSuccess) return hip_fail(e, "hipMemsetAsync");
    return fail(LBM_ENONFINITE, "a forward step produced rho <= 0, T <= 0 or NaN");
  }
  return LBM_OK;
}

void lbm_adjoint_destroy(lbm_adjoint* a) { delete a; }

}  // extern "C"
