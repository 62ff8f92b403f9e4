"""The workloads that this library's performance is judged on.

A case is a dict of plain values. `listed()` gives the fixed ones, `draw(rng)`
one more of the same ranges, `prepare(case, seed)` what a program has in hand
before the call (fields on the GPU, the handle, a tuned batch), `run(state)`
one pass through the public entry points, `work(case)` the bytes and
operations a pass cannot do without, and `exact(case, seed)` the same outputs
from a plain FP64 torch implementation of the method (no code of the library).

Kinds of case:
  single     one problem: lbm_init, `steps` time steps, the moment fields
             (kernel and shape as lbm_create picks them)
  batch      many uneven problems: lbm_batch_init, `steps` steps, the moment
             fields of every instance (schedule from the autotuner, as the
             batched form is meant to be used)
  adjoint    `steps` steps forward and the reverse sweep: the misfit of the
             final density and its gradients with respect to the initial
             fields and log s_1..s_16 (through autograd's simulate(), or with
             an Adjoint handle kept between calls)
  stability  |omega|_max over a wavenumber grid for the paper's Fig. 2 cases
"""

import math

import numpy as np
import torch

from paper_1106_0785_amd import autograd, inputs, lbm, stability
from paper_1106_0785_amd.batch import Batch

FIELDS = ("rho", "ux", "uy", "T")

# FP64 operations of one node update that any form of the method needs: the
# structured moment transform and its inverse (about 80 and 70), the
# equilibrium moments and the relaxation with the energy-flux modification
# (about 90), and the Lax-Wendroff increments (24 axis terms of 6).
NODE_FLOPS = 380
# The adjoint step: the transposed transforms and stencil, and the derivative
# of the equilibria along the four conserved moments.
ADJOINT_FLOPS = 1200
# One squaring of a 16 x 16 complex matrix, and how many a radius takes.
SQUARING_FLOPS = 4 * 2 * 16**3
SQUARINGS = 48


def listed():
    return [
        # The paper's thermal Couette channel (Sec. IV.A): the smallest problem, in short calls of a program that
        # looks at the fields every 100 steps; latency is all that counts.
        {"name": "couette_4x64", "kind": "single", "problem": "couette", "nx": 4, "ny": 64, "steps": 100},
        # The Sod tube on a narrow grid (Sec. IV.B(a)): 2000 x 4 nodes, far too few to fill the chip.
        {"name": "sod_2000x4", "kind": "single", "problem": "riemann", "nx": 2000, "ny": 4, "steps": 500},
        # A wide channel between non-equilibrium walls with the version-2 equilibria: ragged strips, walls.
        {"name": "channel_130x96_v2", "kind": "single", "problem": "couette", "nx": 130, "ny": 96, "steps": 100,
         "eq_version": 2},
        # The paper's shock-bubble run (Figs. 7-8) at its own size: fixed inflow, extrapolation, reflection.
        {"name": "bubble_600x100", "kind": "single", "problem": "bubble", "nx": 600, "ny": 100, "steps": 200},
        # The shock/interface problem, cache-resident.
        {"name": "rm_1024x256", "kind": "single", "problem": "rm", "nx": 1024, "ny": 256, "steps": 200},
        # The same problem beyond the caches: the benchmark's headline workload.
        {"name": "rm_4096x1024", "kind": "single", "problem": "rm", "nx": 4096, "ny": 1024, "steps": 40},
        # The flux-limited scheme with a sharp interface on odd sizes.
        {"name": "limited_1023x257", "kind": "single", "problem": "rm", "nx": 1023, "ny": 257, "steps": 100,
         "scheme": 1},
        # A parameter study over one-dimensional problems: 512 uneven lines (the benchmark's batch).
        {"name": "batch_lines_512", "kind": "batch", "problem": "lines", "n": 512, "longest": 4096, "shapes": 0,
         "steps": 200},
        # A parameter study over two-dimensional problems: 96 uneven shock/interface set-ups.
        {"name": "batch_rm2d_96", "kind": "batch", "problem": "rm2d", "n": 96, "longest": 512, "shapes": 0,
         "steps": 50},
        # One gradient of an optimisation over rates and initial fields, at the benchmark's size (a short window of it).
        {"name": "adjoint_512x128", "kind": "adjoint", "nx": 512, "ny": 128, "steps": 100, "api": "simulate"},
        # The same beyond the caches, with the handle kept between iterations.
        {"name": "adjoint_2048x1024", "kind": "adjoint", "nx": 2048, "ny": 1024, "steps": 16, "api": "handle"},
        # The stability map of Fig. 2, cases (a)-(d).
        {"name": "stability_512x512", "kind": "stability", "grid": 512, "eq_version": 1},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges above: sizes log-uniform and odd as they come, every option in use."""
    kind = rng.choice(["couette", "riemann", "channel", "bubble", "rm", "rm", "limited", "lines", "rm2d", "mixed",
                       "adjoint", "stability"])
    version = rng.choice([1, 1, 2, 3])
    modified = rng.choice([1, 1, 0, 2])
    if kind == "couette":
        nx = rng.randint(1, 6)
        return {"kind": "single", "problem": "couette", "nx": nx, "ny": _log_int(rng, 9, 512 // nx),
                "steps": _log_int(rng, 20, 400), "eq_version": version, "modified": modified}
    if kind == "riemann":
        return {"kind": "single", "problem": "riemann", "nx": _log_int(rng, 600, 20000), "ny": rng.randint(1, 16),
                "steps": _log_int(rng, 50, 300), "modified": modified}
    if kind == "channel":
        return {"kind": "single", "problem": "couette", "nx": _log_int(rng, 17, 600), "ny": _log_int(rng, 40, 400),
                "steps": _log_int(rng, 20, 200), "eq_version": version, "modified": modified}
    if kind == "bubble":
        nx = _log_int(rng, 240, 1500)
        return {"kind": "single", "problem": "bubble", "nx": nx, "ny": max(40, nx // rng.randint(3, 6)),
                "steps": _log_int(rng, 20, 200), "modified": modified}
    if kind in ("rm", "limited"):
        nx = _log_int(rng, 200, 4096)
        ny = _log_int(rng, 32, max(33, min(nx // 2, 1024)))
        steps = max(5, min(200, 160_000_000 // (nx * ny)))
        case = {"kind": "single", "problem": "rm", "nx": nx, "ny": ny, "steps": steps if kind == "rm" else steps // 2 + 3}
        case.update({"eq_version": version, "modified": modified} if kind == "rm" else {"scheme": 1})
        return case
    if kind == "lines":
        return {"kind": "batch", "problem": "lines", "n": _log_int(rng, 16, 500), "longest": _log_int(rng, 600, 4000),
                "shapes": rng.randrange(1 << 20), "steps": _log_int(rng, 20, 200)}
    if kind == "rm2d":
        return {"kind": "batch", "problem": "rm2d", "n": _log_int(rng, 6, 90), "longest": _log_int(rng, 150, 500),
                "shapes": rng.randrange(1 << 20), "steps": _log_int(rng, 10, 50)}
    if kind == "mixed":
        return {"kind": "batch", "problem": "mixed", "n": _log_int(rng, 12, 96), "longest": _log_int(rng, 100, 320),
                "shapes": rng.randrange(1 << 20), "steps": _log_int(rng, 10, 60)}
    if kind == "adjoint":
        nx = _log_int(rng, 200, 1500)
        ny = _log_int(rng, 32, nx // 2)
        return {"kind": "adjoint", "nx": nx, "ny": ny, "steps": max(7, min(90, 6_000_000 // (nx * ny))),
                "api": rng.choice(["simulate", "handle"]), "eq_version": rng.choice([1, 1, 2]), "modified": modified}
    return {"kind": "stability", "grid": _log_int(rng, 12, 500), "eq_version": version}


# ---------------------------------------------------------------------------
# Inputs, from the case and the seed alone.
# ---------------------------------------------------------------------------
def _single_problem(case, seed):
    """(params, host fields) of a single or adjoint case."""
    rng = np.random.default_rng([seed, 11])
    nx, ny = case["nx"], case["ny"]
    problem = case.get("problem", "rm")
    modified = case.get("modified", 1)
    if problem == "couette":
        p, f, _ = inputs.couette(float(rng.uniform(0.5, 2.0)), nx=nx, ny=ny, u0=float(rng.uniform(0.05, 0.15)),
                                 T1=float(rng.uniform(1.005, 1.02)), modified=modified)
    elif problem == "riemann":
        (rl, ul, pl), (rr, ur, pr) = inputs.RIEMANN_STATES["sod"]
        k = rng.uniform(0.8, 1.2, size=4)
        dx = 1.0 / nx
        dt = min(1e-5, dx / 8.0)
        p, f, _ = inputs.riemann("sod", nx=nx, ny=ny, dt=dt, modified=modified,
                                 states=((rl * k[0], ul, pl * k[1]), (rr * k[2], ur, pr * k[3])))
    elif problem == "bubble":
        p, f, _ = inputs.shock_bubble(s5=1e4, s7=float(10.0 ** rng.uniform(4.0, 5.0)), nx=nx, ny=ny, modified=modified,
                                      bubble_rho=float(rng.uniform(0.13, 0.2)),
                                      radius=0.2 * ny * float(rng.uniform(0.9, 1.1)))
    else:
        limited = case.get("scheme", 0) == 1
        p, f, _ = inputs.rm(seed=seed, nx=nx, ny=ny, modified=modified, width_cells=0.5 if limited else 3.0)
        p["scheme"] = case.get("scheme", 0)
    p["eq_version"] = case.get("eq_version", 1)
    return p, _stir(p, f, rng)


def _stir(p, f, rng):
    """A weak smooth transverse motion (5 % of the sound speed of the quiet gas, none at y walls), so that both
    velocity components are alive in one-dimensional set-ups too."""
    nx, ny = p["nx"], p["ny"]
    x, y = (np.arange(nx)[None, :] + 0.5) / nx, (np.arange(ny)[:, None] + 0.5) / ny
    amp, phase = float(rng.uniform(0.03, 0.07)), float(rng.uniform(0.0, 2.0 * math.pi))
    if nx == 1:
        f["ux"] = f["ux"] + amp * np.sin(math.pi * y) ** 2
        f["uy"] = f["uy"] + amp * np.sin(math.pi * y) ** 2
    else:
        shape = np.sin(math.pi * y) ** 2 if p["bc"][2] in ("specular", "neq_wall") else np.ones_like(y)
        f["uy"] = f["uy"] + amp * np.sin(2.0 * math.pi * x + phase) * shape
    return f


def _batch_problems(case, seed):
    """The instances' sizes and set-ups belong to the case; their densities, transverse motion and Prandtl numbers to
    the seed."""
    n, longest, shapes = case["n"], case["longest"], case["shapes"]
    if case["problem"] == "lines":
        items = inputs.batch(seed=shapes, n=n, riemann_n=(256, longest), couette_h=(32, 256))
    elif case["problem"] == "rm2d":
        items = inputs.rm_batch(seed=shapes, n=n, nx=(128, longest), ny=(32, max(33, longest // 4)))
    else:
        items = inputs.mixed_batch(seed=shapes, n=n, rm_nx=(64, longest), rm_ny=(8, 72))
    rng = np.random.default_rng([seed, 14])
    params, fields = [], []
    for _, p, f in items:
        s = list(p["s"])
        s[6] = s[7] = s[6] * float(rng.uniform(0.9, 1.0))
        params.append(dict(p, s=s))
        fields.append(_stir(p, dict(f, rho=f["rho"] * float(rng.uniform(0.9, 1.1))), rng))
    return params, fields


def _concat(fields, device):
    return [torch.from_numpy(np.concatenate([np.ascontiguousarray(f[k], dtype=np.float64).ravel() for f in fields]))
            .to(device) for k in FIELDS]


def _stability_sets(case, seed):
    rng = np.random.default_rng([seed, 12])
    params, states = inputs.fig2_stability_sets((case["eq_version"],))
    jitter = rng.uniform(0.98, 1.02, size=(len(states), 4))
    states = [tuple(float(v) for v in np.asarray(s) * j) for s, j in zip(states, jitter)]
    return params, states, torch.from_numpy(inputs.wavenumber_grid(case["grid"]))


def _target(rho, seed):
    """The density that an adjoint case's final state is compared with."""
    rng = np.random.default_rng([seed, 13])
    return rho * torch.from_numpy(rng.uniform(0.95, 1.05, size=tuple(rho.shape))).to(rho.device)


def prepare(case, seed):
    device = torch.device("cuda")
    state = {"case": case}
    if case["kind"] == "single":
        p, f = _single_problem(case, seed)
        state["fields"] = [torch.from_numpy(np.ascontiguousarray(f[k])).to(device) for k in FIELDS]
        state["sim"] = lbm.Simulation(p)
    elif case["kind"] == "batch":
        params, fields = _batch_problems(case, seed)
        batch = Batch(params)
        batch.init(fields)
        batch.tune(probe_steps=32, use_cache=False)
        state["batch"] = batch
        state["fields"] = _concat(fields, device)
    elif case["kind"] == "adjoint":
        p, f = _single_problem(case, seed)
        state["params"] = p
        state["fields"] = [torch.from_numpy(np.ascontiguousarray(f[k])).to(device) for k in FIELDS]
        state["log_s"] = torch.tensor([math.log(v) for v in p["s"]], dtype=torch.float64, device=device)
        state["target"] = _target(state["fields"][0], seed)
        if case["api"] == "handle":
            state["adjoint"] = autograd.Adjoint(p, case["steps"])
    else:
        state["params"], state["states"], theta = _stability_sets(case, seed)
        state["theta"] = theta.to(device)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "single":
        sim = state["sim"]
        sim.init(*state["fields"])
        sim.step(case["steps"])
        return sim.moments()
    if case["kind"] == "batch":
        batch = state["batch"]
        # the fields are on the GPU already: the C entry point itself (Batch.init takes host fields)
        lbm._check(lbm.load().lbm_batch_init(batch.handle, *[lbm._ptr(t) for t in state["fields"]]))
        batch.step(case["steps"])
        return batch.moments()
    if case["kind"] == "adjoint":
        if case["api"] == "simulate":
            leaves = [t.detach().requires_grad_() for t in state["fields"]] + [state["log_s"].detach().requires_grad_()]
            out = autograd.simulate(*leaves, state["params"], case["steps"])
            loss = 0.5 * ((out[0] - state["target"]) ** 2).sum()
            grads = torch.autograd.grad(loss, leaves)
            return {"rho": out[0].detach(), "loss": loss.detach(), "fields": list(grads[:4]), "log_s": grads[4]}
        adjoint = state["adjoint"]
        rho = adjoint.forward(*state["fields"])["rho"]
        misfit = rho - state["target"]
        grads, grad_s = adjoint.backward(misfit)
        return {"rho": rho, "loss": 0.5 * (misfit * misfit).sum(), "fields": grads, "log_s": grad_s * state["log_s"].exp()}
    return stability.omega_max(state["params"], state["states"], state["theta"])


# ---------------------------------------------------------------------------
# What a pass cannot do without.
# ---------------------------------------------------------------------------
def work(case):
    if case["kind"] == "single":
        n = case["nx"] * case["ny"]
        # four fields in, five out
        return {"bytes": 9 * 8 * n, "flops": NODE_FLOPS * n * case["steps"]}
    if case["kind"] == "batch":
        n = sum(p["nx"] * p["ny"] for p in _batch_problems(case, 0)[0])
        return {"bytes": 9 * 8 * n, "flops": NODE_FLOPS * n * case["steps"]}
    if case["kind"] == "adjoint":
        n = case["nx"] * case["ny"]
        # four fields and the target in, the final density and four gradients out; the forward sweep once
        return {"bytes": 10 * 8 * n, "flops": (NODE_FLOPS + ADJOINT_FLOPS) * n * case["steps"]}
    points = 4 * case["grid"] ** 2
    return {"bytes": 8 * points + 16 * case["grid"] ** 2, "flops": points * SQUARINGS * SQUARING_FLOPS}


# ---------------------------------------------------------------------------
# The same outputs in plain FP64 torch: dense 16 x 16 transforms, gathered
# neighbours, ghost points appended to the node list. Several problems of any
# shape are advanced as one list of nodes.
# ---------------------------------------------------------------------------
_VX = np.array([1, 0, -1, 0, 1, -1, -1, 1, 2, 0, -2, 0, 2, -2, -2, 2], dtype=np.float64)
_VY = np.array([0, 1, 0, -1, 1, 1, -1, -1, 0, 2, 0, -2, 2, 2, -2, -2], dtype=np.float64)


def _moment_matrix():
    z = _VX + 1j * _VY
    v2 = _VX**2 + _VY**2
    return np.stack([np.ones(16), _VX, _VY, v2 / 2, _VX**2 - _VY**2, _VX * _VY, _VX * v2 / 2, _VY * v2 / 2, (z**3).real,
                     (z**3).imag, v2**2 / 4, (z**4).real, v2 * (_VX**2 - _VY**2), v2 * _VX * _VY, (z**5).real,
                     -(z**5).imag])


_M = _moment_matrix()


def _mirror(sx, sy):
    index = {(a, b): i for i, (a, b) in enumerate(zip(_VX, _VY))}
    return [index[(sx * a, sy * b)] for a, b in zip(_VX, _VY)]


def _equilibrium(rho, ux, uy, T, version):
    """The 16 equilibrium moments (Eqs. 14a-14i and the version's free moments), stacked."""
    jx, jy = rho * ux, rho * uy
    u2 = ux * ux + uy * uy
    e = rho * (T + 0.5 * u2)
    zero = torch.zeros_like(rho)
    h = e / rho + T
    j2 = jx * jx + jy * jy
    w = (6.0 * rho * e - 2.0 * j2) / rho**3
    q = [rho, jx, jy, e, (jx * jx - jy * jy) / rho, jx * jy / rho, h * jx, h * jy, (jx * jx - 3.0 * jy * jy) * jx / rho**2,
         (3.0 * jx * jx - jy * jy) * jy / rho**2, 2.0 * e * e / rho - 0.25 * j2 * j2 / rho**3, zero,
         w * (jx * jx - jy * jy), w * jx * jy, zero, zero]
    if version == 2:
        d = 5.0 * ux * ux - 5.0 * uy * uy
        q[14], q[15] = jx * (-4.0 + 10.0 * T + d), jy * (4.0 - 10.0 * T + d)
    elif version == 3:
        f = torch.stack([rho / (2.0 * math.pi * T) * torch.exp(-((a - ux) ** 2 + (b - uy) ** 2) / (2.0 * T))
                         for a, b in zip(_VX, _VY)])
        top = torch.from_numpy(_M[[11, 14, 15]]).to(rho.device) @ f
        q[11], q[14], q[15] = top[0], top[1], top[2]
    return torch.stack(q)


class _Reference:
    def __init__(self, params, device):
        self.device = device
        self.m = torch.from_numpy(_M).to(device)
        self.mi = torch.from_numpy(np.linalg.inv(_M)).to(device)
        sizes = [p["nx"] * p["ny"] for p in params]
        self.offsets = np.concatenate([[0], np.cumsum(sizes)])
        total = int(self.offsets[-1])
        self.radius = 2 if any(p.get("scheme", 0) for p in params) else 1
        assert self.radius == 1 or len(params) == 1
        source, mode, fixed = [], [], []  # the ghost points: node read, how, and the fixed state
        offsets = [(d, 0) for d in range(1, self.radius + 1)] + [(-d, 0) for d in range(1, self.radius + 1)]
        offsets += [(b, a) for a, b in offsets]
        near = {o: [] for o in offsets}
        wall, fluid, wall_state, self.ghosts = [], [], [], 0
        for p, first in zip(params, self.offsets[:-1]):
            nx, ny, bc = p["nx"], p["ny"], p["bc"]
            x, y = np.meshgrid(np.arange(nx), np.arange(ny))
            for o in offsets:
                gx, gy = x + o[0], y + o[1]
                index = np.empty((ny, nx), dtype=np.int64)
                inside = (gx >= 0) & (gx < nx) & (gy >= 0) & (gy < ny)
                index[inside] = first + (gy * nx + gx)[inside]
                for side, out in enumerate((gx < 0, gx >= nx, gy < 0, gy >= ny)):
                    if not out.any():
                        continue
                    g, n = (gx, nx) if side < 2 else (gy, ny)
                    kind = bc[side]
                    at = g[out]
                    if kind == "periodic":
                        k, how = at % n, 0
                    elif kind == "specular":
                        k = np.clip(-1 - at if side % 2 == 0 else 2 * n - 1 - at, 0, n - 1)
                        how = 1 if side < 2 else 2
                    else:
                        k, how = np.full(at.shape, 0 if side % 2 == 0 else n - 1), 3 if kind == "dirichlet_eq" else 0
                    node = first + (y[out] * nx + k if side < 2 else k * nx + x[out])
                    if how == 0:
                        index[out] = node
                    else:
                        index[out] = total + self.ghosts + np.arange(node.size)
                        self.ghosts += node.size
                        source.append(node)
                        mode.append(np.full(node.size, how))
                        fixed.append(np.tile(np.asarray(p["wall"][side])[:, None], (1, node.size)))
                near[o].append(index.ravel())
            for side, (line, next_) in enumerate(((x == 0, 1), (x == nx - 1, -1), (y == 0, nx), (y == ny - 1, -nx))):
                if bc[side] == "neq_wall":
                    node = first + (y * nx + x)[line]
                    wall.append(node)
                    fluid.append(node + next_)
                    wall_state.append(np.tile(np.asarray(p["wall"][side])[:, None], (1, node.size)))
        tensor = lambda a: torch.from_numpy(np.concatenate(a, axis=-1)).to(device)  # noqa: E731
        self.near = {o: tensor(v) for o, v in near.items()}
        if self.ghosts:
            self.source, self.mode, self.fixed = tensor(source), tensor(mode), tensor(fixed)
        self.wall = tensor(wall) if wall else None
        if wall:
            self.fluid, self.wall_state = tensor(fluid), tensor(wall_state)
        # per-node parameters (one column for a single problem)
        self.versions = sorted({p["eq_version"] for p in params})
        self.problem = None
        if len(params) > 1:
            self.problem = torch.from_numpy(np.repeat(np.arange(len(params)), sizes)).to(device)
        column = lambda v: self.spread(torch.tensor(np.array(v, dtype=np.float64), device=device))  # noqa: E731
        self.dt, self.dx, self.dy = (column([[p[k] for p in params]]) for k in ("dt", "dx", "dy"))
        self.s = column([p["s"] for p in params]).T if self.problem is None else column(np.array([p["s"] for p in params]).T)
        self.sign = column([[{0: 0.0, 1: -1.0, 2: 1.0}[p["modified"]] for p in params]])
        self.on = column([[1.0 if p["modified"] else 0.0 for p in params]])
        self.version = column([[p["eq_version"] for p in params]])
        self.vx, self.vy = (torch.from_numpy(v).to(device)[:, None] for v in (_VX, _VY))

    def spread(self, a):
        return a if self.problem is None else a[:, self.problem]

    def equilibrium(self, rho, ux, uy, T, where=None):
        if len(self.versions) == 1:
            return _equilibrium(rho, ux, uy, T, self.versions[0])
        version = self.version[0] if where is None else self.version[0, where]
        out = _equilibrium(rho, ux, uy, T, self.versions[0])
        for v in self.versions[1:]:
            out = torch.where(version == v, _equilibrium(rho, ux, uy, T, v), out)
        return out

    def initial(self, rho, ux, uy, T):
        return self.mi @ self.equilibrium(rho, ux, uy, T)

    @staticmethod
    def fields(f, m):
        rho, jx, jy, e = m[0] @ f, m[1] @ f, m[2] @ f, m[3] @ f
        ux, uy = jx / rho, jy / rho
        return rho, ux, uy, e / rho - 0.5 * (ux * ux + uy * uy)

    def extended(self, f):
        if not self.ghosts:
            return f
        g = f[:, self.source]
        g = torch.where(self.mode == 1, g[_mirror(-1, 1)], torch.where(self.mode == 2, g[_mirror(1, -1)], g))
        if bool((self.mode == 3).any()):
            # (ghosts of fixed states belong to problems of one version each)
            state = torch.where(self.mode == 3, self.fixed, torch.ones_like(self.fixed))
            g = torch.where(self.mode == 3, self.mi @ self.equilibrium(*state, where=self.source), g)
        return torch.cat([f, g], dim=1)

    def step(self, f, s):
        ext = self.extended(f)
        get = lambda dx, dy: ext[:, self.near[(dx, dy)]]  # noqa: E731
        xp, xm, yp, ym = get(1, 0), get(-1, 0), get(0, 1), get(0, -1)
        rho_e = self.m[0] @ ext
        ux_e, uy_e = (self.m[1] @ ext) / rho_e, (self.m[2] @ ext) / rho_e
        grad = lambda a, d, h: (a[self.near[d]] - a[self.near[(-d[0], -d[1])]]) / (2.0 * h[0])  # noqa: E731
        A = grad(ux_e, (1, 0), self.dx) - grad(uy_e, (0, 1), self.dy)
        B = grad(uy_e, (1, 0), self.dx) + grad(ux_e, (0, 1), self.dy)
        m = self.m @ f
        rho, ux, uy, T = self.fields(f, self.m)
        col = -self.dt * s * (m - self.equilibrium(rho, ux, uy, T))
        g7 = self.on[0] * rho * T * ((s[6] / s[4] - 1.0) * ux * A + (s[6] / s[5] - 1.0) * uy * B)
        g8 = rho * T * (self.on[0] * (s[7] / s[5] - 1.0) * ux * B + self.sign[0] * (s[7] / s[4] - 1.0) * uy * A)
        rows = list(col)
        rows[:4] = [torch.zeros_like(rho)] * 4
        rows[6], rows[7] = rows[6] - self.dt[0] * g7, rows[7] - self.dt[0] * g8
        new = f + self.mi @ torch.stack(rows)
        cx, cy = self.vx * self.dt / self.dx, self.vy * self.dt / self.dy
        if self.radius == 1:
            new = new + 0.5 * (cx * cx - cx) * (xp - f) + 0.5 * (cx * cx + cx) * (xm - f)
            new = new + 0.5 * (cy * cy - cy) * (yp - f) + 0.5 * (cy * cy + cy) * (ym - f)
        else:
            new = new + self.limited(cx, get(-2, 0), xm, f, xp, get(2, 0))
            new = new + self.limited(cy, get(0, -2), ym, f, yp, get(0, 2))
        if self.wall is not None:
            fn = new[:, self.fluid]
            rn, un, vn, tn = self.fields(fn, self.m)
            w = self.wall_state
            fw = fn + self.mi @ (self.equilibrium(rn, w[1], w[2], w[3], where=self.wall)
                                 - self.equilibrium(rn, un, vn, tn, where=self.wall))
            new = new.index_copy(1, self.wall, fw)
        return new

    @staticmethod
    def limited(c, f2m, f1m, f, f1p, f2p):
        minmod = lambda a, b: torch.where(a * b > 0, torch.where(a.abs() < b.abs(), a, b), torch.zeros_like(a))  # noqa: E731
        a = c.abs()
        k = 0.5 * a * (1.0 - a)
        dm, dp = f - f1m, f1p - f
        up = -a * dm - k * (minmod(dp, dm) - minmod(dm, f1m - f2m))
        down = a * dp - k * (minmod(dp, f2p - f1p) - minmod(dm, dp))
        return torch.where(c > 0, up, torch.where(c < 0, down, torch.zeros_like(up)))

    def moments(self, f):
        rho, ux, uy, T = self.fields(f, self.m)
        return {"rho": rho, "ux": ux, "uy": uy, "T": T, "p": rho * T}


def _exact_radius(p, state, theta):
    """|omega|_max in the moment basis by repeated squaring with exact rescaling."""
    device = theta.device
    M, Mi = torch.from_numpy(_M), torch.from_numpy(np.linalg.inv(_M))
    rho, ux, uy, T = (torch.tensor(v, dtype=torch.float64) for v in state)
    conserved = torch.stack([rho, rho * ux, rho * uy, rho * (T + 0.5 * (ux * ux + uy * uy))])

    def of_conserved(c):
        u, v = c[1] / c[0], c[2] / c[0]
        return _equilibrium(c[0], u, v, c[3] / c[0] - 0.5 * (u * u + v * v), p["eq_version"])

    D = torch.zeros(16, 16, dtype=torch.float64)
    D[:, :4] = torch.autograd.functional.jacobian(of_conserved, conserved)
    s = torch.tensor(p["s"], dtype=torch.float64)
    s[:4] = 0.0
    dt, dx, dy = p["dt"], p["dx"], p["dy"]
    eye = torch.eye(16, dtype=torch.float64)
    P0 = eye - dt * s[:, None] * (eye - D)
    cx, cy = torch.from_numpy(_VX) * dt / dx, torch.from_numpy(_VY) * dt / dy
    Bx, By = M @ torch.diag(cx * cx) @ Mi, M @ torch.diag(cy * cy) @ Mi
    Qx, Qy = -M @ torch.diag(cx) @ Mi, -M @ torch.diag(cy) @ Mi
    if p["modified"]:
        du, dv = torch.zeros(16, dtype=torch.float64), torch.zeros(16, dtype=torch.float64)
        du[0], du[1], dv[0], dv[2] = -ux / rho, 1.0 / rho, -uy / rho, 1.0 / rho
        s5, s6, s7, s8 = p["s"][4:8]
        sign = 1.0 if p["modified"] == 2 else -1.0
        rT = rho * T
        # A = i (gx du - gy dv), B = i (gx dv + gy du) with gx = sin tx / dx, gy = sin ty / dy
        a7, b7 = (s7 / s5 - 1.0) * rT * ux, (s7 / s6 - 1.0) * rT * uy
        a8, b8 = sign * (s8 / s5 - 1.0) * rT * uy, (s8 / s6 - 1.0) * rT * ux
        for row, a, b in ((6, a7, b7), (7, a8, b8)):
            Qx[row] -= dt / dx * (a * du + b * dv)
            Qy[row] -= dt / dy * (-a * dv + b * du)
    P0, Bx, By, Qx, Qy = (t.to(device) for t in (P0, Bx, By, Qx, Qy))
    out = []
    for th in theta.split(65536):
        tx, ty = th[:, 0, None, None], th[:, 1, None, None]
        re = (P0 - 2.0 * torch.sin(0.5 * tx) ** 2 * Bx - 2.0 * torch.sin(0.5 * ty) ** 2 * By).contiguous()
        im = (torch.sin(tx) * Qx + torch.sin(ty) * Qy).contiguous()
        total = torch.zeros(len(th), dtype=torch.float64, device=device)
        for j in range(SQUARINGS + 1):
            if j:
                re, im = torch.bmm(re, re) - torch.bmm(im, im), torch.bmm(re, im) + torch.bmm(im, re)
            big = torch.maximum(re.abs().amax((1, 2)), im.abs().amax((1, 2)))
            power = torch.floor(torch.log2(big))
            scale = torch.exp2(-power)[:, None, None]
            re, im = re * scale, im * scale
            total += power * 2.0**-j
        last = torch.log2(torch.maximum(re.abs().amax((1, 2)), im.abs().amax((1, 2))))
        out.append(torch.exp2(total + last * 2.0**-SQUARINGS))
    return torch.cat(out)


def exact(case, seed):
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if case["kind"] == "stability":
        params, states, theta = _stability_sets(case, seed)
        theta = theta.to(device)
        return torch.stack([_exact_radius(p, s, theta) for p, s in zip(params, states)])
    if case["kind"] == "batch":
        params, fields = _batch_problems(case, seed)
        ref = _Reference(params, device)
        f = ref.initial(*_concat(fields, device))
        for _ in range(case["steps"]):
            f = ref.step(f, ref.s)
        return ref.moments(f)
    p, host = _single_problem(case, seed)
    ref = _Reference([p], device)
    fields = [torch.from_numpy(np.ascontiguousarray(host[k])).to(device) for k in FIELDS]
    shape = (case["ny"], case["nx"])
    if case["kind"] == "single":
        f = ref.initial(*[t.reshape(-1) for t in fields])
        for _ in range(case["steps"]):
            f = ref.step(f, ref.s)
        return {k: v.reshape(shape) for k, v in ref.moments(f).items()}
    target = _target(fields[0], seed)
    leaves = [t.requires_grad_() for t in fields]
    log_s = torch.tensor([math.log(v) for v in p["s"]], dtype=torch.float64, device=device).requires_grad_()
    rates = torch.exp(log_s)[:, None]
    f = ref.initial(*[t.reshape(-1) for t in leaves])
    for _ in range(case["steps"]):
        f = torch.utils.checkpoint.checkpoint(ref.step, f, rates, use_reentrant=False)
    rho = ref.moments(f)["rho"].reshape(shape)
    loss = 0.5 * ((rho - target) ** 2).sum()
    grads = torch.autograd.grad(loss, leaves + [log_s])
    return {"rho": rho.detach(), "loss": loss.detach(), "fields": list(grads[:4]), "log_s": grads[4]}
