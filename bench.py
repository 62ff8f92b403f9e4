"""Benchmark of the MRT FD-LBM hot path on one MI355X.

Prints ONE JSON line. The headline workload is the Richtmyer-Meshkov-shaped
problem at 4096 x 1024 nodes (HBM-resident: 2 x 537 MB of distributions, far
beyond the 256 MB Infinity Cache): one step = one time step of every node
(moments, equilibria, relaxation with the energy-flux modification,
back-transform, Lax-Wendroff convection, store). value = MLUPS (million node
updates per second) with the state resident in HBM. The roofline object
prices the step kernel against the 8 TB/s HBM peak with 256 algorithmic
bytes per node update (16 FP64 loads + 16 FP64 stores). Side results: the
1024 x 256 problem itself, the paper's small configurations, and the oracle
timed on the host cores.
"""

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK = 8.0e12  # bytes/s, MI355X HBM3E
BYTES_PER_NODE = 256  # 16 FP64 reads + 16 FP64 writes per node update
ADJ_BYTES_PER_NODE = 384  # adjoint step: lambda^{n+1} and f^n read, lambda^n written (16 FP64 each)
KERNEL_SOURCES = ["paper_1106_0785_amd/csrc/lbm_kernels.h", "paper_1106_0785_amd/csrc/lbm_step.h",
                  "paper_1106_0785_amd/csrc/lbm_node.h", "paper_1106_0785_amd/csrc/lbm_consts.h",
                  "paper_1106_0785_amd/csrc/lbm_fused2.h"]


def kernel_hash():
    h = hashlib.sha256()
    for s in KERNEL_SOURCES:
        with open(os.path.join(ROOT, s), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def time_steps(sim, steps, warmup):
    import torch

    sim.step(warmup)
    torch.cuda.synchronize()
    start = torch.cuda.Event(enable_timing=True)
    stop = torch.cuda.Event(enable_timing=True)
    start.record()
    sim.step(steps)
    stop.record()
    torch.cuda.synchronize()
    return start.elapsed_time(stop) / 1e3  # seconds


VARIANT_KERNELS = {0: "k_step_fused", 1: "k_step_plain", 2: "k_step_window", 3: "k_step_window", 4: "k_step_fused2"}


def run_problem(p, fields, steps, warmup, rows=None, tune=False):
    from paper_1106_0785_amd import lbm

    sim = lbm.Simulation(p)
    if rows:
        sim.set_tile(rows)
    sim.init(**fields)
    tuned = None
    if tune:
        tuned = sim.tune(probe_steps=10)
    t = time_steps(sim, steps, warmup)
    sim.check()
    nodes = p["nx"] * p["ny"]
    variant = sim.variant()
    window = sim.window() if variant == 3 else None
    stores = "nontemporal" if sim.store_mode() else "ordinary"
    if tuned and variant == 4:
        tuned = sim.tile()
    sim.close()
    out = {"seconds": t, "steps": steps, "nodes": nodes, "mlups": nodes * steps / t / 1e6,
           "ms_per_step": 1e3 * t / steps, "gbps": nodes * steps * BYTES_PER_NODE / t / 1e9,
           "kernel": VARIANT_KERNELS[variant]}
    if window:
        out["window_cols"], out["window_rows"], out["window_steps"] = window
    elif tuned:
        out["tile_rows"], out["tile_waves"] = tuned[0], tuned[1]
    if variant in (0, 4):
        out["stores"] = stores
    if variant == 4:
        out["steps_per_launch"] = 2
    return out


def bench_batch(steps, seed=0, n=512, plain=True, two_d=False):
    """The 512-instance uneven batch of lines (two_d: the 96-instance batch
    of 2-D shock/interface problems): K steps of the batched form (autotuned
    schedule, graph replays) against the same K steps of the plain path
    called once per instance (lbm_step on each instance in turn; skipped
    with plain=False)."""
    import torch

    from paper_1106_0785_amd import inputs, lbm
    from paper_1106_0785_amd.batch import Batch

    items = inputs.rm_batch(seed=seed, n=n) if two_d else inputs.batch(seed=seed, n=n)
    b = Batch([p for _, p, _ in items])
    b.init([f for _, _, f in items])
    sched = b.tune(probe_steps=32, use_cache=False)
    nodes = b.total_nodes
    b.step(steps)  # warm-up: graph capture for this step count
    torch.cuda.synchronize()
    b.init([f for _, _, f in items])
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    b.step(steps)
    stop.record()
    torch.cuda.synchronize()
    tb = start.elapsed_time(stop) / 1e3
    b.check()
    # both launch forms of the line instances at the tuned schedule, each
    # captured in a graph: one launch per block of h steps, and one
    # persistent launch per equilibrium version (each chunk waits for its
    # neighbours' previous block)
    forms = {}
    for name, pers in (("per_block", False), ("persistent", True)) if sched["chunks"] else ():
        b.set_persistent(pers)
        b.init([f for _, _, f in items])
        b.step(steps)  # warm-up: graph capture
        torch.cuda.synchronize()
        b.init([f for _, _, f in items])
        start.record()
        b.step(steps)
        stop.record()
        torch.cuda.synchronize()
        t = start.elapsed_time(stop) / 1e3
        b.check()
        forms[name] = {"seconds": t, "mlups": nodes * steps / t / 1e6}
    if forms:
        forms["persistent"]["grid"] = b.persistent()["grid"]
        b.set_persistent(sched["persistent"])
    # per-instance step budgets (seeded, uniform in [K/4, K]): instances stop at their own budget
    rng = np.random.default_rng(seed + 1)
    budgets = [int(v) for v in rng.integers(steps // 4, steps + 1, size=n)]
    b.init([f for _, _, f in items])
    b.set_budgets(budgets)
    b.step(steps)  # warm-up (graph capture)
    torch.cuda.synchronize()
    b.init([f for _, _, f in items])
    start.record()
    b.step(steps)
    stop.record()
    torch.cuda.synchronize()
    tbb = start.elapsed_time(stop) / 1e3
    b.check()
    budget_node_steps = sum(int(p["nx"]) * int(p["ny"]) * k for (_, p, _), k in zip(items, budgets))
    b.close()

    out = {"instances": n, "nodes": nodes, "steps": steps, "batched_seconds": tb,
           "batched_mlups": nodes * steps / tb / 1e6,
           "budgets_seconds": tbb, "budgets_node_steps": budget_node_steps,
           "budgets_mlups": budget_node_steps / tbb / 1e6,
           "schedule": {k: sched[k] for k in ("region", "steps_per_launch", "persistent", "chunks", "tile_rows",
                                              "tiles", "two_step", "tile_rows2", "tiles2")}}
    if forms:
        out["launch_forms"] = forms
    if not plain:
        return out
    sims = []
    for _, p, f in items:
        s = lbm.Simulation(p)
        s.init(**f)
        sims.append(s)
    for s in sims:
        s.step(2)
    torch.cuda.synchronize()
    start.record()
    for s in sims:
        s.step(steps)
    stop.record()
    torch.cuda.synchronize()
    tp = start.elapsed_time(stop) / 1e3
    for s in sims:
        s.check()
        s.close()
    mp = nodes * steps / tp / 1e6
    out.update({"plain_seconds": tp, "plain_mlups": mp, "batched_over_plain": out["batched_mlups"] / mp})
    return out


def bench_adjoint(nx=512, ny=128, steps=2000):
    """Shock/interface problem (512 x 128 x 2000 steps by default; 4096 x
    1024 x 36 steps for the HBM-resident figure): plain forward time against
    the adjoint form's checkpointed forward and its backward sweep (loss =
    half the squared misfit of the final density)."""
    import torch

    from paper_1106_0785_amd import inputs, lbm
    from paper_1106_0785_amd.autograd import Adjoint

    p, fl, meta = inputs.rm(seed=0, nx=nx, ny=ny)
    sim = lbm.Simulation(p)
    sim.init(**fl)
    tf = time_steps(sim, steps, 20)
    sim.check()
    sim.close()

    dev = torch.device("cuda")
    f0 = [torch.from_numpy(np.ascontiguousarray(fl[k])).to(dev) for k in ("rho", "ux", "uy", "T")]
    adj = Adjoint(p, steps)
    adj.forward(*f0)  # warm-up
    adj.backward(torch.ones(ny, nx, dtype=torch.float64, device=dev))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    out = adj.forward(*f0)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    g = out["rho"] - 1.0
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    adj.backward(g)
    torch.cuda.synchronize()
    t3 = time.perf_counter()
    adj.close()
    node_steps = nx * ny * steps
    bwd_bytes = (ADJ_BYTES_PER_NODE + BYTES_PER_NODE) * node_steps
    return {"nodes": nx * ny, "steps": steps, "plain_forward_seconds": tf,
            "adjoint_forward_seconds": t1 - t0, "adjoint_backward_seconds": t3 - t2,
            "backward_over_forward": (t3 - t2) / tf, "forward_plus_backward_over_forward": (t1 - t0 + t3 - t2) / tf,
            "backward_gbps": bwd_bytes / (t3 - t2) / 1e9, "backward_hbm_frac": bwd_bytes / (t3 - t2) / HBM_PEAK,
            "backward_algorithmic_bytes_per_node_step": ADJ_BYTES_PER_NODE + BYTES_PER_NODE}


def traffic_from_profiles(kernel_name, workload):
    """HBM bytes per launch from committed rocprofv3 counter summaries, if
    they were taken on the current kernel source."""
    path = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(path):
        return None
    try:
        d = json.load(open(path))
        e = d.get(workload)
        if e and e.get("kernel_hash") == kernel_hash() and e.get("kernel") == kernel_name:
            return e["bytes_per_launch"]
    except Exception:
        return None
    return None


STAB_FLOPS_PER_SQUARING = 4 * 2 * 16 ** 3  # complex 16x16 product as four real ones


def bench_stability(n=512, squarings=48, reps=5, cpu_points=400):
    """Von Neumann map of the paper's Fig. 2 cases (a)-(d): |omega|_max on an
    n x n wavenumber grid over [0, pi]^2 per case (squarings of G on the FP64
    matrix cores), against the oracle's eigenvalues on a sample of points."""
    import torch

    import oracle.stability as so
    from paper_1106_0785_amd import inputs, stability

    params, states = inputs.fig2_stability_sets((1,))
    th_h = inputs.wavenumber_grid(n)
    th = torch.tensor(th_h, device="cuda")
    stability.omega_max(params, states, th, squarings)  # warm-up
    torch.cuda.synchronize()
    ts = []
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        r = stability.omega_max(params, states, th, squarings)
        e1.record()
        torch.cuda.synchronize()
        ts.append(e0.elapsed_time(e1) / 1e3)
    t = sorted(ts)[len(ts) // 2]
    pts = len(params) * th_h.shape[0]
    flops = pts * squarings * STAB_FLOPS_PER_SQUARING
    out = {"sets": len(params), "points": pts, "squarings": squarings, "seconds": t, "points_per_s": pts / t,
           # of 48 products per point; the powers that become rank one need fewer
           "equivalent_tflops": flops / t / 1e12,
           "max_omega": [float(v) for v in r.max(dim=1).values.cpu()]}
    idx = np.random.default_rng(0).integers(0, th_h.shape[0], size=cpu_points // len(params))
    t0 = time.perf_counter()
    for k in range(len(params)):
        so.omega_max(params[k], states[k], th_h[idx])
    tc = time.perf_counter() - t0
    out["cpu_oracle_points_per_s"] = len(params) * len(idx) / tc
    return out


def copy_ceiling(nx, ny, reps=20):
    """Bandwidth of two plain copies of the distribution layout, as context
    for the roofline: the library's streaming probe (the step kernel's access
    pattern, no arithmetic) and a device-to-device copy (torch copy_)."""
    import torch

    from paper_1106_0785_amd import lbm

    pitch = (nx + 63) // 64 * 64
    n = 16 * ny * pitch
    a = torch.ones(n, dtype=torch.float64, device="cuda")
    b = torch.empty_like(a)
    out = {"bytes_per_copy": 2 * n * 8}
    for name, fn in (("stream_probe", lambda: lbm.lbm_stream_copy(a, b, nx, ny)), ("device_copy", lambda: b.copy_(a))):
        for _ in range(3):
            fn()
        torch.cuda.synchronize()
        ts = []
        for _ in range(reps):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            fn()
            e1.record()
            torch.cuda.synchronize()
            ts.append(e0.elapsed_time(e1) / 1e3)
        t = sorted(ts)[len(ts) // 2]
        out[name + "_gbps"] = 2 * n * 8 / t / 1e9
    del a, b
    return out


def _median_rate(fn, work, reps=3):
    """Median rate (work / s) of `reps` timed calls of fn after one warm-up."""
    fn()
    ts = []
    for _ in range(reps):
        t0 = time.perf_counter()
        fn()
        ts.append(time.perf_counter() - t0)
    return work / sorted(ts)[len(ts) // 2]


def cpu_baseline():
    """The oracle, built -O3 -march=native on this host (the same source as
    the -O2 parity build), timed on samples of the five workloads, on every
    host thread and on one thread, median of three runs after a warm-up:
    thermal Couette 4 x 64 (2000 steps), Sod 2000 x 4 (200 steps), the
    1024 x 256 shock/interface problem (8 steps), 16 instances of the uneven
    batch (100 steps; instances run side by side on the threads), and the
    complex-step run that checks the adjoint (512 x 128, 4 steps in complex
    arithmetic). Rates are node updates per second (MLUPS). value: the
    1024 x 256 sample on every thread."""
    from concurrent.futures import ThreadPoolExecutor

    import oracle
    from paper_1106_0785_amd import inputs

    nt = oracle.max_threads()
    cfg = {}

    def plain(name, p, fl, steps, sample):
        f0 = oracle.init(p, **fl)
        work = p["nx"] * p["ny"] * steps / 1e6
        r_all = _median_rate(lambda: oracle.run(p, f0, steps, nthreads=nt, variant="native"), work)
        r_one = _median_rate(lambda: oracle.run(p, f0, steps, nthreads=1, variant="native"), work)
        cfg[name] = {"mlups_all_threads": r_all, "mlups_1_thread": r_one, "sample": sample}

    pc, flc, _ = inputs.couette(1.0)
    plain("couette_4x64", pc, flc, 2000, "4x64 thermal Couette, 2000 steps")
    pr, flr, _ = inputs.riemann("sod", nx=2000, ny=4)
    plain("riemann_2000x4", pr, flr, 200, "2000x4 Sod tube, 200 steps")
    p3, fl3, _ = inputs.rm(seed=0, nx=1024, ny=256)
    plain("rm_1024x256", p3, fl3, 8, "1024x256 shock/interface problem, 8 steps")

    items = inputs.batch(seed=0, n=512)[::32]
    f0s = [oracle.init(p, **fl) for _, p, fl in items]
    work = sum(p["nx"] * p["ny"] for _, p, _ in items) * 100 / 1e6

    def batch(threads):
        with ThreadPoolExecutor(max_workers=threads) as ex:
            list(ex.map(lambda pf: oracle.run(pf[0], pf[1], 100, nthreads=1, variant="native"),
                        [(p, f) for (_, p, _), f in zip(items, f0s)]))

    cfg["batch_512"] = {"mlups_all_threads": _median_rate(lambda: batch(nt), work),
                        "mlups_1_thread": _median_rate(lambda: batch(1), work),
                        "sample": "16 of the 512 instances (every 32nd), 100 steps each"}

    p5, fl5, _ = inputs.rm(seed=0, nx=512, ny=128)
    rng = np.random.default_rng(21)
    h = 1e-30
    cf = {k: fl5[k] + 1j * h * rng.standard_normal(fl5[k].shape) for k in ("rho", "ux", "uy", "T")}
    fc = oracle.init_complex(p5, cf["rho"], cf["ux"], cf["uy"], cf["T"])
    s_im = h * np.array(p5["s"]) * rng.standard_normal(16)
    work = 512 * 128 * 4 / 1e6
    cfg["adjoint_check_512x128"] = {
        "mlups_all_threads": _median_rate(lambda: oracle.run_complex(p5, fc, 4, s_im=s_im, nthreads=nt,
                                                                     variant="native"), work),
        "mlups_1_thread": _median_rate(lambda: oracle.run_complex(p5, fc, 4, s_im=s_im, nthreads=1,
                                                                  variant="native"), work),
        "sample": "512x128 shock/interface problem, 4 steps in complex arithmetic (one directional derivative)"}
    model = ""
    try:
        with open("/proc/cpuinfo") as fh:
            model = next((l.split(":", 1)[1].strip() for l in fh if l.startswith("model name")), "")
    except OSError:
        pass
    head = cfg["rm_1024x256"]
    return {"value": head["mlups_all_threads"], "unit": "MLUPS", "cores": nt, "kind": "oracle",
            "sample": "1024x256 shock/interface problem, 8 time steps, median of 3 runs, all threads",
            "build": "g++ -O3 -march=native -fopenmp (same source as the -O2 parity build)",
            "value_1_thread": head["mlups_1_thread"], "configs": cfg, "cpu_model": model,
            "logical_cpus": os.cpu_count()}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle baseline")
    ap.add_argument("--quick", action="store_true", help="headline workload only")
    ap.add_argument("--only", choices=["batch", "batch2d", "adjoint", "adjoint_hbm", "limited", "stability", "couette", "riemann"], help="run one side measurement alone and print "
                    "its JSON (for profiling; not the benchmark line)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU: the library runs on a single MI355X (no multi-GPU path); "
              "run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_1106_0785_amd import inputs, lbm

    lbm.load()
    torch.cuda.set_device(0)
    if args.only == "batch":
        print(json.dumps(bench_batch(1000, plain=False)), flush=True)
        return
    if args.only == "batch2d":
        print(json.dumps(bench_batch(200, n=96, plain=False, two_d=True)), flush=True)
        return
    if args.only == "adjoint":
        print(json.dumps(bench_adjoint()), flush=True)
        return
    if args.only == "adjoint_hbm":
        print(json.dumps(bench_adjoint(4096, 1024, 36)), flush=True)
        return
    if args.only == "stability":
        print(json.dumps(bench_stability(reps=2, cpu_points=8)), flush=True)
        return
    if args.only == "couette":
        pc, flc, _ = inputs.couette(1.0)
        print(json.dumps(run_problem(pc, flc, 20000, 100)), flush=True)
        return
    if args.only == "riemann":
        pr, flr, _ = inputs.riemann("sod", nx=2000, ny=4)
        print(json.dumps(run_problem(pr, flr, 20000, 100, tune=True)), flush=True)
        return
    if args.only == "limited":
        pl, fll, _ = inputs.rm(seed=0, nx=4096, ny=1024, width_cells=0.5)
        pl["scheme"] = 1
        print(json.dumps(run_problem(pl, fll, args.steps, args.warmup, tune=True)), flush=True)
        return

    # headline: HBM-resident RM-shaped problem
    nx, ny = 4096, 1024
    p, fl, _ = inputs.rm(seed=0, nx=nx, ny=ny)
    log("headline rm %dx%d: %d warm-up + %d timed steps" % (nx, ny, args.warmup, args.steps))
    head = run_problem(p, fl, args.steps, args.warmup, tune=True)
    extra = {}
    if not args.quick:
        p3, fl3, _ = inputs.rm(seed=0, nx=1024, ny=256)
        log("rm 1024x256")
        extra["rm_1024x256"] = run_problem(p3, fl3, 1000, 50, tune=True)
        pc, flc, _ = inputs.couette(1.0)
        log("couette 4x64")
        extra["couette_4x64"] = run_problem(pc, flc, 2000, 100)
        pr, flr, _ = inputs.riemann("sod", nx=2000, ny=4)
        log("riemann 2000x4")
        extra["riemann_2000x4"] = run_problem(pr, flr, 2000, 100, tune=True)
        pl, fll, _ = inputs.rm(seed=0, nx=nx, ny=ny, width_cells=0.5)
        pl["scheme"] = 1
        log("rm %dx%d, flux-limited scheme, sharp interface" % (nx, ny))
        extra["rm_%dx%d_limited" % (nx, ny)] = run_problem(pl, fll, 100, 10, tune=True)
        log("batch: 512 uneven instances, batched form vs plain path")
        extra["batch_512"] = bench_batch(1000)
        log("batch: 96 uneven 2-D shock/interface instances, batched form vs plain path")
        extra["batch_rm2d_96"] = bench_batch(200, n=96, two_d=True)
        log("adjoint rm 512x128, 2000 steps")
        extra["adjoint_rm_512x128"] = bench_adjoint()
        log("adjoint rm 4096x1024, 36 steps (HBM-resident)")
        extra["adjoint_rm_4096x1024"] = bench_adjoint(4096, 1024, 36)
        log("stability map: Fig. 2 cases, 512 x 512 wavenumbers")
        extra["stability_fig2_512x512"] = bench_stability()

    log("copy ceiling")
    extra["copy_ceiling_%dx%d" % (nx, ny)] = copy_ceiling(nx, ny)
    kernel = head["kernel"]  # the kernel the tuner kept at this size
    workload = "rm_%dx%d" % (nx, ny)
    # algorithmic bytes: 256 per node-step times the node-steps of one launch
    # (one step per launch, or two for the two-step kernel); the launch time
    # is the timed region over its launches (an even step count is all
    # two-step launches)
    spl = head.get("steps_per_launch", 1)
    bytes_per_launch = BYTES_PER_NODE * nx * ny * spl
    launch_s = head["seconds"] / (head["steps"] / spl)
    achieved = bytes_per_launch / launch_s / 1e9
    roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK / 1e9, "unit": "GB/s",
                "frac": round(achieved * 1e9 / HBM_PEAK, 4), "traffic": traffic_from_profiles(kernel, workload),
                "kernel": kernel, "steps_per_launch": spl, "launch_us": round(launch_s * 1e6, 1),
                "algorithmic_bytes_per_launch": bytes_per_launch,
                "tile_rows": head.get("tile_rows"), "tile_waves": head.get("tile_waves"), "stores": head.get("stores")}
    out = {
        "metric": "MLUPS (FP64 node updates/s) and fraction of HBM roofline",
        "value": round(head["mlups"], 1),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(head["ms_per_step"], 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": workload, "nx": nx, "ny": ny, "problem": "planar shock on a perturbed light/heavy "
                   "interface, reflecting x walls, periodic y, Pr 0.71", "parallelism": "single GPU"},
        "roofline": roofline,
        "extra": extra,
        "kernel_hash": kernel_hash(),
    }
    if not args.no_cpu:
        log("cpu baseline (oracle)")
        out["cpu_baseline"] = cpu_baseline()
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
