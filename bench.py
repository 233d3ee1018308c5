#!/usr/bin/env python3
"""Benchmark of the fTWA hot path on one MI355X.

Metric: trajectory x RK4-steps per second on the 198-site honeycomb flake
(10 x 20 brick wall with its two dangling corners trimmed), Neel start,
U/t = 3.3, 32768 trajectories, dt = 0.005/t to T = 20/t (4000 RK4 steps),
records every 10 steps; FP32 trajectories with FP64 ensemble moments, next to
the FP64 run on identical samples and the observable error between them.

One benchmark step is one pass of the whole hot path over the batch:
sampling of rho(0) (Eq. (7) of arXiv:2212.04352), RK4 integration of Eq. (6)
for every trajectory with FP64 moments at every record, and the observables
(Eq. (5), Eq. (10)).  Inputs are generated on the device (nothing crosses
PCIe in the timed region).  Warm-up steps run first; then exactly --steps
steps are timed between device synchronisations.

Prints one JSON line.  `--gpus` above 1 is refused: this build runs on one GPU.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
FP32_VECTOR_PEAK_TFLOPS = 157.3   # published; the dual-issue (packed) FP32 rate
FP32_PLAIN_PEAK_TFLOPS = 78.6     # without packed FP32 (which this build does not emit)
# arithmetic of one stored complex element and Runge-Kutta stage: six neighbour
# sums (8), col - row (2), the t and U factors (4), the U term (4), the stage
# input and accumulator updates (8)
FLOPS_PER_ELEMENT_STAGE = 26


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--traj", type=int, default=None, help="override the trajectory count")
    ap.add_argument("--horizon-steps", type=int, default=None,
                    help="override the number of RK4 steps (default: the full horizon)")
    ap.add_argument("--path", default="auto", choices=["auto", "stream", "resident"])
    ap.add_argument("--config", type=int, default=-1,
                    help="force a resident kernel configuration (default: autotuned)")
    ap.add_argument("--no-autotune", action="store_true",
                    help="skip the configuration autotuner (first fitting configuration)")
    ap.add_argument("--fp64-traj", type=int, default=4096,
                    help="trajectories of the FP64 comparison (the first ones of the batch)")
    ap.add_argument("--fp64-steps", type=int, default=None,
                    help="RK4 steps of the FP64 comparison run (default: full horizon)")
    ap.add_argument("--no-fp64", action="store_true")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-adjoint-checks", action="store_true",
                    help="adjoint workload: skip the FP64 gradient and finite-difference report")
    ap.add_argument("--cpu-traj", type=int, default=96)
    ap.add_argument("--cpu-steps", type=int, default=800)
    ap.add_argument("--workload", default="flake198",
                    choices=["flake198", "torus54", "batch", "adjoint", "sizes", "thermal",
                             "pulse", "longrange", "peierls"],
                    help="flake198: the headline metric (default); torus54: FP32 against FP64 on "
                         "identical samples on the 54-site torus at U/t = 1 and 3.3 (throughput "
                         "and the stated accuracy); batch: the 64-instance mixed "
                         "batch as one graph launch; adjoint: the 54-site gradient workload; "
                         "sizes: resident throughput per lattice size; thermal: sampling of "
                         "thermal (fractional-occupation) starts on the 198-site flake; pulse: "
                         "a time-dependent staggered potential on the 198-site flake; "
                         "longrange: a general density-density interaction on the same; "
                         "peierls: complex time-dependent hopping (a field pulse) on the same")
    ap.add_argument("--sizes", default=None,
                    help="sizes workload: comma-separated site counts to run (default: all of "
                         "12, 54, 96, 150, 198)")
    ap.add_argument("--batch-steps", type=int, default=2000)
    ap.add_argument("--batch-traj", type=int, default=2048)
    ap.add_argument("--sequential", action="store_true",
                    help="batch: also time one ftwa_evolve per instance")
    ap.add_argument("--dtypes", default="f32,f64",
                    help="pulse, longrange, peierls: the precisions to run (comma list)")
    ap.add_argument("--paths", default=None,
                    help="pulse, longrange, peierls: the paths to run (comma list; default "
                         "resident,stream for pulse, stream,auto for the others)")
    ap.add_argument("--lattice", default="flake198", choices=sorted(VARIANT_LATTICES),
                    help="pulse, longrange, peierls: the lattice (flake198: the 198-site flake, "
                         "4096 trajectories by default; torus54: the 3x9 torus, 16384; torus12: "
                         "the 2x3 torus, 65536)")
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="first run one plain device-to-device copy of this many MiB (a "
                         "known-size reference dispatch for HBM byte counters)")
    return ap.parse_args()


KERNEL_SOURCES = {"rk4_resident": ("rk4_resident.h", "resident_config.h", "resident_f32_spin.hip",
                                  "device_common.h", "ftwa_internal.h"),
                  "rk4_stage_stream": ("evolve_stream.hip", "device_common.h", "ftwa_internal.h")}


def kernel_source_hash(kernel: str) -> str:
    """Hash of the source files that define a kernel (its code and argument
    layouts): counters taken on other sources are not reported."""
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2212_04352_amd", "csrc")
    for f in KERNEL_SOURCES[kernel]:
        with open(os.path.join(csrc, f), "rb") as fh:
            h.update(f.encode() + fh.read())
    return h.hexdigest()[:16]


def counter_record(kernel: str, dtype: str, config=None):
    """The committed rocprofv3 counter record of this kernel configuration
    (profiles/hbm_counters.json), if it was taken on the current kernel
    sources; else None."""
    path = os.path.join(ROOT, "profiles", "hbm_counters.json")
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        data = json.load(fh)
    rec = data.get(f"{kernel}:{dtype}:{config}")
    if not rec or rec.get("source_hash") != kernel_source_hash(kernel):
        return None
    return rec


def counter_traffic(kernel: str, dtype: str, traj_steps_per_launch: float, config=None):
    """HBM bytes per launch of this run from committed rocprofv3 FETCH_SIZE /
    WRITE_SIZE runs of the same kernel configuration (calibrated against a plain
    copy of known size, scaled from the counter run's trajectory-steps to this
    launch's), if the counters were taken on the current kernel sources; else
    None."""
    rec = counter_record(kernel, dtype, config)
    if not rec or "bytes_per_traj_step" not in rec:
        return None
    return rec["bytes_per_traj_step"] * traj_steps_per_launch


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def run_pass(ft, torch, W, lat, n0, dtype, M, n_steps, path, seed, workspace, config=-1):
    """One pass of the hot path; returns (problem, workspace, timing, observables)."""
    prob = ft.Problem.allocate(lat, W.U, M, n0, dtype)
    ft.sample(prob, seed)
    timing = ft.new_timing()
    workspace = ft.evolve(prob, W.dt, n_steps, W.record_every, path=path, workspace=workspace,
                          timing=timing, config=config)
    obs = ft.observables(prob)
    return prob, workspace, timing, obs


def resolved_path(ft, lat, dtype, path):
    """The path ftwa_evolve takes for this lattice and dtype under `path`."""
    if path != "auto":
        return path
    import torch
    prob = ft.Problem.allocate(lat, 0.0, 1, [0.0] * (2 * lat.N), dtype)
    try:
        ft.evolve(prob, 0.0, 0, 1, path="resident")
        return "resident"
    except ft.FtwaError:
        return "stream"
    finally:
        del prob, torch


def host_cpus():
    """(threads the oracle may use, the host's CPU count, the CPU model).  The
    threads are every CPU this process may run on (its affinity mask), within
    OMP_NUM_THREADS when that is set (the GPU host gives one GPU's job a share
    of its CPUs that way)."""
    total = os.cpu_count() or 1
    try:
        avail = len(os.sched_getaffinity(0))
    except AttributeError:
        avail = total
    omp = os.environ.get("OMP_NUM_THREADS", "")
    threads = min(avail, int(omp)) if omp.isdigit() and int(omp) > 0 else avail
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return threads, total, model


def cpu_baseline(W, n_traj, n_steps):
    import numpy as np
    import oracle
    threads, total, model = host_cpus()
    oracle.set_num_threads(threads)
    lat = oracle.Lattice(W.kind, W.a, W.b)
    n0 = oracle.fock_start(lat, W.start, W.seed)
    rho0 = oracle.sample(lat, n0, W.seed, n_traj)
    t0 = time.perf_counter()
    oracle.evolve(lat, W.U, rho0, W.dt, n_steps, W.record_every, precision="f64")
    dt = time.perf_counter() - t0
    del np
    return {"value": n_traj * n_steps / dt, "unit": "trajectory*RK4-steps/s", "cores": threads,
            "host_cpus": total, "cpu_model": model, "kind": "oracle",
            "sample": f"first {n_traj} trajectories x {n_steps} RK4 steps of the same workload, "
                      f"FP64, {dt:.1f} s"}


def run_torus54(args):
    """The 54-site torus (3 x 9 cells), random half-filled Fock start,
    16384 trajectories, dt = 0.01 to T = 20, at U/t = 1 and 3.3: FP64 and FP32
    on identical samples, their throughput, and the FP32 accuracy against
    FP64 (observable error against time; the stated contract of the FP32 form:
    1e-4 up to t32(U), statistical equivalence after)."""
    import numpy as np
    import torch
    import paper_2212_04352_amd as ft
    from workloads import FP32_HORIZON, MID_TORUS as W, fp32_contract
    lat = ft.Lattice(W.kind, W.a, W.b, W.t_hop)
    n0 = lat.fock_start(W.start, W.seed)
    M = args.traj or W.n_traj
    steps = args.horizon_steps or W.n_steps
    times = np.arange(steps // W.record_every + 1) * W.record_every * W.dt
    rows = []
    for U in (1.0, 3.3):
        runs = {}
        for dtype in ("f64", "f32"):
            p = ft.Problem.allocate(lat, U, M, n0, dtype)
            ft.sample(p, W.seed)
            ws = ft.evolve(p, W.dt, 20, W.record_every)  # warm-up
            ft.sample(p, W.seed)
            timing = ft.new_timing()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ft.evolve(p, W.dt, steps, W.record_every, workspace=ws, timing=timing)
            torch.cuda.synchronize()
            el = time.perf_counter() - t0
            n, C, _ = ft.observables(p)
            runs[dtype] = {"value": M * steps / el, "seconds": el,
                           "kernel_value": timing["work"].value / (timing["ms"].value * 1e-3),
                           "n": n.cpu().numpy(), "C": C.cpu().numpy(),
                           "S1": p.S1.cpu().numpy(), "S2": p.S2.cpu().numpy()}
            log(f"torus54 U={U} {dtype}: {M * steps / el:.3e} traj-steps/s")
            del p, ws
        r32, r64 = runs["f32"], runs["f64"]
        t32 = FP32_HORIZON[U]
        contract = fp32_contract(r32["n"], r32["C"], r64["n"], r64["C"], r64["S1"], r64["S2"],
                                 M, times, t32)
        dn = np.abs(r32["n"] - r64["n"]).max(axis=1)
        D = r64["n"].shape[1]
        off = ~np.eye(D, dtype=bool)
        dC = np.abs(r32["C"] - r64["C"])[:, off].max(axis=1)
        curve = {f"t<={T}": {"max_abs_dn": float(dn[times <= T + 1e-9].max()),
                             "max_abs_dC": float(dC[times <= T + 1e-9].max())}
                 for T in (2, 4, 6, 8, 10, 12, 14, 16, 18, 20)}
        rows.append({"U": U, "fp64": {k: r64[k] for k in ("value", "seconds", "kernel_value")},
                     "fp32": {k: r32[k] for k in ("value", "seconds", "kernel_value")},
                     "fp32_over_fp64": r32["value"] / r64["value"], "error_vs_t": curve,
                     "contract": contract})
        log(f"torus54 U={U}: FP32/FP64 {r32['value'] / r64['value']:.2f}, contract "
            f"{'holds' if contract['holds'] else 'FAILS'} (t32 = {t32})")
    print(json.dumps({
        "metric": "trajectory*RK4-steps/s at N=54, FP32 vs FP64 on identical samples, "
                  "with the FP32 observable error",
        "unit": "trajectory*RK4-steps/s", "rows": rows,
        "config": {"workload": W.name, "lattice": "torus 3x9, N=54", "start": "random half filling",
                   "trajectories": M, "dt": W.dt, "rk4_steps": steps,
                   "record_every": W.record_every, "moments": "f64"}}))
    lat.close()


def run_batch(args):
    """The mixed batch: 64 instances (hex flakes of 24/54/96/150 sites and the
    198-site flake, U/t on [0, 4], random Fock starts), FP32, integrated by one
    graph launch of the persistent per-configuration kernels."""
    import torch
    import paper_2212_04352_amd as ft
    from workloads import BATCH_SEED, batch_instances
    specs = batch_instances(n_traj=args.batch_traj)
    lats = {}
    probs = []
    for d in specs:
        key = (d["kind"], d["a"], d["b"])
        if key not in lats:
            lats[key] = ft.Lattice(*key)
        lat = lats[key]
        p = ft.Problem.allocate(lat, d["U"], d["n_traj"],
                                lat.fock_start("random", BATCH_SEED, d["instance"]), "f32",
                                instance=d["instance"])
        ft.sample(p, BATCH_SEED)
        probs.append(p)
    steps = args.batch_steps
    cfgs = ft.autotune(probs, probe_steps=10)
    log(f"batch: {len(probs)} instances, autotuned configurations {sorted(set(cfgs))}")
    work = sum(p.n_traj for p in probs) * steps
    g = ft.EvolveGraph(probs, 0.01, steps, 10)
    log("batch: graph captured; warm-up launch")
    g.launch()
    g.check()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        g.launch()
    torch.cuda.synchronize()
    el = (time.perf_counter() - t0) / args.steps
    g.check()
    out = {"metric": "trajectory*RK4-steps/s, mixed 64-instance batch, one graph launch",
           "value": work / el, "unit": "trajectory*RK4-steps/s", "seconds_per_launch": el,
           "dtype": "f32", "data": "synthetic",
           "config": {"workload": "batch64", "instances": len(probs),
                      "trajectories_per_instance": args.batch_traj, "rk4_steps": steps,
                      "dt": 0.01, "record_every": 10,
                      "sites": sorted(set(p.lat.N for p in probs)),
                      "configurations": sorted(set(cfgs))}}
    g.close()
    # per configuration group: its instances alone through one ftwa_evolve,
    # kernel time by HIP events, and the byte-equivalent rate of its state
    # traffic (one read and one write of both FP32 spin blocks per
    # trajectory-step) against 8 TB/s
    groups = {}
    for p, c in zip(probs, cfgs):
        groups.setdefault(c, []).append(p)
    rows, total_bytes = [], 0.0
    for c, ps in sorted(groups.items()):
        for p in ps:
            ft.sample(p, BATCH_SEED)
        timing = ft.new_timing()
        torch.cuda.synchronize()
        ft.evolve(ps, 0.01, steps, 10, timing=timing)
        torch.cuda.synchronize()
        ms = timing["ms"].value
        gbytes = sum(p.n_traj * 2 * 2 * p.lat.N ** 2 * 4 for p in ps) * steps
        total_bytes += gbytes
        rows.append({"configuration": c, "instances": len(ps),
                     "sites": sorted(set(p.lat.N for p in ps)),
                     "trajectories": sum(p.n_traj for p in ps), "kernel_ms": ms,
                     "trajectory_steps_per_s": sum(p.n_traj for p in ps) * steps / (ms * 1e-3),
                     "byte_equivalent_GBps": gbytes / (ms * 1e-3) / 1e9})
    out["groups"] = rows
    out["roofline"] = {"bound": "hbm", "achieved": total_bytes / el / 1e9, "peak": HBM_PEAK_GBS,
                       "unit": "GB/s", "frac": total_bytes / el / 1e9 / HBM_PEAK_GBS,
                       "note": "byte-equivalent rate of the batch's algorithmic state traffic "
                               "over the graph launch (the resident kernels keep the state on "
                               "chip)"}
    if args.sequential:
        for p in probs:
            ft.sample(p, BATCH_SEED)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for p in probs:
            ft.evolve(p, 0.01, steps, 10)
        torch.cuda.synchronize()
        es = time.perf_counter() - t0
        out["sequential"] = {"value": work / es, "seconds": es,
                             "note": "one ftwa_evolve per instance"}
    print(json.dumps(out))


def run_adjoint(args):
    """The gradient workload: 54-site torus, 4096 trajectories, FP32, 2000
    steps with checkpoints every 50; loss = sum (nbar(t_r) - target)^2 with the
    target from the forward pass at U/t = 3.3, gradient at U/t = 2.5."""
    import torch
    import paper_2212_04352_amd as ft
    from workloads import ADJOINT_54 as W
    from paper_2212_04352_amd.autodiff import OccupationSpec, occupations
    lat = ft.Lattice(W.kind, W.a, W.b, W.t_hop)
    steps = args.horizon_steps or W.n_steps
    spec = OccupationSpec(W.kind, W.a, W.b, lat.fock_start(W.start, W.seed), seed=W.seed,
                          n_traj=W.n_traj, dt=W.dt, n_steps=steps,
                          record_every=W.record_every, dtype="f32", ckpt_every=50)
    f64 = torch.float64
    dev = torch.device("cuda")
    zero = torch.zeros((2, lat.N), dtype=f64, device=dev)
    with torch.no_grad():
        target = occupations(torch.tensor(3.3, dtype=f64), torch.tensor(W.t_hop, dtype=f64),
                             zero, spec)
    U = torch.tensor(W.U, dtype=f64, requires_grad=True)
    t = torch.tensor(W.t_hop, dtype=f64, requires_grad=True)
    delta = torch.zeros(lat.N, dtype=f64, device=dev, requires_grad=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    nbar = occupations(U, t, delta.expand(2, lat.N), spec)
    loss = torch.sum((nbar - target) ** 2)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    gU, gt, gd = torch.autograd.grad(loss, (U, t, delta))
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    work = W.n_traj * steps
    g32 = np.concatenate([[float(gU), float(gt)], gd.detach().cpu().numpy()])
    checks = {} if args.no_adjoint_checks else adjoint_checks(W, lat, steps, g32)
    print(json.dumps({
        "metric": "adjoint gradient, 54-site torus",
        "forward_seconds": t1 - t0, "backward_seconds": t2 - t1,
        "backward_over_forward": (t2 - t1) / (t1 - t0),
        "forward_value": work / (t1 - t0), "backward_value": work / (t2 - t1),
        "unit": "trajectory*RK4-steps/s", "dtype": "f32 state, f64 gradient sums",
        "loss": float(loss.detach()), "dL_dU": float(gU), "dL_dt": float(gt),
        "dL_ddelta_norm": float(gd.norm()), **checks,
        "config": {"workload": W.name, "trajectories": W.n_traj, "rk4_steps": steps,
                   "dt": W.dt, "ckpt_every": 50, "U_eval": W.U, "U_target": 3.3}}))


def _occupation_grad(W, lat, steps, dtype, U_eval, t_eval=None, delta=None):
    """(loss, [dL/dU, dL/dt, dL/ddelta]) of the gradient workload's loss in
    `dtype`, target from the U/t = 3.3 run in the same dtype."""
    import torch
    from paper_2212_04352_amd.autodiff import OccupationSpec, occupations
    spec = OccupationSpec(W.kind, W.a, W.b, lat.fock_start(W.start, W.seed), seed=W.seed,
                          n_traj=W.n_traj, dt=W.dt, n_steps=steps,
                          record_every=W.record_every, dtype=dtype, ckpt_every=50)
    f64 = torch.float64
    dev = torch.device("cuda")
    zero = torch.zeros((2, lat.N), dtype=f64, device=dev)
    with torch.no_grad():
        target = occupations(torch.tensor(3.3, dtype=f64), torch.tensor(W.t_hop, dtype=f64),
                             zero, spec)
    U = torch.tensor(U_eval, dtype=f64, requires_grad=True)
    t = torch.tensor(W.t_hop if t_eval is None else t_eval, dtype=f64, requires_grad=True)
    d = torch.zeros(lat.N, dtype=f64, device=dev) if delta is None else delta.clone()
    d.requires_grad_(True)
    loss = torch.sum((occupations(U, t, d.expand(2, lat.N), spec) - target) ** 2)
    gU, gt, gd = torch.autograd.grad(loss, (U, t, d))
    return float(loss.detach()), np.concatenate([[float(gU), float(gt)],
                                                 gd.detach().cpu().numpy()])


def adjoint_checks(W, lat, steps, g32):
    """The accuracy report of the gradient workload: the FP32 gradient against
    the FP64 one at the full size and horizon (reported, not asserted: at
    T = 20 the chaotic sensitivity amplifies rounding), and central finite
    differences (h = 1e-6, FP64) of the loss against the FP64 adjoint at
    T = 5 along U, t and one random direction of the per-site offsets."""
    import torch
    _, g64 = _occupation_grad(W, lat, steps, "f64", W.U)
    scale = float(np.max(np.abs(g64)))
    out = {"fp32_vs_fp64_adjoint": {
        "T": steps * W.dt, "max_abs_diff_over_max_abs": float(np.max(np.abs(g32 - g64))) / scale,
        "dL_dU": [float(g32[0]), float(g64[0])], "dL_dt": [float(g32[1]), float(g64[1])],
        "rel_dU": abs(g32[0] - g64[0]) / abs(g64[0]), "rel_dt": abs(g32[1] - g64[1]) / abs(g64[1]),
        "rel_ddelta_norm": float(np.linalg.norm(g32[2:] - g64[2:]) / np.linalg.norm(g64[2:]))}}
    s5 = min(steps, 500)
    _, g = _occupation_grad(W, lat, s5, "f64", W.U)
    h = 1e-6
    v = np.random.default_rng(W.seed).standard_normal(lat.N)
    vt = torch.from_numpy(v).cuda()

    spec5, target5 = _fd_setup(W, lat, s5)

    def L(dU=0.0, dt=0.0, dd=0.0):
        with torch.no_grad():
            return _fd_loss(spec5, target5, lat, W.U + dU, W.t_hop + dt, dd * vt)
    fd = [(L(dU=h) - L(dU=-h)) / (2 * h), (L(dt=h) - L(dt=-h)) / (2 * h),
          (L(dd=h) - L(dd=-h)) / (2 * h)]
    ad = [g[0], g[1], float(np.dot(g[2:], v))]
    out["finite_difference_fp64"] = {
        "T": s5 * W.dt, "h": h, "directions": ["U", "t", "random offset direction"],
        "adjoint": ad, "central_difference": fd,
        "rel_err": [abs(a - f) / max(abs(a), 1e-300) for a, f in zip(ad, fd)]}
    return out


def _fd_setup(W, lat, steps):
    """FP64 occupation spec of the finite-difference check and its target."""
    import torch
    from paper_2212_04352_amd.autodiff import OccupationSpec, occupations
    spec = OccupationSpec(W.kind, W.a, W.b, lat.fock_start(W.start, W.seed), seed=W.seed,
                          n_traj=W.n_traj, dt=W.dt, n_steps=steps,
                          record_every=W.record_every, dtype="f64", ckpt_every=50)
    f64 = torch.float64
    zero = torch.zeros((2, lat.N), dtype=f64, device=torch.device("cuda"))
    with torch.no_grad():
        target = occupations(torch.tensor(3.3, dtype=f64), torch.tensor(W.t_hop, dtype=f64),
                             zero, spec)
    return spec, target


def _fd_loss(spec, target, lat, U, t, delta):
    import torch
    from paper_2212_04352_amd.autodiff import occupations
    f64 = torch.float64
    nbar = occupations(torch.tensor(U, dtype=f64), torch.tensor(t, dtype=f64),
                       delta.expand(2, lat.N), spec)
    return float(torch.sum((nbar - target) ** 2))


def run_sizes(args):
    """Resident-kernel throughput per lattice size (FP32 and FP64), autotuned."""
    import torch
    import paper_2212_04352_amd as ft
    rows = []
    wanted = {int(x) for x in args.sizes.split(",")} if args.sizes else None
    for kind, a, b, n in [("torus", 2, 3, 12), ("torus", 3, 9, 54), ("hex", 4, 0, 96),
                          ("hex", 5, 0, 150), ("armchair", 10, 20, 198)]:
        if wanted is not None and n not in wanted:
            continue
        lat = ft.Lattice(kind, a, b)
        for dtype in ("f32", "f64"):
            M = 16384 if lat.N <= 54 else 8192
            steps = 400
            p = ft.Problem.allocate(lat, 3.3, M, lat.fock_start("neel"), dtype)
            ft.sample(p, 7)
            cfg = ft.autotune(p, probe_steps=10)[0]
            ft.evolve(p, 0.005, 20, 10)
            timing = ft.new_timing()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ft.evolve(p, 0.005, steps, 10, timing=timing)
            torch.cuda.synchronize()
            el = time.perf_counter() - t0
            rows.append({"lattice": f"{kind} {a}x{b}", "N": lat.N, "dtype": dtype,
                         "configuration": cfg, "trajectories": M, "rk4_steps": steps,
                         "value": M * steps / el,
                         "kernel_value": timing["work"].value / (timing["ms"].value * 1e-3)})
            log(f"{kind} N={lat.N} {dtype}: config {cfg}, {M * steps / el:.3e} traj-steps/s")
            del p
    print(json.dumps({"metric": "trajectory*RK4-steps/s by lattice size (autotuned path)",
                      "unit": "trajectory*RK4-steps/s", "rows": rows}))


def run_thermal(args):
    """Thermal initial states on the 198-site flake: ftwa_sample_thermal of
    32768 trajectories (fractional occupations), its rate against the HBM
    roofline of the sampler's output, then 400 FP32 RK4 steps from them."""
    import numpy as np
    import torch
    import paper_2212_04352_amd as ft
    lat = ft.Lattice("armchair", 10, 20)
    N = lat.N
    M = args.traj or 32768
    rng = np.random.default_rng(12)
    n0 = rng.uniform(0.2, 0.8, size=(2, N))  # a seeded fractional filling
    p = ft.Problem.allocate(lat, 3.3, M, n0, "f32")
    P = N * (N + 1) // 2
    ft.sample(p, 9, thermal=True)  # warm-up
    torch.cuda.synchronize()
    reps = 5
    t0 = time.perf_counter()
    for _ in range(reps):
        ft.sample(p, 9, thermal=True)
    torch.cuda.synchronize()
    ts = (time.perf_counter() - t0) / reps
    out_bytes = 2 * P * M * 8  # FP32 complex output, the sampler's only HBM traffic
    steps = args.horizon_steps or 400
    ft.autotune(p, probe_steps=50)
    timing = ft.new_timing()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ft.evolve(p, 0.005, steps, 10, timing=timing)
    torch.cuda.synchronize()
    te = time.perf_counter() - t1
    log(f"thermal: sample {ts * 1e3:.2f} ms ({out_bytes / ts / 1e9:.0f} GB/s), "
        f"evolve {M * steps / te:.3e} traj-steps/s")
    print(json.dumps({
        "metric": "thermal initial states, 198-site flake: sampling rate and FP32 evolution",
        "sample_seconds": ts, "sample_elements_per_s": 2 * P * M / ts,
        "sample_roofline": {"bound": "hbm", "achieved": out_bytes / ts / 1e9,
                            "peak": HBM_PEAK_GBS, "unit": "GB/s",
                            "frac": out_bytes / ts / 1e9 / HBM_PEAK_GBS},
        "evolve_value": M * steps / te, "unit": "trajectory*RK4-steps/s",
        "config": {"workload": "flake198_thermal", "trajectories": M, "rk4_steps": steps,
                   "occupations": "uniform on [0.2, 0.8], seeded", "dtype": "f32"}}))


# Lattices of the pulse, longrange and peierls workloads: (kind, a, b), the
# default trajectory count, and a name for the metric.
VARIANT_LATTICES = {
    "flake198": (("armchair", 10, 20), 4096, "198-site flake"),
    "torus54": (("torus", 3, 9), 16384, "54-site torus"),
    "torus12": (("torus", 2, 3), 65536, "12-site torus"),
}


def variant_lattice(ft, args):
    (kind, a, b), m, name = VARIANT_LATTICES[args.lattice]
    return ft.Lattice(kind, a, b), args.traj or m, name


def run_pulse(args):
    """A time-dependent staggered potential on the 198-site flake (the
    external-potential term of Eq. (6)): V_i(t) = A(t) (+1 on one sublattice,
    -1 on the other), A a Gaussian pulse with a carrier; 4096 trajectories x
    400 steps, FP32 and FP64 on the resident kernels (FP32 spin split, FP64
    split kernel) and on the stream kernels, each with and without the
    potential (the cost of the term).  --lattice torus54: the same on the
    3x9 torus (16384 trajectories; the shared-block tiles' variant)."""
    import numpy as np
    import torch
    import paper_2212_04352_amd as ft
    lat, M, lname = variant_lattice(ft, args)
    N = lat.N
    steps = args.horizon_steps or 400
    dt = 0.005
    tau = np.arange(2 * steps + 1) * dt / 2
    env = 1.0 * np.exp(-((tau - 0.5) / 0.2) ** 2) * np.cos(6.0 * tau)
    sub = np.asarray(lat.sub, dtype=np.float64)
    v = 1.0 - 2.0 * sub
    rows = []
    runs = [(d, q) for d in args.dtypes.split(",")
            for q in (args.paths or "resident,stream").split(",")]
    for dtype, path in runs:
        for with_pot in (False, True):
            p = ft.Problem.allocate(lat, 3.3, M, lat.fock_start("neel"), dtype)
            if with_pot:
                p.v_site = torch.from_numpy(v).cuda()
                p.v_env = torch.from_numpy(env).cuda()
            ft.sample(p, 5)
            ws = ft.evolve(p, dt, 2, 1, path=path)  # warm-up (the envelope's first samples)
            ft.sample(p, 5)
            timing = ft.new_timing()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ft.evolve(p, dt, steps, 10, path=path, workspace=ws, timing=timing)
            torch.cuda.synchronize()
            el = time.perf_counter() - t0
            kernel_s = timing["ms"].value / 1e3
            word = 4 if dtype == "f32" else 8
            alg = 2 * 2 * N * N * word * M * steps  # one read + one write of the state per step
            rows.append({"dtype": dtype, "path": path, "potential": with_pot,
                         "value": M * steps / el,
                         "kernel_value": M * steps / kernel_s,
                         "roofline": {"bound": "hbm", "achieved": alg / kernel_s / 1e9,
                                      "peak": HBM_PEAK_GBS, "unit": "GB/s",
                                      "frac": alg / kernel_s / 1e9 / HBM_PEAK_GBS}})
            log(f"pulse: {dtype} {path} potential={with_pot}: {M * steps / el:.3e} traj-steps/s")
            del p, ws
    print(json.dumps({
        "metric": f"trajectory*RK4-steps/s with a time-dependent staggered potential, {lname}",
        "unit": "trajectory*RK4-steps/s", "rows": rows,
        "config": {"workload": f"{args.lattice}_pulse", "trajectories": M, "rk4_steps": steps, "dt": dt,
                   "envelope": "exp(-((t-0.5)/0.2)^2) cos(6t)",
                   "profile": "+1 / -1 by sublattice"}}))


def run_longrange(args):
    """A general density-density interaction on the 198-site flake: u_ii = 3.3,
    u_ij = exp(-d_ij) / 2 between sites (d_ij the graph distance, a screened
    tail), FP32 and FP64, 4096 trajectories x 400 steps, on the stream kernels
    and on the automatic path (the general-interaction variants of the FP32
    spin-split and FP64 split resident kernels), next to the on-site run of
    the same paths.  --lattice torus54: the same on the 3x9 torus (16384
    trajectories; the shared-block tiles' variant)."""
    import numpy as np
    import torch
    from collections import deque
    import paper_2212_04352_amd as ft
    lat, M, lname = variant_lattice(ft, args)
    N = lat.N
    dist = np.full((N, N), np.inf)
    for r in range(N):  # breadth-first graph distances
        dist[r, r] = 0
        q = deque([r])
        while q:
            x = q.popleft()
            for y in lat.nbr[x][:lat.deg[x]]:
                if dist[r, y] == np.inf:
                    dist[r, y] = dist[r, x] + 1
                    q.append(y)
    u = 0.5 * np.exp(-dist)
    np.fill_diagonal(u, 3.3)
    steps = args.horizon_steps or 400
    rows = []
    for dtype in args.dtypes.split(","):
        for path in (args.paths or "stream,auto").split(","):
            for general in (False, True):
                p = ft.Problem.allocate(lat, 3.3, M, lat.fock_start("neel"), dtype)
                if general:
                    p.u_mat = torch.from_numpy(u).cuda()
                ft.sample(p, 5)
                ws = ft.evolve(p, 0.005, steps, 10, path=path)  # warm-up, workspace
                ft.sample(p, 5)
                timing = ft.new_timing()
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                ft.evolve(p, 0.005, steps, 10, path=path, workspace=ws, timing=timing)
                torch.cuda.synchronize()
                el = time.perf_counter() - t0
                rows.append({"dtype": dtype, "path": path,
                             "interaction": "general" if general else "on-site",
                             "value": M * steps / el,
                             "kernel_value": timing["work"].value / (timing["ms"].value * 1e-3)})
                log(f"longrange: {dtype} {path} general={general}: {M * steps / el:.3e} "
                    f"traj-steps/s")
                del p, ws
    print(json.dumps({
        "metric": f"trajectory*RK4-steps/s with a general density-density interaction, {lname}",
        "unit": "trajectory*RK4-steps/s", "rows": rows,
        "config": {"workload": f"{args.lattice}_longrange", "trajectories": M, "rk4_steps": steps,
                   "dt": 0.005, "paths": ["stream", "auto"],
                   "interaction": "u_ii = 3.3, u_ij = exp(-graph distance) / 2"}}))


def run_peierls(args):
    """Complex time-dependent hopping on the 198-site flake: a field pulse
    j_ik(tau) = t exp(i (x_k - x_i) B(tau)), x the graph distance from site 0
    (a stand-in for the coordinate along the field), B(tau) = 0.5 sin(2 tau),
    tables at half steps; FP32 and FP64, 4096 trajectories x 400 steps, on the
    stream kernels and on the automatic path (the complex-hopping variants of
    the FP32 spin-split and FP64 split resident kernels), next to real
    hopping on the same paths.  --lattice torus54: the same on the 3x9 torus
    (16384 trajectories; the shared-block tiles' variant)."""
    import numpy as np
    import torch
    from collections import deque
    import paper_2212_04352_amd as ft
    lat, M, lname = variant_lattice(ft, args)
    N = lat.N
    x = np.full(N, -1.0)
    x[0] = 0
    q = deque([0])
    while q:  # breadth-first graph distance from site 0
        a = q.popleft()
        for b in lat.nbr[a][:lat.deg[a]]:
            if x[b] < 0:
                x[b] = x[a] + 1
                q.append(b)
    steps = args.horizon_steps or 400
    dt = 0.005
    Bh = 0.5 * np.sin(2.0 * 0.5 * dt * np.arange(2 * steps + 1))
    nbr = lat.nbr.astype(np.int64)
    ii = np.arange(N)[:, None]
    fwd = ii < nbr  # the direction i < k carries exp(i d B), the other its conjugate
    d = np.where(fwd, x[nbr] - x[ii], x[ii] - x[nbr])
    z = np.exp(1j * d[None] * Bh[:, None, None])
    w = np.where(fwd[None], z, np.conj(z))
    w[:, np.arange(3)[None, :] >= lat.deg[:, None]] = 0
    rows = []
    for dtype in args.dtypes.split(","):
        for path in (args.paths or "stream,auto").split(","):
            for peierls in (False, True):
                p = ft.Problem.allocate(lat, 3.3, M, lat.fock_start("neel"), dtype)
                if peierls:
                    p.hop_w = torch.from_numpy(np.ascontiguousarray(w)).cuda()
                ft.sample(p, 5)
                ws = ft.evolve(p, dt, steps, 10, path=path)  # warm-up, workspace
                ft.sample(p, 5)
                timing = ft.new_timing()
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                ft.evolve(p, dt, steps, 10, path=path, workspace=ws, timing=timing)
                torch.cuda.synchronize()
                el = time.perf_counter() - t0
                rows.append({"dtype": dtype, "path": path,
                             "hopping": "complex" if peierls else "real",
                             "value": M * steps / el,
                             "kernel_value": timing["work"].value / (timing["ms"].value * 1e-3)})
                log(f"peierls: {dtype} {path} complex={peierls}: {M * steps / el:.3e} traj-steps/s")
                del p, ws
    print(json.dumps({
        "metric": f"trajectory*RK4-steps/s with complex time-dependent hopping, {lname}",
        "unit": "trajectory*RK4-steps/s", "rows": rows,
        "config": {"workload": f"{args.lattice}_peierls", "trajectories": M, "rk4_steps": steps,
                   "dt": dt, "paths": ["stream", "auto"], "U": 3.3,
                   "hopping": "t exp(i (x_k - x_i) 0.5 sin(2 tau)), x = graph distance"}}))


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU; --gpus must be 1"}))
        sys.exit(2)
    import torch
    import paper_2212_04352_amd as ft
    from workloads import FLAKE_198 as W

    torch.cuda.set_device(0)
    if args.workload == "torus54":
        return run_torus54(args)
    if args.workload == "batch":
        return run_batch(args)
    if args.workload == "adjoint":
        return run_adjoint(args)
    if args.workload == "thermal":
        return run_thermal(args)
    if args.workload == "sizes":
        return run_sizes(args)
    if args.workload == "pulse":
        return run_pulse(args)
    if args.workload == "longrange":
        return run_longrange(args)
    if args.workload == "peierls":
        return run_peierls(args)

    torch.cuda.set_device(0)
    if args.copy_calibration_mib > 0:
        nbytes = args.copy_calibration_mib << 20
        src = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        log(f"calibration copy of {args.copy_calibration_mib} MiB done")
        del src, dst
    M = args.traj or W.n_traj
    n_steps = args.horizon_steps or W.n_steps
    lat = ft.Lattice(W.kind, W.a, W.b, W.t_hop)
    n0 = lat.fock_start(W.start, W.seed)
    N = lat.N

    # ---------------------------------------------------------------- FP32 (headline)
    tuned = None
    if args.config < 0 and not args.no_autotune and args.path == "auto":
        probe = ft.Problem.allocate(lat, W.U, min(M, 2048), n0, "f32")
        ft.sample(probe, W.seed)
        tuned = ft.autotune(probe, probe_steps=200)[0]
        del probe
        log(f"autotuned configuration for N={N} f32: {tuned} (-1 = stream path)")
    if args.config >= 0:
        path32 = "resident"
    elif tuned is not None:
        path32 = "resident" if tuned >= 0 else "stream"
    else:
        path32 = resolved_path(ft, lat, "f32", args.path)
    ws = None
    for k in range(args.warmup):
        log(f"warmup pass {k + 1}/{args.warmup} (f32, {path32}, {M} trajectories x {n_steps} steps)")
        prob, ws, _, _ = run_pass(ft, torch, W, lat, n0, "f32", M, n_steps, path32, W.seed, ws,
                                  args.config)
        del prob
    torch.cuda.synchronize()
    kernel_ms = 0.0
    launches = 0
    work = 0.0
    log(f"timing {args.steps} pass(es)")
    t0 = time.perf_counter()
    for _ in range(args.steps):
        prob32, ws, timing, obs32 = run_pass(ft, torch, W, lat, n0, "f32", M, n_steps, path32,
                                             W.seed, ws, args.config)
        kernel_ms += timing["ms"].value
        launches += timing["launches"].value
        work += timing["work"].value
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    log(f"f32 done: {elapsed:.2f} s")
    value = M * n_steps * args.steps / elapsed
    bytes_per_ts_f32 = 2 * (2 * N * N) * 4
    avg_ms = kernel_ms / max(launches, 1)
    work_per_launch = work / max(launches, 1)
    achieved = bytes_per_ts_f32 * work_per_launch / (avg_ms * 1e-3) / 1e9
    kernel_name = "rk4_resident" if path32 == "resident" else "rk4_stage_stream"
    run_config = args.config if args.config >= 0 else tuned
    traffic = counter_traffic(kernel_name, "f32", work_per_launch, run_config)
    flops_per_ts = FLOPS_PER_ELEMENT_STAGE * 4 * 2 * (N * (N + 1) // 2)
    tflops = flops_per_ts * work_per_launch / (avg_ms * 1e-3) / 1e12
    issue = counter_record(kernel_name, "f32", run_config) or {}
    result = {
        "metric": "trajectory*RK4-steps/s at N=198, FP32 vs FP64 plain, at stated obs. error",
        "value": value,
        "unit": "trajectory*RK4-steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": elapsed / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic (seeded Philox Gaussian samples around a Neel Fock state)",
        "config": {"workload": W.name, "lattice": "armchair 10x20 trimmed, N=198", "U": W.U,
                   "trajectories": M, "dt": W.dt, "rk4_steps": n_steps,
                   "record_every": W.record_every, "moments": "f64", "path": path32,
                   "kernel_config": run_config},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "kernel": kernel_name, "kernel_avg_ms": avg_ms,
                     "algorithmic_bytes_per_traj_step": bytes_per_ts_f32,
                     "traj_steps_per_launch": work_per_launch,
                     "note": "the resident kernel keeps each trajectory on chip: achieved is the "
                             "byte-equivalent rate of the state's algorithmic traffic; alu and "
                             "issue give the on-chip view",
                     "alu": {"achieved": tflops, "unit": "TFLOP/s",
                             "peak": FP32_VECTOR_PEAK_TFLOPS,
                             "frac": tflops / FP32_VECTOR_PEAK_TFLOPS,
                             "peak_plain_fp32": FP32_PLAIN_PEAK_TFLOPS,
                             "frac_plain_fp32": tflops / FP32_PLAIN_PEAK_TFLOPS,
                             "algorithmic_flops_per_traj_step": flops_per_ts},
                     "issue": {k: issue[k] for k in ("valu_busy", "lds_busy", "lds_bank_conflict",
                                                     "valu_insts_per_element_stage",
                                                     "lds_insts_per_element_stage")
                               if k in issue} or None},
    }
    del ws

    # ---------------------------------------------------------------- FP64 on identical samples
    if not args.no_fp64:
        M64 = min(args.fp64_traj, M)
        steps64 = args.fp64_steps or n_steps
        path64 = resolved_path(ft, lat, "f64", args.path)
        log(f"f64 comparison ({path64}, first {M64} trajectories x {steps64} steps)")
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        prob64, ws64, timing64, obs64 = run_pass(ft, torch, W, lat, n0, "f64", M64, steps64,
                                                 path64, W.seed, None)
        torch.cuda.synchronize()
        el64 = time.perf_counter() - t0
        v64 = M64 * steps64 / el64
        log(f"f64 done: {el64:.2f} s; f32 on the same trajectories")
        _, _, _, obs32s = run_pass(ft, torch, W, lat, n0, "f32", M64, steps64, path32, W.seed, None)
        n32, C32, _ = obs32s
        n64, C64, _ = obs64
        dn = (n32 - n64).abs().amax(dim=1).cpu().numpy()
        dC = (C32 - C64).abs().amax(dim=(1, 2)).cpu().numpy()
        times = [r * W.record_every * W.dt for r in range(n64.shape[0])]

        def upto(arr, tmax):
            sel = [a for a, t in zip(arr, times) if t <= tmax + 1e-9]
            return float(max(sel)) if sel else None

        result["fp64"] = {"value": v64, "unit": "trajectory*RK4-steps/s", "path": path64,
                          "trajectories": M64, "rk4_steps": steps64,
                          "kernel_avg_ms": timing64["ms"].value / max(timing64["launches"].value, 1)}
        result["fp32_over_fp64"] = value / v64
        result["obs_error_fp32_vs_fp64"] = {
            "trajectories": M64,
            "max_abs_dn": {"t<=5": upto(dn, 5), "t<=8": upto(dn, 8), "t<=10": upto(dn, 10),
                           "t<=20": upto(dn, 20)},
            "max_abs_dC": {"t<=5": upto(dC, 5), "t<=8": upto(dC, 8), "t<=10": upto(dC, 10),
                           "t<=20": upto(dC, 20)},
        }
        # the stated accuracy (every other record, to bound host memory)
        from workloads import FP32_HORIZON, fp32_contract
        sl = slice(None, None, 2)
        result["obs_error_fp32_vs_fp64"]["contract"] = fp32_contract(
            n32[sl].cpu().numpy(), C32[sl].cpu().numpy(), n64[sl].cpu().numpy(),
            C64[sl].cpu().numpy(), prob64.S1[sl].cpu().numpy(), prob64.S2[sl].cpu().numpy(),
            M64, times[::2], FP32_HORIZON[W.U])
        del prob64, ws64

    if not args.no_cpu_baseline:
        log(f"cpu baseline: oracle, {args.cpu_traj} trajectories x {args.cpu_steps} steps")
        result["cpu_baseline"] = cpu_baseline(W, args.cpu_traj, args.cpu_steps)
    print(json.dumps(result), flush=True)
    # explicit teardown: device buffers and the lattice's tables are released
    # here, while the HIP runtime is certainly up, not by finalizers at exit
    del prob32, obs32
    if not args.no_fp64:
        del obs64, obs32s
    torch.cuda.synchronize()
    lat.close()


if __name__ == "__main__":
    main()
