"""Benchmark: time-to-solution of the monolithic blocked AMG hot path on one GPU.

One step = the whole hot path on one synthetic block system already resident
in HBM: hierarchy setup on the GPU (strength graph, aggregation, tentative P,
Galerkin products, smoother data, coarsest inverse) followed by the
right-preconditioned GMRES solve to rtol 1e-8.  Forms: plain FP64, the FP32
V-cycle inside FP64 flexible GMRES, and that refined form with the trained
per-aggregate weights (the fixed-weight hierarchy judges it and replaces it
when its measured convergence factor is worse; both builds are inside the
timed step).  Prints one JSON line.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME]
"""
from __future__ import annotations

import argparse
import json
import os
import platform
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "time-to-solve (rtol 1e-8) + V-cycle HBM GB/s: FP64 vs FP32-refined vs learned"
HBM_PEAK_GBS = 8000.0
WORKLOAD_LABEL = {
    "2d-32": "2D 32x32 nodes, 6 dofs/node (6,144 unknowns), gamma 0.1",
    "2d-256": "2D 256x256 nodes, 6 dofs/node (393,216 unknowns), gamma 0.5",
    "3d-64": "3D 64^3 nodes, 8 dofs/node (2,097,152 unknowns), gamma 0.5",
    "2d-512-lognormal": "2D 512x512 nodes, 6 dofs/node, lognormal kappa sigma 1, gamma 5",
    "3d-128-lognormal": "3D 128^3 nodes, 8 dofs/node (16,777,216 unknowns), lognormal kappa sigma 1, gamma 2",
}


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="3d-128-lognormal")
    ap.add_argument("--seed", type=int, default=1)
    ap.add_argument("--rtol", type=float, default=1e-8)
    ap.add_argument("--forms", default="fp64,fp32,learned")
    ap.add_argument("--weights", default=None, help="trained network (JSON); default: the committed one")
    ap.add_argument("--vcycles", type=int, default=20, help="V-cycles timed for the V-cycle bandwidth figure")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-sample-n", type=int, default=0, help="grid size of the oracle sample (0: automatic)")
    ap.add_argument("--counter-run", action="store_true",
                    help="for hardware-counter profiling: one setup of the first of --forms, a 1 GiB calibration "
                         "copy, then a few V-cycles and operator applies (no solve)")
    return ap.parse_args()


def counter_run(args):
    """Short, fixed sequence of kernels for per-dispatch counter collection."""
    import torch
    from paper_2103_07537_amd import mbamg
    from paper_2103_07537_amd.inputs import workload
    mbamg.lib()
    torch.cuda.set_device(0)
    system = workload(args.workload, seed=args.seed)
    blocks = mbamg.to_device(system)
    b = torch.from_numpy(system.b).cuda()
    precision, use_mlp = FORMS[args.forms.split(",")[0]]
    mlp = None
    if use_mlp:
        from paper_2103_07537_amd import learned
        mlp = learned.load(args.weights or learned.DEFAULT_WEIGHTS)
    h = mbamg.Hierarchy(blocks, system.dofs, system.n_vec, precision=precision, mlp=mlp)
    log("[counters] setup done")
    src = torch.ones(1 << 27, dtype=torch.float64, device="cuda")      # 1 GiB
    dst = torch.empty_like(src)
    dst.copy_(src)                                                      # calibration: 1 GiB read, 1 GiB written
    torch.cuda.synchronize()
    z = torch.empty_like(b)
    w = torch.empty_like(b)
    for _ in range(3):
        h.vcycle(b, z)
        h.apply(z, w)
    torch.cuda.synchronize()
    log("[counters] done")
    print(json.dumps({"counter_run": args.workload, "calibration_bytes": 1 << 30}), flush=True)


FORMS = {
    # name: (precision, learned network)
    "fp64": (0, False),
    "fp32": (1, False),
    "learned": (1, True),      # the full chosen form: FP32 cycle in FP64 FGMRES + learned weights, judged
    "learned64": (0, True),
}


def run_step(blocks, system, b, form, rtol, timing, mlp=None):
    """One step: setup + solve.  timing: the library's event mode (0 off; 1
    every kind; 2 whole V-cycles; 3 V-cycles and levels), for the untimed
    profiling steps only."""
    from paper_2103_07537_amd import mbamg
    import torch
    precision, use_mlp = FORMS[form]
    t0 = time.perf_counter()
    h = mbamg.Hierarchy(blocks, system.dofs, system.n_vec, precision=precision, mlp=mlp if use_mlp else None)
    t1 = time.perf_counter()
    if timing:
        h.timing_enable(timing)
    x = torch.zeros_like(b)
    info = h.solve(b, x, rtol=rtol)
    t2 = time.perf_counter()
    log(f"[bench]   {form}: hierarchy {1e3 * (t1 - t0):.1f} ms, solve {1e3 * (t2 - t1):.1f} ms (wall)"
        + (f" [profiling step, event mode {timing}]" if timing else ""))
    return h, x, info


def profile_steps(blocks, system, b, form, rtol, mlp):
    """Untimed steps with HIP events: the V-cycle as the solver applies it
    (mode 2, nothing else timed), each level's share (mode 3), and for the FP64
    form the finest level's kernels (mode 1)."""
    out = {}
    h, _, info = run_step(blocks, system, b, form, rtol, 2, mlp)
    v = h.timing_get(4)
    out["vcycle_in_solve_ms"] = v["total_ms"] / max(v["launches"], 1)
    out["vcycle_in_solve_count"] = v["launches"]
    bytes_total = h.vcycle_bytes()
    h.close()
    h, _, info = run_step(blocks, system, b, form, rtol, 3, mlp)
    levels = []
    for l in range(h.num_levels()):
        down_b, up_b = h.level_vcycle_bytes(l)
        dn, up = h.timing_get(16 + 2 * l), h.timing_get(17 + 2 * l)
        cyc = max(dn["launches"], 1)
        ms = (dn["total_ms"] + up["total_ms"]) / cyc
        levels.append({"level": l, "nodes": h.level_nodes(l), "ms_per_cycle": ms,
                       "down_ms": dn["total_ms"] / cyc, "up_ms": up["total_ms"] / cyc,
                       "alg_bytes": down_b + up_b,
                       "alg_GBps": (down_b + up_b) / (ms * 1e-3) / 1e9 if ms > 0 else None})
    out["levels"] = levels
    h.close()
    out["vcycle_bytes"] = bytes_total
    # every launch of the smoother, residual and transfer kernels bracketed by events (mode 1)
    h, _, info = run_step(blocks, system, b, form, rtol, 1, mlp)
    if form == "fp64":
        out["kernel_stats"] = {k: h.timing_get(k) for k in (0, 1, 2, 3)}
    cycles = max(h.timing_get(4)["launches"], 1)
    names = {0: "smoother, post", 1: "residual", 3: "smoother, other", 5: "restriction", 6: "prolongation"}
    launches = []
    for l in range(h.num_levels() - 1):
        for k, nm in names.items():
            st = h.timing_get(k if l == 0 else 64 + 8 * l + k)
            if st["launches"] == 0:
                continue
            launches.append({"level": l, "kind": nm, "launches_per_cycle": st["launches"] / cycles,
                             "us_per_cycle": 1e3 * st["total_ms"] / cycles,
                             "avg_us": 1e3 * st["total_ms"] / st["launches"],
                             "alg_GBps": st["bytes"] / (st["total_ms"] * 1e-3) / 1e9 if st["total_ms"] else None})
    out["launch_stats"] = launches
    h.close()
    return out


def vcycle_rate(h, b, reps):
    import torch
    z = torch.empty_like(b)
    for _ in range(3):
        h.vcycle(b, z)
    torch.cuda.synchronize()
    times = []
    for _ in range(reps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        h.vcycle(b, z)
        e1.record()
        e1.synchronize()
        times.append(e0.elapsed_time(e1))
    ms = float(np.median(times))
    return ms, h.vcycle_bytes()


def stream_copy_rate():
    """Device-to-device copy of 1 GiB (1 GiB read + 1 GiB written): the
    bandwidth a plain streaming kernel reaches on this GPU, reported beside
    the 8 TB/s specification."""
    import torch
    src = torch.ones(1 << 27, dtype=torch.float64, device="cuda")
    dst = torch.empty_like(src)
    for _ in range(2):
        dst.copy_(src)
    torch.cuda.synchronize()
    times = []
    for _ in range(5):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        dst.copy_(src)
        e1.record()
        e1.synchronize()
        times.append(e0.elapsed_time(e1))
    del src, dst
    return 2.0 * (1 << 30) / (float(np.median(times)) * 1e-3) / 1e9


def host_cpu():
    model = None
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    try:
        usable = len(os.sched_getaffinity(0))
    except AttributeError:
        usable = os.cpu_count()
    return {"model": model or platform.processor() or platform.machine(), "nproc": os.cpu_count(),
            "usable_cpus": usable}


def cpu_baseline(args, form, gpu_iters, mlp):
    """The oracle, single-threaded, on a bounded sample of the same workload
    family (the same generator on a smaller grid) doing the same work as the
    reported form: for the learned form the oracle runs the same network
    (bfloat16-emulated) on its own features, builds the fixed hierarchy too and
    lets the two probes judge.  The sample is timed as it stands; `value` is
    that time extrapolated linearly to the full workload (by the unknown ratio,
    and for the solve to the GPU's iteration count) and is labelled so.  The
    GPU solves the same sample system in the same form, and its solution's
    difference from the oracle's is reported."""
    import torch
    from threadpoolctl import threadpool_limits
    from oracle import amg
    from paper_2103_07537_amd import mbamg
    from paper_2103_07537_amd.inputs import WORKLOADS, make_system
    kw = dict(WORKLOADS[args.workload])
    full_n = kw["n"]
    dim = kw["dim"]
    n_s = min(args.cpu_sample_n or (48 if dim == 3 else 256), full_n)
    kw["n"] = n_s
    s = make_system(seed=args.seed, **kw)
    learned_form = FORMS[form][1] and mlp is not None
    weights = None
    if learned_form:
        from oracle import learned as ol
        theta = np.asarray(mlp[:5122], dtype=np.float64)
        mean, std = mlp[5122:5134], mlp[5134:5146]

        def weights(level, n_agg, F):
            out, _ = ol.forward(theta, ((F.astype(np.float32) - mean) / std).astype(np.float64), emulate=True)
            return out[:, 0], out[:, 1]
    with threadpool_limits(1):
        t0 = time.perf_counter()
        h = amg.setup(s.blocks, s.dofs, amg.Params(weights=weights), n_vec=s.n_vec)
        used_learned = learned_form
        if learned_form:
            hf = amg.setup(s.blocks, s.dofs, amg.Params(), n_vec=s.n_vec)
            if not amg.probe(h, 10, 12345) < amg.probe(hf, 10, 12345):
                h = hf
                used_learned = False
        t1 = time.perf_counter()
        xo, info = amg.gmres(h, s.b, rtol=args.rtol)
        t2 = time.perf_counter()
    # the GPU on the same sample system, same form
    precision, _ = FORMS[form]
    hg = mbamg.Hierarchy(mbamg.to_device(s), s.dofs, s.n_vec, precision=precision,
                         mlp=mlp if learned_form else None)
    bg = torch.from_numpy(s.b).cuda()
    xg = torch.zeros_like(bg)
    ginfo = hg.solve(bg, xg, rtol=args.rtol)
    xg = xg.cpu().numpy()
    hg.close()
    err = float(np.linalg.norm(xg - xo) / np.linalg.norm(xo))
    ratio = (full_n / n_s) ** dim
    per_it = (t2 - t1) / max(info.iterations, 1)
    est_ms = 1e3 * ((t1 - t0) * ratio + per_it * ratio * gpu_iters)
    what = ("learned and fixed setups, both probes, " if learned_form else "setup, ") + "GMRES(30)"
    return {
        "value": est_ms, "unit": "ms", "cores": 1, "kind": "oracle",
        "extrapolated": n_s < full_n,
        "sample": (f"oracle ({what}, FP64, one thread) on the same generator at {n_s}^{dim} nodes "
                   f"({s.n_dofs} unknowns): {1e3 * (t1 - t0):.0f} ms setup + {1e3 * (t2 - t1):.0f} ms for "
                   f"{info.iterations} iterations, measured; value = that time extrapolated linearly by the "
                   f"unknown ratio {ratio:.1f} and to the GPU's {gpu_iters} iterations"
                   + ("" if n_s < full_n else " (the sample is the full workload: no extrapolation)")),
        "sample_measured": {"n": n_s, "unknowns": s.n_dofs, "setup_ms": 1e3 * (t1 - t0),
                            "solve_ms": 1e3 * (t2 - t1), "iterations": info.iterations,
                            "used_learned": bool(used_learned)},
        "gpu_on_sample": {"iterations": ginfo["iterations"], "used_learned": ginfo["used_learned"],
                          "t_setup_ms": ginfo["t_setup_ms"], "t_solve_ms": ginfo["t_solve_ms"],
                          "rel_diff_vs_oracle_solution": err},
        "host": host_cpu(),
        "threads": 1,
    }


# what a launch moves is decided here: the solve's kernels, and the layouts and launches around them
TRAFFIC_SOURCES = ("solve_kernels.hip", "solve_kernels.h", "solve_device.h", "sweep_kernels.hip", "dpp.h",
                   "setup_kernels.hip", "hierarchy.hip")


def traffic_source_hash():
    """SHA-256 over those of TRAFFIC_SOURCES that are there, in order."""
    import hashlib
    sha = hashlib.sha256()
    for name in TRAFFIC_SOURCES:
        path = os.path.join(ROOT, "paper_2103_07537_amd", "csrc", name)
        if os.path.exists(path):
            sha.update(open(path, "rb").read())
    return sha.hexdigest()


def measured_traffic(workload_name, kind, form="fp64"):
    """HBM bytes per launch of a kind of launch, and of the form's whole
    V-cycle, from the committed counter summaries, or None where none matches
    this workload, form and source."""
    import glob
    sha = traffic_source_hash()
    for path in sorted(glob.glob(os.path.join(ROOT, "profiles", "traffic_*.txt"))):
        kv = {}
        for line in open(path):
            if "=" in line and not line.startswith(" "):
                k, v = line.strip().split("=", 1)
                kv[k] = v
        if (kv.get("workload") == workload_name and kv.get("kind") == str(kind)
                and kv.get("form", "fp64") == form and kv.get("source_sha256") == sha):
            vc = float(kv["vcycle_traffic_bytes"]) if "vcycle_traffic_bytes" in kv else None
            return float(kv["traffic_bytes_per_launch"]), os.path.relpath(path, ROOT), vc
    return None, None, None


def main():
    args = parse()
    if args.counter_run:
        counter_run(args)
        return
    if args.gpus != 1:
        print(json.dumps({"error": "the solver runs on one GPU; --gpus must be 1 (sharding the hierarchy "
                                   "over several GPUs is not implemented)"}))
        sys.exit(2)
    import torch
    from paper_2103_07537_amd import mbamg
    from paper_2103_07537_amd.inputs import workload
    mbamg.lib()
    torch.cuda.set_device(0)
    log(f"[bench] generating {args.workload} seed {args.seed}")
    t0 = time.perf_counter()
    system = workload(args.workload, seed=args.seed)
    log(f"[bench] generated {system.n_dofs} unknowns in {time.perf_counter() - t0:.1f} s")
    blocks = mbamg.to_device(system)
    b = torch.from_numpy(system.b).cuda()
    torch.cuda.synchronize()
    forms = [f for f in args.forms.split(",") if f]
    for f in forms:
        if f not in FORMS:
            raise SystemExit(f"unknown form {f}; choose from {sorted(FORMS)}")
    mlp = None
    if any(FORMS[f][1] for f in forms):
        from paper_2103_07537_amd import learned
        wpath = args.weights or learned.DEFAULT_WEIGHTS
        if os.path.exists(wpath):
            mlp = learned.load(wpath)
        else:
            log(f"[bench] no trained network at {wpath}; skipping the learned forms")
            forms = [f for f in forms if not FORMS[f][1]]
    results = {}
    xs = {}
    for form in forms:
        for w in range(args.warmup):
            h, x, info = run_step(blocks, system, b, form, args.rtol, 0, mlp)
            log(f"[bench] warmup {form} {w}: its {info['iterations']} setup {info['t_setup_ms']:.1f} ms "
                f"solve {info['t_solve_ms']:.1f} ms")
            h.close()
        torch.cuda.synchronize()
        t_start = time.perf_counter()
        infos = []
        for k in range(args.steps):
            h, x, info = run_step(blocks, system, b, form, args.rtol, 0, mlp)
            infos.append(info)
            if k < args.steps - 1:
                tc = time.perf_counter()
                h.close()
                log(f"[bench]   {form}: release {1e3 * (time.perf_counter() - tc):.1f} ms (wall)")
        torch.cuda.synchronize()
        t_total = time.perf_counter() - t_start
        ms_step = 1e3 * t_total / args.steps
        last = infos[-1]
        log(f"[bench] {form}: {ms_step:.1f} ms/step, its {last['iterations']}, rel {last['rel_residual']:.2e}")
        vc_ms, vc_bytes = vcycle_rate(h, b, args.vcycles)
        xs[form] = x.cpu().numpy()
        h.close()
        prof = profile_steps(blocks, system, b, form, args.rtol, mlp)
        vin = prof["vcycle_in_solve_ms"]
        vc_traffic = measured_traffic(args.workload, 0, form)[2]
        results[form] = {
            "ms_per_step": ms_step,
            "t_setup_ms": float(np.median([i["t_setup_ms"] for i in infos])),
            "t_solve_ms": float(np.median([i["t_solve_ms"] for i in infos])),
            "iterations": last["iterations"],
            "rel_residual": last["rel_residual"],
            "levels": last["levels"],
            "used_learned": last["used_learned"],
            "conv_factor": last["conv_factor"],
            "op_complexity": last["op_complexity"],
            "vcycle_bytes": vc_bytes,
            # the V-cycle as GMRES applies it (colour-order vectors; HIP events around each one
            # in an untimed profiling step)
            "vcycle_ms": vin,
            # the matrix's structural bytes (the byte model's) over that time: a measure of the method, not
            # of the memory, which moves less (blocks are stored by what determines them)
            "vcycle_alg_GBps": vc_bytes / (vin * 1e-3) / 1e9,
            # counted HBM bytes of a V-cycle over that time, and against the peak
            "vcycle_measured_bytes": vc_traffic,
            "vcycle_measured_GBps": vc_traffic / (vin * 1e-3) / 1e9 if vc_traffic else None,
            "vcycle_hbm_frac": vc_traffic / (vin * 1e-3) / 1e9 / HBM_PEAK_GBS if vc_traffic else None,
            # the V-cycle through mbamg_vcycle: adds the natural <-> colour reordering of r and z
            "vcycle_abi_ms": vc_ms,
            "per_level": prof["levels"],
            "per_launch_kind": prof["launch_stats"],
            "kernel_stats": prof.get("kernel_stats"),
        }
    ref = "fp64" if "fp64" in xs else forms[0]
    for form in forms:
        results[form]["rel_diff_vs_fp64"] = float(np.linalg.norm(xs[form] - xs[ref]) / np.linalg.norm(xs[ref]))

    chosen = next((f for f in ("learned", "fp32") if f in results), forms[0])
    # roofline of the dominant finest-level kernel in the FP64 form (HIP events around every launch of
    # the finest level's kernels during an untimed profiling step: the timed steps carry no events): the
    # HBM bytes counted for a launch over its time.  Without a counter summary for this workload and
    # source the rate is not known: the byte model's structural bytes are more than a launch moves.
    roof = None
    st = results.get("fp64", {}).get("kernel_stats")
    if st:
        names = {0: "block Gauss-Seidel colour pass (post-smoother, finest level)",
                 1: "residual (finest level)", 2: "operator apply (finest level)",
                 3: "block Gauss-Seidel colour pass (pre-smoother, finest level)"}
        kind = max((0, 1, 2, 3), key=lambda k: st[k]["total_ms"])
        s = st[kind]
        per_launch_bytes = s["bytes"] / max(s["launches"], 1)
        avg_ms = s["total_ms"] / max(s["launches"], 1)
        traffic, tsrc, _ = measured_traffic(args.workload, kind)
        achieved = traffic / (avg_ms * 1e-3) / 1e9 if traffic else None
        roof = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": achieved / HBM_PEAK_GBS if traffic else None, "traffic": traffic, "kernel": names[kind],
                "launches": s["launches"], "avg_us": avg_ms * 1e3, "alg_bytes_per_launch": per_launch_bytes,
                "alg_GBps": per_launch_bytes / (avg_ms * 1e-3) / 1e9,
                "traffic_source": tsrc, "stream_copy_GBps": stream_copy_rate()}
    cpu = None
    if not args.no_cpu_baseline:
        log("[bench] cpu baseline (oracle sample)")
        cpu = cpu_baseline(args, chosen, results[chosen]["iterations"], mlp)
    out = {
        "metric": METRIC,
        "value": results[chosen]["ms_per_step"],
        "unit": "ms",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": results[chosen]["ms_per_step"],
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32 V-cycle in f64 FGMRES" if FORMS[chosen][0] == 1 else "f64",
        "data": "synthetic",
        "config": {"workload": WORKLOAD_LABEL.get(args.workload, args.workload), "name": args.workload,
                   "unknowns": system.n_dofs, "rtol": args.rtol, "krylov": "GMRES(30) right-preconditioned",
                   "form": chosen},
        "forms": results,
        "roofline": roof,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
