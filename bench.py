"""Benchmark: space-time DOF/s of the multigrid solve to relative residual 1e-8.

One step = one full solve L_h u = f from u = 0 (V(1,1) cycles of the
time-parallel multigrid with the damped block-Jacobi slab smoother, iterated
in the spatial eigenbasis) until ||f - L_h u||_2 <= 1e-8 ||f||_2, on the
largest single-GPU workload by default: unit square, p = 2, 256 x 256
elements, 1024 slabs x 1 time element (201,326,592 unknowns), right-hand side
from 8 random Fourier modes (seed 4).  Inputs are resident in HBM when the
timed region starts; setup and right-hand-side assembly are outside it.

The timed region launches the solve's kernels eagerly with speculative
cycles (the library default).  The headline is the plain FP64 method; the
same workload is then solved with FP32 and BF16x3 spatial transforms (FP64
defect correction around reduced-precision inner solves) and reported beside
it with its error against the FP64 result.  The JSON line also carries the
roofline of the dominant kernel class on the finest multigrid level (HIP
events on the solve's stream around each of its launches there, in an eager
pass of the same K solves right after the timed region; HBM traffic from the
committed rocprofv3 counter summary when it matches the kernel sources), a
short serving leg (the serving request mix through the library's server: its
saturation rate and p50/p99 latency at 0.8 of it) and the FP64 CPU oracle
timed on a bounded sample of the same workload.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "space-time DOF/s to rel.res 1e-8, FP64 vs mixed; serve p50/p99 latency"
PEAKS = {  # MI355X published peaks
    "hbm": 8.0e12,            # bytes/s
    "fp64": 78.6e12,          # FLOP/s, vector = matrix
    "fp32": 157.3e12,
    "bf16": 2.5e15,
}
# dominant-class roofline: which bound applies to each kernel class
CLASS_BOUND = {"residual": "hbm", "xform_x": "mfma", "xform_s": "mfma", "xform_axis": "mfma", "timemix": "hbm",
               "restrict": "hbm", "prolong": "hbm", "norm": "hbm", "other": "hbm", "xform_2d": "mfma",
               "eig_smooth": "hbm", "eig_resid": "hbm", "resnorm": "mfma", "eig_cycle_end": "hbm",
               "eig_cycle_close": "hbm", "eig_coarse": "hbm", "minres": "hbm"}


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def host_cpu():
    """CPU model and the cores this process may use."""
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        usable = len(os.sched_getaffinity(0))
    except AttributeError:
        usable = os.cpu_count()
    return model, usable


def _cpu_baseline_child(cfg_name, sample_slabs, conn):
    """FP64 oracle direct solve of the workload (one SuperLU factorization of
    the slab matrix A_n, then slab-wise forward substitution), single-threaded
    like the paper's single-core timings; assembly excluded as in the paper.
    The factorization is timed whole; the forward substitution on the first
    `sample_slabs` slabs, scaled to all slabs.  Runs in a spawned interpreter
    (numpy, scipy and the oracle only) while the GPU part of the bench runs."""
    try:
        from threadpoolctl import threadpool_limits
        import scipy.sparse.linalg as spla
        import workloads as W
        from oracle.spacetime import Problem, assemble_rhs
        from oracle.solve import SlabSystem

        cfg = W.CONFIGS[cfg_name]
        prob = Problem(cfg.dim, cfg.n_elem, cfg.degree, cfg.n_slabs, cfg.n_elem_t, cfg.T, cfg.theta)
        with threadpool_limits(limits=1):
            t0 = time.perf_counter()
            sysm = SlabSystem.assemble(prob)
            f = assemble_rhs(prob, cfg.modes(), slabs=range(sample_slabs))
            t_asm = time.perf_counter() - t0
            t0 = time.perf_counter()
            lu = spla.splu(sysm.A)
            t_fact = time.perf_counter() - t0
            F = f.reshape(sample_slabs, -1)
            t0 = time.perf_counter()
            u = lu.solve(F[0])
            for k in range(1, sample_slabs):
                u = lu.solve(F[k] + sysm.B @ u)
            t_solve = (time.perf_counter() - t0) / sample_slabs
        conn.send({"t_asm": t_asm, "t_fact": t_fact, "t_slab": t_solve})
    except Exception as e:                     # reported, not raised: the GPU result stands
        conn.send({"error": repr(e)})
    conn.close()


def start_cpu_baseline(cfg, sample_slabs):
    import multiprocessing as mp
    ctx = mp.get_context("spawn")              # a fresh interpreter: no GPU state is inherited
    rd, wr = ctx.Pipe(duplex=False)
    proc = ctx.Process(target=_cpu_baseline_child, args=(cfg.name, sample_slabs, wr), daemon=True)
    proc.start()
    wr.close()
    return proc, rd, time.perf_counter()


def finish_cpu_baseline(cfg, sample_slabs, started, limit_s):
    proc, rd, t_start = started
    left = max(1.0, limit_s - (time.perf_counter() - t_start))
    res = rd.recv() if rd.poll(left) else {"error": f"not finished within {limit_s:.0f} s"}
    proc.join(5)
    if proc.is_alive():
        proc.kill()
    model, usable = host_cpu()
    if "error" in res:
        log(f"cpu baseline: {res['error']}")
        return {"value": None, "unit": "DOF/s", "cores": 1, "kind": "oracle", "host_cpu": model,
                "host_cores": usable, "sample": f"oracle direct solve, not measured: {res['error']}"}
    est = res["t_fact"] + cfg.n_slabs * res["t_slab"]
    log(f"cpu baseline: oracle assembly {res['t_asm']:.1f} s (excluded), factorization {res['t_fact']:.2f} s, "
        f"{res['t_slab'] * 1e3:.1f} ms per slab solve")
    return {
        "value": cfg.unknowns / est,
        "unit": "DOF/s",
        "cores": 1,
        "kind": "oracle",
        "host_cpu": model,
        "host_cores": usable,
        "solve_phase_value": cfg.unknowns / (cfg.n_slabs * res["t_slab"]),
        "sample": (f"oracle direct solve (SuperLU factorization of the slab matrix, timed whole, + forward "
                   f"substitution timed on {sample_slabs} of {cfg.n_slabs} slabs and scaled to all), one thread "
                   f"of {usable} on the host ({model}; SuperLU is sequential and the forward substitution is "
                   f"sequential in time); assembly excluded (factorization {res['t_fact']:.2f} s, "
                   f"{res['t_slab'] * 1e3:.1f} ms/slab); solve_phase_value leaves out the factorization "
                   f"(the paper's setup)"),
    }


# the sources a kernel class compiles from (the committed HBM counters of a
# class stay valid while these are unchanged); other classes: every kernel file
KERNEL_FILES = ("kernels.hpp", "kernels_common.hpp", "k_residual.hip", "k_xform2d.hip", "k_xform_axis.hip",
                "k_xform_panel.hip", "k_xform_eo.hip", "k_xform2d_eo.hip", "k_cycles.hip", "k_eigen.hip", "k_misc.hip",
                "k_minres.hip")
CLASS_SOURCES = {
    "eig_cycle_close": ("kernels_common.hpp", "k_eigen.hip", "k_cycles.hip"),
    "eig_cycle_end": ("kernels_common.hpp", "k_eigen.hip"),
    "eig_smooth": ("kernels_common.hpp", "k_eigen.hip", "k_cycles.hip"),
    "xform_axis": ("kernels_common.hpp", "k_xform_axis.hip", "k_xform_panel.hip", "k_xform_eo.hip"),
    "xform_2d": ("kernels_common.hpp", "k_xform2d.hip", "k_xform2d_eo.hip"),
    "residual": ("kernels_common.hpp", "k_residual.hip"),
}


def kernel_source_hash(kclass=None):
    import hashlib
    h = hashlib.sha256()
    for name in CLASS_SOURCES.get(kclass, KERNEL_FILES):
        with open(os.path.join(ROOT, "paper_1802_09277_amd", "csrc", name), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def measured_traffic(cfg_name, basis, prec, kclass):
    """HBM bytes per launch of the dominant kernel class from the committed
    rocprofv3 counter summary (FETCH_SIZE + WRITE_SIZE, scaled by a plain copy
    of known size); None when there is none for this workload or when the
    kernel sources changed since the counters were taken."""
    path = os.path.join(ROOT, "profiles", f"{cfg_name.lower()}_{basis}_{prec}_traffic.md")
    if not os.path.exists(path):
        return None
    fields = {}
    with open(path) as fh:
        for line in fh:
            if line.startswith("- ") and ": " in line:
                k, v = line[2:].split(": ", 1)
                fields[k.strip().strip("`")] = v.strip().strip("`")
    if fields.get("kernel_class") != kclass or fields.get("kernel_sources_sha256") != kernel_source_hash(kclass):
        return None
    return float(fields["traffic_bytes_per_launch"])


def serve_measure(n_requests, slots, budget_gib, basis, loads, graphs, prec):
    """Serving workload: 2-D requests with n_elem in {32..256}, p in {2,3,4},
    slabs in {16..512}, random-mode right-hand sides seeded by the request id,
    rtol 1e-8.  A closed burst measures the saturation rate (after a cold
    burst that fills the setup cache); Poisson arrivals at fractions of it
    give p50/p99 latency (submit -> solution in the caller's buffer)."""
    import threading
    import numpy as np
    import torch
    import paper_1802_09277_amd as sth
    import workloads as W

    torch.cuda.set_device(0)
    reqs = W.serving_requests(n_requests, seed=0)
    srv = sth.Server(budget_gib << 30, slots)
    if graphs:
        srv.use_graphs(True)
    shape = lambda c: dict(dim=c.dim, n_elem=c.n_elem, degree=c.degree, n_slabs=c.n_slabs, n_elem_t=c.n_elem_t)

    def burst():
        t0 = time.perf_counter()
        outs, tickets = [], []
        for c in reqs:
            u = torch.empty(sth.problem_vector_len(**shape(c)), dtype=torch.float64, device="cuda")
            outs.append(u)
            tickets.append(srv.submit(c.modes(), u, rtol=1e-8, maxit=100, basis=basis, prec=prec, **shape(c)))
        stats = [srv.wait(t) for t in tickets]
        torch.cuda.synchronize()
        return time.perf_counter() - t0, stats

    t_cold, _ = burst()
    t_warm, stats = burst()
    bad = [st["message"] for st in stats if st["status"] != 0]
    if bad:
        raise RuntimeError(f"serving: {len(bad)} requests failed: {bad[:3]}")
    total_dof = sum(c.unknowns for c in reqs)
    sat_rps = len(reqs) / t_warm
    log(f"serve: cold burst {t_cold:.2f} s, warm burst {t_warm:.2f} s, {sat_rps:.1f} requests/s")
    rng = np.random.default_rng(1)
    rates = []
    for load in loads:
        lam = load * sat_rps
        arrivals = np.cumsum(rng.exponential(1.0 / lam, size=len(reqs)))
        tickets, outs = [None] * len(reqs), [None] * len(reqs)

        def client():
            t0 = time.perf_counter()
            for i, c in enumerate(reqs):
                delay = arrivals[i] - (time.perf_counter() - t0)
                if delay > 0:
                    time.sleep(delay)
                outs[i] = torch.empty(sth.problem_vector_len(**shape(c)), dtype=torch.float64, device="cuda")
                tickets[i] = srv.submit(c.modes(), outs[i], rtol=1e-8, maxit=100, basis=basis, prec=prec,
                                        **shape(c))

        t0 = time.perf_counter()
        th = threading.Thread(target=client)
        th.start()
        th.join()
        lat = [srv.wait(t)["latency_ms"] for t in tickets]
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        rates.append({"load": load, "offered_rps": lam, "achieved_rps": len(reqs) / wall,
                      "dof_per_s": total_dof / wall, "p50_ms": float(np.percentile(lat, 50)),
                      "p99_ms": float(np.percentile(lat, 99))})
        log(f"serve: load {load}: p50 {rates[-1]['p50_ms']:.1f} ms, p99 {rates[-1]['p99_ms']:.1f} ms")
    resident, setups = srv.resident()
    srv.close()
    return {"requests": len(reqs), "streams": slots, "graphs": bool(graphs), "transform_prec": prec,
            "saturation_rps": sat_rps,
            "saturation_dof_per_s": total_dof / t_warm, "unknowns_total": total_dof, "cold_burst_s": t_cold,
            "warm_burst_s": t_warm, "mean_cycles": float(np.mean([st["iters"] for st in stats])),
            "cached_setups": setups, "resident_gib": resident / 2 ** 30, "poisson": rates}


def serve_bench(args):
    sv = serve_measure(args.serve_requests, args.serve_slots, args.serve_budget_gib, args.basis,
                       (0.5, 0.8, 0.95), args.serve_graphs, args.serve_prec)
    out = {
        "metric": METRIC,
        "value": sv["saturation_dof_per_s"],
        "unit": "DOF/s",
        "n_gpus": 1,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": f"serving: {sv['requests']} 2D requests, n_elem 32-256, p 2-4, 16-512 slabs x 2 "
                               f"time elems, random modes seeded by request id, rtol 1e-8",
                   "iterate_basis": args.basis, "streams": args.serve_slots,
                   "hbm_budget_gib": args.serve_budget_gib, "unknowns_total": sv["unknowns_total"]},
        "serving": sv,
    }
    print(json.dumps(out), flush=True)


# kernel classes merged for the choice of the dominant class: the two
# per-axis transform kernels are one transform
MERGED = {"xform_axis": ("xform_x", "xform_s")}


def merged_classes(names):
    out = {}
    for k in names:
        tgt = next((m for m, parts in MERGED.items() if k in parts), k)
        out.setdefault(tgt, []).append(k)
    return out


def report_sum(s, parts):
    reps = [s.timing_report(k) for k in parts]
    return {key: sum(r[key] for r in reps) for key in ("launches", "ms", "flops", "bytes")}


def make_solver(cfg, prec, args):
    import paper_1802_09277_amd as sth
    s = sth.Solver(cfg.dim, cfg.n_elem, cfg.degree, cfg.n_slabs, cfg.n_elem_t, cfg.T, cfg.theta,
                   prec=prec, basis=args.basis, coarse_slabs=args.coarse_slabs, space_ratio=args.space_ratio,
                   minres_iters=args.minres_iters)
    if args.no_speculate:
        s.speculate(False)
    return s


def timed_solves(s, f, u, args, steps):
    """K solves from u = 0 between two device synchronisations; ms per solve."""
    import torch
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    iters = relres = None
    for _ in range(steps):
        u.zero_()
        iters, relres, _ = s.solve(f, u, rtol=args.rtol, maxit=200)
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) * 1e3 / steps, iters, relres


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", default="C4")
    ap.add_argument("--prec", default="fp64", choices=["fp64", "fp32", "bf16x3"],
                    help="transform precision of the headline solve")
    ap.add_argument("--rtol", type=float, default=1e-8)
    ap.add_argument("--basis", default="eigen", choices=["nodal", "eigen"],
                    help="iterate on B-spline coefficients or in the spatial eigenbasis (same iterates)")
    ap.add_argument("--coarse-slabs", type=int, default=None,
                    help="coarsest multigrid level: at most this many slabs (library default 128)")
    ap.add_argument("--cpu-sample-slabs", type=int, default=None,
                    help="slabs of the oracle's forward substitution timed for the CPU baseline")
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="run a plain device copy of this many MiB three times first (the reference "
                         "kernel of known size that scales the HBM counters of a --pmc run)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-limit-s", type=float, default=420.0,
                    help="time the CPU oracle may take (it runs beside the GPU part)")
    ap.add_argument("--no-precision-forms", action="store_true",
                    help="skip the FP32 / BF16x3 solves reported beside the headline")
    ap.add_argument("--slabs", type=int, default=None,
                    help="profiling runs only: override the workload's slab count (the line then names a "
                         "different workload)")
    ap.add_argument("--minres-iters", type=int, default=0,
                    help="smoother slab inverse by this many MinRes iterations per temporal pair (Theorem 3.10 "
                         "preconditioner; B-spline coefficient iteration only; 0: exact)")
    ap.add_argument("--space-ratio", type=float, default=0.0,
                    help="coarsen in space too where tau/h^2 >= this (B-spline coefficient iteration only; "
                         "0: time only)")
    ap.add_argument("--no-speculate", action="store_true",
                    help="wait for each cycle's norm before enqueueing the next (library default: speculate)")
    ap.add_argument("--serve", action="store_true", help="serving workload (p50/p99 latency) instead")
    ap.add_argument("--serve-requests", type=int, default=200)
    ap.add_argument("--serve-slots", type=int, default=8)
    ap.add_argument("--serve-budget-gib", type=int, default=160)
    ap.add_argument("--serve-prec", default="fp64", choices=["fp64", "fp32", "bf16x3"],
                    help="transform precision of the serving requests (FP64 is the faster on this mix)")
    ap.add_argument("--serve-graphs", action="store_true",
                    help="serving: replay captured solve iterations instead of eager launches")
    ap.add_argument("--serve-leg-requests", type=int, default=48,
                    help="requests of the short serving leg of the default run (0: none)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: the slab solver runs on a single MI355X; "
              "run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    if args.serve:
        return serve_bench(args)

    import torch
    import paper_1802_09277_amd as sth
    import workloads as W

    cfg = W.CONFIGS[args.config]
    if args.slabs:
        # the same slab length and slab problem on fewer (or more) slabs
        import dataclasses
        cfg = dataclasses.replace(cfg, name=f"{cfg.name}-{args.slabs}slabs", n_slabs=args.slabs,
                                  T=cfg.T * args.slabs / cfg.n_slabs,
                                  note=f"{cfg.note}; cut to {args.slabs} slabs of the same length")
    sample_slabs = args.cpu_sample_slabs or min(4, cfg.n_slabs)
    # the CPU oracle runs in its own process beside the GPU part
    cpu_job = None if args.no_cpu_baseline else start_cpu_baseline(cfg, sample_slabs)
    torch.cuda.set_device(0)
    stream = torch.cuda.Stream()          # the solves run on a non-default stream
    torch.cuda.set_stream(stream)
    s = make_solver(cfg, args.prec, args)
    f = s.new_vector()
    s.load_rhs(cfg.modes(), f)
    u = s.new_vector()
    torch.cuda.synchronize()
    if args.copy_calibration_mib > 0:
        n = args.copy_calibration_mib * (1 << 20) // 8
        src = torch.ones(n, dtype=torch.float64, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        log(f"copy calibration: 3 copies of {n * 8} bytes")
        del src, dst

    # one untimed solve first: the first launch of each kernel loads its code,
    # which the per-class times below must not include
    u.zero_()
    s.solve(f, u, rtol=args.rtol, maxit=200)
    torch.cuda.synchronize()
    # warm-up with every kernel class timed on the finest level, to find the
    # dominant kernel class there (the coarser levels hold half the work)
    s.timing((1 << len(sth.KCLASS)) - 1, level=0)
    for _ in range(max(args.warmup, 1)):
        u.zero_()
        s.solve(f, u, rtol=args.rtol, maxit=200)
    totals = {k: s.timing_report(k) for k in sth.KCLASS}
    groups = merged_classes([k for k, v in totals.items() if v["launches"]])
    group_ms = {g: sum(totals[k]["ms"] for k in parts) for g, parts in groups.items()}
    dominant = max(group_ms, key=group_ms.get)
    log("warm-up kernel classes on the finest level (ms per solve): " +
        ", ".join(f"{g}={v / max(args.warmup, 1):.3f}" for g, v in group_ms.items()))
    s.timing(0)

    # timed region: K solves, eager launches with speculative cycles
    timed_solves(s, f, u, args, 1)
    ms, iters, relres = timed_solves(s, f, u, args, args.steps)
    u_head = u.clone()

    # roofline pass: the same K solves with HIP events around every launch
    # of the dominant kernel class on the finest level (events need
    # individually launched kernels)
    parts = groups[dominant]
    mask = 0
    for k in parts:
        mask |= 1 << sth.KCLASS[k]
    s.timing(mask, level=0)
    ms_events, _, _ = timed_solves(s, f, u, args, args.steps)
    rep = report_sum(s, parts)
    s.timing(0)
    bound = CLASS_BOUND[dominant]
    if bound == "mfma":
        peak_key = {"fp64": "fp64", "fp32": "fp32", "bf16x3": "bf16"}[args.prec]
        products = 3.0 if args.prec == "bf16x3" else 1.0      # three bf16 MFMA products per product
        achieved = products * rep["flops"] / (rep["ms"] * 1e-3)
        peak = PEAKS[peak_key]
        roof = {"bound": "mfma", "achieved": achieved / 1e12, "peak": peak / 1e12, "unit": "TFLOP/s"}
        roof["algorithmic_flops_per_launch"] = rep["flops"] / max(rep["launches"], 1)
    else:
        achieved = rep["bytes"] / (rep["ms"] * 1e-3)
        roof = {"bound": "hbm", "achieved": achieved / 1e9, "peak": PEAKS["hbm"] / 1e9, "unit": "GB/s"}
        roof["algorithmic_bytes_per_launch"] = rep["bytes"] / max(rep["launches"], 1)
    roof["frac"] = roof["achieved"] / roof["peak"]
    roof["traffic"] = measured_traffic(cfg.name, args.basis, args.prec, dominant)
    roof["kernel_class"] = dominant
    roof["level"] = 0
    roof["launches_per_step"] = rep["launches"] / args.steps
    roof["mean_launch_us"] = rep["ms"] * 1e3 / max(rep["launches"], 1)
    roof["events_pass_ms_per_step"] = ms_events
    levels, coarse_slabs = s.num_levels, s.coarse_slabs
    level_elems = [s.level_elems(l) for l in range(levels)]
    s.close()

    forms = {args.prec: {"value": cfg.unknowns / (ms * 1e-3), "ms_per_step": ms, "v_cycles": iters,
                         "final_relres": relres}}
    if not args.no_precision_forms and args.basis == "eigen":
        # the same solve with reduced-precision transforms, error against the headline result
        for prec in ("fp64", "fp32", "bf16x3"):
            if prec == args.prec:
                continue
            sp = make_solver(cfg, prec, args)
            up = sp.new_vector()
            timed_solves(sp, f, up, args, max(args.warmup, 1))
            msp, itp, rrp = timed_solves(sp, f, up, args, args.steps)
            err = float(torch.linalg.vector_norm(up - u_head) / torch.linalg.vector_norm(u_head))
            sp.close()
            del up
            forms[prec] = {"value": cfg.unknowns / (msp * 1e-3), "ms_per_step": msp, "v_cycles": itp,
                           "final_relres": rrp, f"rel_diff_vs_{args.prec}": err}
            log(f"precision form {prec}: {msp:.2f} ms per solve, {itp} cycles, relres {rrp:.2e}, "
                f"|u - u_{args.prec}| / |u_{args.prec}| {err:.2e}")

    out = {
        "metric": METRIC,
        "value": cfg.unknowns / (ms * 1e-3),
        "unit": "DOF/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if args.prec == "fp64" else f"f64+{args.prec}",
        "data": "synthetic",
        "config": {
            "workload": cfg.note,
            "name": cfg.name,
            "unknowns": cfg.unknowns,
            "coefficients_incl_dirichlet": cfg.coefficients,
            "theta": cfg.theta,
            "transform_prec": args.prec,
            "iterate_basis": args.basis,
            "v_cycles": iters,
            "final_relres": relres,
            "levels": levels,
            "coarse_slabs": coarse_slabs,
            "space_ratio": args.space_ratio,
            "minres_iters": args.minres_iters,
            "level_elems": level_elems,
            "speculative_cycles": not args.no_speculate,
        },
        "precision_forms": forms,
        "roofline": roof,
    }
    if args.serve_leg_requests > 0:
        # a short serving leg (the C5 request mix, one Poisson load at 0.8 of
        # the measured saturation rate): p50/p99 latency beside the throughput
        torch.cuda.synchronize()
        sv = serve_measure(args.serve_leg_requests, args.serve_slots, args.serve_budget_gib, args.basis, (0.8,),
                           args.serve_graphs, args.serve_prec)
        out["serving"] = sv
    if cpu_job is not None:
        out["cpu_baseline"] = finish_cpu_baseline(cfg, sample_slabs, cpu_job, args.cpu_limit_s)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
