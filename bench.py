"""Benchmark: square Poisson solve (F_T -> U), n = 4096, FP64, on one MI355X.

One step = one full solve through the C ABI: the J-step iterate of Algorithm 2 from
the n^2 Chebyshev coefficients of F to the (n+2)^2 of U, as four dense products in
the eigenbasis of A~.  Inputs are resident in HBM before timing starts.
Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "dof/s, square Poisson n=4096 at rel err ≤1e-12; % of HBM roofline"
HBM_PEAK_GBS = 8000.0
FP64_MFMA_PEAK_TFLOPS = 78.6  # dense FP64 matrix peak of MI355X


def output_zero_share(n, s):
    """Share of the output map's parity-s block that the products skip: the
    coefficients k of mode x that decay like J_k(x) below 2e-19, by groups of 64."""
    m, mo = (n - s + 1) // 2, (n + 3 - s) // 2
    cut = 0
    for b0 in range(0, mo, 64):
        k, lo = float(2 * b0 + s), 0.0
        hi = k
        for _ in range(60 if k > 0 else 0):
            x = 0.5 * (lo + hi)
            t = x / k
            if k * (math.acosh(1.0 / t) - math.sqrt(1.0 - t * t)) >= 43.0:
                lo = x
            else:
                hi = x
        a = min(m, max(0, math.floor(lo / math.pi - 0.5 * (s + 1))))
        cut += (a // 32 * 32) * min(64, mo - b0)
    return cut / (m * mo)


def product_flops(n):
    """Operations of the four product launches of one Chebyshev-output square
    solve, per launch: the parity blocks' dense products (m modes and mo
    output coefficients per parity), less the skipped zeros of the output map."""
    m = ((n + 1) // 2, n // 2)
    mo = ((n + 3) // 2, (n + 2) // 2)
    z = [1.0 - output_zero_share(n, s) for s in (0, 1)]
    st = [(s, t) for s in (0, 1) for t in (0, 1)]
    return [sum(2.0 * m[s] * m[t] * m[t] for s, t in st), sum(2.0 * m[s] * m[s] * m[t] for s, t in st),
            sum(2.0 * m[s] * m[t] * mo[t] * z[t] for s, t in st),
            sum(2.0 * m[s] * mo[s] * mo[t] * z[s] for s, t in st)]


def product_roofline(n, times_ms):
    """Roofline of the solve's dominant kernel, the FP64 matrix-core product
    (k_gemm): four launches per solve, times_ms their event-timed durations
    in launch order over one or more solves."""
    fl = product_flops(n)
    per = [sum(times_ms[i::4]) / max(len(times_ms[i::4]), 1) for i in range(4)]
    tf = sum(fl) / (sum(per) * 1e-3) / 1e12
    return {"bound": "mfma_f64", "achieved": round(tf, 2), "peak": FP64_MFMA_PEAK_TFLOPS,
            "unit": "TFLOP/s", "frac": round(tf / FP64_MFMA_PEAK_TFLOPS, 4), "traffic": None,
            "traffic_note": "the solve is four dense products bound by the FP64 matrix cores; no HBM "
                            "counters were taken",
            "kernel": "eigenbasis products (k_gemm), four launches per solve",
            "flops_per_launch": fl, "avg_launch_us": [round(t * 1e3, 2) for t in per],
            "launches_timed": len(times_ms),
            "timing": "HIP events recording each dispatch's start and end (hipExtLaunchKernelGGL), "
                      "separate pass of the same solves"}


def bench_sweeps(fps, torch, plan, G, ws):
    """The ADI half-sweeps of the stage entry point fps_adi_native (half-step 1
    reads its input and writes its output, 16 B per dof; half-step 2 also reads
    G, 24 B), every launch event-timed on one stream."""
    n = plan.n
    Y = torch.empty((n, n), dtype=torch.float64, device=G.device)
    fps.adi_native(plan, G, out=Y, ws=ws)
    plan.set_sweep_timing(2 * plan.J)
    fps.adi_native(plan, G, out=Y, ws=ws)
    torch.cuda.synchronize()
    t = plan.sweep_time()
    plan.set_sweep_timing(0)
    dof = float(n) * n
    t1 = sum(t[0::2]) / max(len(t[0::2]), 1) * 1e-3
    t2 = sum(t[1::2]) / max(len(t[1::2]), 1) * 1e-3
    b1, b2 = 16.0 * dof, 24.0 * dof
    return {"n": n, "bytes_per_launch": {"half_step_1": b1, "half_step_2": b2},
            "avg_launch_us": {"half_step_1": round(t1 * 1e6, 2), "half_step_2": round(t2 * 1e6, 2)},
            "achieved_GBs": round((b1 + b2) / (t1 + t2) / 1e9, 1),
            "frac": round((b1 + b2) / (t1 + t2) / 1e9 / HBM_PEAK_GBS, 4),
            "traffic": None, "launches_timed": len(t)}


def copy_rate(torch, dev, mib=1024, reps=5):
    """Achievable HBM rate of a plain copy kernel: GB/s (bytes read plus
    bytes written) of a device-to-device copy of `mib` MiB, far larger than
    the last-level cache."""
    nbytes = mib << 20
    src = torch.ones(nbytes // 8, dtype=torch.float64, device=dev)
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        dst.copy_(src)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    del src, dst
    torch.cuda.empty_cache()
    return 2.0 * nbytes / (ms * 1e-3) / 1e9


def stream_rate(fps, torch, dev, mib=1024, reps=5):
    """Achievable HBM rate of the library's own streaming pass
    (fps.probe_stream: c = a + b, two reads and one write per element in
    16-byte accesses) on three arrays of `mib` MiB each, far larger than the
    last-level cache: GB/s of bytes read plus bytes written."""
    nel = (mib << 20) // 8
    a = torch.ones(nel, dtype=torch.float64, device=dev)
    b = torch.full((nel,), 2.0, dtype=torch.float64, device=dev)
    c = torch.empty_like(a)
    fps.probe_stream(a, b, c)
    torch.cuda.synchronize()
    ok = bool((c[:: max(1, nel // 4096)] == 3.0).all())
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        fps.probe_stream(a, b, c)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    del a, b, c
    torch.cuda.empty_cache()
    return {"GBs": round(3.0 * nel * 8 / (ms * 1e-3) / 1e9, 1), "array_MiB": mib, "arrays": 3,
            "us_per_pass": round(ms * 1e3, 2), "result_ok": ok}


def host_info():
    """The host the oracle runs on: CPU model, logical CPUs this process may
    use, and the BLAS library numpy and scipy call with its thread count."""
    model = None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        cpus = len(os.sched_getaffinity(0))
    except AttributeError:
        cpus = os.cpu_count()
    blas = []
    try:
        import threadpoolctl
        for d in threadpoolctl.threadpool_info():
            blas.append({k: d.get(k) for k in ("user_api", "internal_api", "version",
                                               "num_threads", "threading_layer", "architecture")})
    except Exception as exc:  # threadpoolctl missing or failing: say so
        blas.append({"error": repr(exc)})
    threads = max([d.get("num_threads") or 1 for d in blas if "num_threads" in d] or [1])
    return {"cpu_model": model, "cpus_available": cpus, "blas": blas, "blas_threads": threads}


def time_oracle(fn, reps=3):
    """One warm-up call, then `reps` timed calls: (median seconds, all times,
    the warm-up call's result)."""
    import statistics
    res = fn()
    times = []
    for _ in range(reps):
        t0 = time.perf_counter()
        fn()
        times.append(time.perf_counter() - t0)
    return statistics.median(times), times, res


_CUBE_ORACLE = {}


def cube_oracle(F_host, n):
    """The oracle's cube solution for the benchmark's cube input (computed
    once per run and shared by the cube forms), with its timing: warm-up
    plus the median of three solves."""
    if n not in _CUBE_ORACLE:
        from oracle import cube
        med, times, Uo = time_oracle(lambda: cube.poisson_cube(F_host))
        _CUBE_ORACLE[n] = (Uo, med, times)
    return _CUBE_ORACLE[n]


def graph_timing(fps, torch, p, F, U_eager, steps):
    """The same solve captured into one HIP graph (fps.SolveGraph): ms per
    replay and whether the replay equals the eager result bit for bit.  The
    capture removes the host's per-launch cost, which shows where a solve
    issues many short launches."""
    g = fps.SolveGraph(p)
    g.F.copy_(F)
    g.replay()
    torch.cuda.synchronize()
    same = bool(torch.equal(g.U, U_eager))
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        g.replay()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    del g
    torch.cuda.empty_cache()
    return ms, same


def calibration_copy(torch, dev, mib):
    """One device-to-device copy of a known size (HBM counter calibration)."""
    nbytes = mib << 20
    src = torch.ones(nbytes // 8, dtype=torch.float64, device=dev)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    dst.copy_(src)
    torch.cuda.synchronize()
    del src, dst
    print(f"# calibration copy {nbytes} bytes read + {nbytes} bytes written", file=sys.stderr)


def bench_batch(fps, workloads, torch, tol, reps=3, tight=True):
    """256 independent square solves (n_b = 32 U{1..32}, seed 1): one graph
    launch per batch (FP64 and FP32-refined) against a sequential loop of
    single FP64 solves, run eagerly and replayed from one HIP graph per
    solve."""
    import numpy as np
    ns, Fs = workloads.batched_problems()
    dof = float(sum(n * n for n in ns))
    res = {"problems": len(ns), "dof": dof,
           "enclosure": "computed spectrum" if tight else "Lemma B.1"}
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)

    def timed(fn, k):
        fn()
        torch.cuda.synchronize()
        ev0.record()
        for _ in range(k):
            fn()
        ev1.record()
        torch.cuda.synchronize()
        return ev0.elapsed_time(ev1) / k

    # sequential single FP64 solves (the same inputs, one plan per size)
    plans = {n: fps.plan(n, tol=tol, tight=tight) for n in sorted(set(ns))}
    ws = torch.empty(max(p.workspace_bytes for p in plans.values()), dtype=torch.uint8,
                     device="cuda")
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    Us = [torch.empty(plans[n].out_shape(), dtype=torch.float64, device="cuda") for n in ns]

    def seq():
        for n, F, U in zip(ns, Fd, Us):
            fps.solve(plans[n], F, out=U, ws=ws)
    t_seq = timed(seq, 1)
    res["sequential_fp64_ms"] = t_seq
    # the same solves, each captured into its own HIP graph (no host launch
    # cost inside a solve): the device-side baseline of the batched launches
    graphs = []
    for n, F in zip(ns, Fd):
        g1 = fps.SolveGraph(plans[n])
        g1.F.copy_(F)
        graphs.append(g1)

    def seq_graphs():
        for g1 in graphs:
            g1.replay()
    t_seq_graph = timed(seq_graphs, reps)
    res["sequential_fp64_graph_equals_eager"] = all(
        bool(torch.equal(g1.U, U)) for g1, U in zip(graphs, Us))
    res["sequential_fp64_graph_ms"] = t_seq_graph
    del graphs
    for prec in ("fp64", "fp32_refined"):
        b = fps.batch(ns, tol=tol, precision=prec, tight=tight)
        g = fps.BatchGraph(b)
        g.F.copy_(b.pack(Fs))
        t = timed(g.replay, reps)
        r = {"ms_per_batch": t, "dof_per_s": dof / (t * 1e-3), "speedup_vs_sequential_fp64":
             t_seq / t, "speedup_vs_sequential_fp64_graph": t_seq_graph / t, "max_J": b.max_J,
             "launch": "one HIP graph"}
        got = b.unpack(g.U)
        worst = 0.0
        for U, Ub in zip(Us, got):
            d = float(torch.linalg.norm(Ub - U) / torch.linalg.norm(U))
            worst = max(worst, d)
        r["max_rel_diff_vs_sequential_fp64"] = worst
        res[prec] = r
        del g, b
    del ws
    torch.cuda.empty_cache()
    return res


def cube_roofline(p, fps, torch, F, U, ws):
    """One cube solve with an event pair around every product launch: total
    time and the rate of its products (per axis and direction 2 n^3 times the
    parity block's length n/2)."""
    p.set_sweep_timing(64)
    fps.solve(p, F, out=U, ws=ws)
    torch.cuda.synchronize()
    t = p.sweep_time()
    p.set_sweep_timing(0)
    flops = 6.0 * float(p.n) ** 4
    tf = flops / (sum(t) * 1e-3) / 1e12
    return {"bound": "mfma_f64", "flops": flops, "launches_timed": len(t),
            "ms_total": round(sum(t), 4), "achieved_TFLOPs": round(tf, 2),
            "frac": round(tf / FP64_MFMA_PEAK_TFLOPS, 4)}


def bench_cube(fps, workloads, torch, tol, n=256, steps=5, check=True, tight=True):
    """Cube n^3 solve (two-level nested ADI's iterate, FP64): time per solve
    and its products' rate."""
    import numpy as np
    F_host = workloads.cube_rhs(n)
    F = torch.from_numpy(F_host).cuda()
    p = fps.plan(n, tol=tol, dim=3, tight=tight)
    counts = p.inner_counts()
    ws = fps.workspace(p, "cuda")
    U = torch.empty(p.out_shape(), dtype=torch.float64, device="cuda")
    fps.solve(p, F, out=U, ws=ws)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        fps.solve(p, F, out=U, ws=ws)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    dof = float(n) ** 3
    res = {"n": n, "dof": dof, "ms_per_solve": ms, "dof_per_s": dof / (ms * 1e-3),
           "enclosure": "computed spectrum" if tight else "Lemma B.1",
           "J_outer": p.J, "inner_steps": sum(counts),
           "products": cube_roofline(p, fps, torch, F, U, ws)}
    if check:
        Uo = cube_oracle(F_host, n)[0]
        Ug = U.cpu().numpy()
        res["rel_frobenius_err_vs_oracle"] = float(np.linalg.norm(Ug - Uo) / np.linalg.norm(Uo))
        res["max_abs_ratio_vs_oracle"] = float(np.abs(Ug - Uo).max() / np.abs(Uo).max())
    del ws
    torch.cuda.empty_cache()
    return res


def bench_cube_zeig(fps, workloads, torch, tol, n=256, steps=3, check=True, tight=True):
    """Cube n^3 solve by the z-eigenbasis method (one ADI per z-slice, FP64, and
    its refined form): time per solve and its products' rate."""
    import numpy as np
    F_host = workloads.cube_rhs(n)
    F = torch.from_numpy(F_host).cuda()
    p = fps.plan(n, tol=tol, dim=3, tight=tight, zeig=True)
    counts = p.slice_counts()
    ws = fps.workspace(p, "cuda")
    U = torch.empty(p.out_shape(), dtype=torch.float64, device="cuda")
    fps.solve(p, F, out=U, ws=ws)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        fps.solve(p, F, out=U, ws=ws)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    ms_g, same_g = graph_timing(fps, torch, p, F, U, steps)
    dof = float(n) ** 3
    res = {"n": n, "dof": dof, "ms_per_solve": ms, "dof_per_s": dof / (ms * 1e-3),
           "enclosure": "computed spectrum" if tight else "Lemma B.1",
           "method": "products into the tensor eigenbasis of A~, the slice iterations' multiplier, "
                     "products out",
           "slice_steps": sum(counts), "max_slice_J": max(counts) if counts else 0,
           "products": cube_roofline(p, fps, torch, F, U, ws),
           "hip_graph": {"ms_per_solve": ms_g, "dof_per_s": dof / (ms_g * 1e-3),
                         "equals_eager": same_g}}
    # the refined form's iterate (rounds of the K-form slice correction)
    pr = fps.plan(n, tol=tol, dim=3, tight=tight, zeig=True, precision="fp32_refined")
    wsr = fps.workspace(pr, "cuda")
    Ur = torch.empty(pr.out_shape(), dtype=torch.float64, device="cuda")
    fps.solve(pr, F, out=Ur, ws=wsr)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(steps):
        fps.solve(pr, F, out=Ur, ws=wsr)
    e1.record()
    torch.cuda.synchronize()
    ms_r = e0.elapsed_time(e1) / steps
    rsteps, rtols = pr.round_steps()
    res["fp32_refined"] = {"ms_per_solve": ms_r, "dof_per_s": dof / (ms_r * 1e-3),
                           "speedup_vs_fp64": ms / ms_r, "rounds": pr.rounds,
                           "round_max_slice_J": rsteps, "round_tols": rtols,
                           "round0_slice_steps": sum(pr.slice_counts())}
    if check:
        Uo, med, times = cube_oracle(F_host, n)
        Ug = U.cpu().numpy()
        res["rel_frobenius_err_vs_oracle"] = float(np.linalg.norm(Ug - Uo) / np.linalg.norm(Uo))
        res["max_abs_ratio_vs_oracle"] = float(np.abs(Ug - Uo).max() / np.abs(Uo).max())
        hi = host_info()
        res["cpu_baseline"] = {
            "value": dof / med, "unit": "dof/s", "cores": hi["blas_threads"], "kind": "oracle",
            "sample": f"full n={n} cube solves by the oracle (Kronecker eigenbasis: three "
                      f"mode products each way, numpy/OpenBLAS FP64), one warm-up then the "
                      f"median of {len(times)}: " + ", ".join(f"{t:.2f}" for t in times) + " s",
            "host": hi}
        Urh = Ur.cpu().numpy()
        res["fp32_refined"]["rel_frobenius_err_vs_oracle"] = float(
            np.linalg.norm(Urh - Uo) / np.linalg.norm(Uo))
        res["fp32_refined"]["max_abs_ratio_vs_oracle"] = float(
            np.abs(Urh - Uo).max() / np.abs(Uo).max())
    del ws, wsr
    torch.cuda.empty_cache()
    return res


def bench_rect_dirichlet(fps, workloads, torch, tol, n=4096, box=(0.0, 2.5, -1.0, 0.25), steps=5,
                         check=True, tight=True):
    """Rectangle [0, 2.5] x [-1, 0.25] with nonzero Dirichlet data (four random
    traces, corners matched), FP64: time per solve with the device-side lift,
    and the same plan's zero-data solve for the lift's overhead."""
    import numpy as np
    F_host, bc_host = workloads.rect_dirichlet_case(n, seed=5)
    F = torch.from_numpy(F_host).cuda()
    bc = torch.from_numpy(bc_host).cuda()
    p = fps.plan(n, tol=tol, box=box, tight=tight, dirichlet=True)
    ws = fps.workspace(p, "cuda")
    U = torch.empty(p.out_shape(), dtype=torch.float64, device="cuda")

    def timed(fn):
        fn()
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(steps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / steps

    ms_d = timed(lambda: fps.solve_dirichlet(p, F, bc, out=U, ws=ws))
    Ud = U.cpu().numpy()
    ms_0 = timed(lambda: fps.solve(p, F, out=U, ws=ws))
    res = {"n": n, "box": list(box), "dof": float(n) ** 2, "J": p.J,
           "ms_per_solve": ms_d, "dof_per_s": n * n / (ms_d * 1e-3),
           "ms_zero_data_same_plan": ms_0, "lift_overhead_ms": ms_d - ms_0,
           "enclosure": "computed spectrum" if tight else "Lemma B.1",
           "shifts": "general (p_j != -q_j): two tables per step"}
    if check:
        from oracle import rect
        Uo = rect.poisson_rect_dirichlet(F_host, bc_host, box)
        res["rel_frobenius_err_vs_oracle"] = float(np.linalg.norm(Ud - Uo) / np.linalg.norm(Uo))
        tr = rect.boundary_traces(Ud)
        res["max_trace_err"] = float(max(np.abs(a - b).max() for a, b in zip(tr, bc_host)))
    del ws
    torch.cuda.empty_cache()
    return res


def bench_cylinder(fps, workloads, torch, n=256, n_theta=256, steps=5, check=True):
    """Cylinder (Sec. 4.1), n Chebyshev coefficients in r and z, n_theta
    Fourier modes, FP64: time per solve (the per-mode systems solved
    exactly in the z-eigenbasis), plan time, and the oracle's per-mode
    solution on a sample of modes covering the three cases."""
    import time as _t
    import numpy as np
    F_host = workloads.cylinder_rhs(n, n_theta, seed=9)
    F = torch.from_numpy(np.ascontiguousarray(np.stack([F_host.real, F_host.imag], axis=1))).cuda()
    t0 = _t.perf_counter()
    p = fps.plan_cylinder(n, n_theta)
    t_plan = _t.perf_counter() - t0
    ws = fps.workspace(p, "cuda")
    U = torch.empty(p.out_shape(), dtype=torch.float64, device="cuda")
    fps.solve(p, F, out=U, ws=ws)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        fps.solve(p, F, out=U, ws=ws)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    ms_g, same_g = graph_timing(fps, torch, p, F, U, steps)
    dof = float(n) * n * n_theta
    # Whole-solve rooflines.  MFMA: the four maps of the modes' own r parity (n <=
    # 256), 4 n_theta n^3 flops (z and r, in and out, n_theta n^3 each, parity
    # blocks).  HBM: every stage reads its operands and writes its result once: F's
    # rows of one parity, right-hand sides written, the banded solves reading five
    # fields of the factor table (the other three only where rows were exchanged) and
    # the right-hand sides twice and writing them and the solution, the solution read,
    # U written.
    x = float(n_theta) * 2 * (n // 2) * n * 8
    flops = 4.0 * n_theta * float(n) ** 3
    hbm = 2 * x + (n_theta // 2 + 1) * 5.0 * (n // 2) * n * 8 + 4 * x + x + U.numel() * 8.0
    res = {"n": n, "n_theta": n_theta, "dof": dof, "ms_per_solve": ms,
           "dof_per_s": dof / (ms * 1e-3), "plan_s": round(t_plan, 2),
           "hip_graph": {"ms_per_solve": ms_g, "dof_per_s": dof / (ms_g * 1e-3),
                         "equals_eager": same_g},
           "method": "z-eigenbasis of A~, host-factored banded r-solves per (mode, z column), "
                     "MFMA GEMM maps",
           "roofline_whole_solve": {
               "hbm_bytes_algorithmic": hbm, "hbm_GBs": round(hbm / (ms * 1e-3) / 1e9, 1),
               "hbm_frac": round(hbm / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
               "mfma_flops": flops, "TFLOPs": round(flops / (ms * 1e-3) / 1e12, 2),
               "fp64_mfma_frac": round(flops / (ms * 1e-3) / 1e12 / FP64_MFMA_PEAK_TFLOPS, 4)}}
    if check:
        from oracle import cylinder
        Ug = U.cpu().numpy()
        worst = 0.0
        for k in (0, 1, -1, 2, -3, 17, n_theta // 4, -(n_theta // 2), n_theta // 2 - 1):
            idx = k + n_theta // 2
            Uo = (cylinder.solve_mode(np.ascontiguousarray(F_host[idx].real), k)
                  + 1j * cylinder.solve_mode(np.ascontiguousarray(F_host[idx].imag), k))
            Uk = Ug[idx, 0] + 1j * Ug[idx, 1]
            worst = max(worst, float(np.linalg.norm(Uk - Uo) / np.linalg.norm(Uo)))
        res["rel_err_vs_oracle_sampled_modes"] = worst
    del ws
    torch.cuda.empty_cache()
    return res


def bench_square_large(fps, workloads, torch, tol, n=10000, steps=3, check=True, tight=True):
    """The square at n = 10^4 (10^8 dof, the size of the paper's own timing
    example): time per FP64 solve and the error against the oracle's exact
    discrete solution."""
    import numpy as np
    F_host = workloads.square_rhs(n, seed=0)
    F = torch.from_numpy(F_host).cuda()
    p = fps.plan(n, tol=tol, tight=tight)
    ws = fps.workspace(p, "cuda")
    U = torch.empty(p.out_shape(), dtype=torch.float64, device="cuda")
    fps.solve(p, F, out=U, ws=ws)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        fps.solve(p, F, out=U, ws=ws)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    p.set_sweep_timing(4)
    fps.solve(p, F, out=U, ws=ws)
    torch.cuda.synchronize()
    t = p.sweep_time()
    p.set_sweep_timing(0)
    dof = float(n) * n
    res = {"n": n, "dof": dof, "J": p.J, "ms_per_solve": ms,
           "dof_per_s": dof / (ms * 1e-3),
           "paper_context": "10^8 dof in under two minutes on a 2017 laptop (MATLAB, one core)",
           "products": product_roofline(n, t), "sweep": bench_sweeps(fps, torch, p, F, ws)}
    fps.solve(p, F, out=U, ws=ws)
    if check:
        from oracle import square
        Uo = square.poisson_square(F_host)
        Ug = U.cpu().numpy()
        res["rel_frobenius_err_vs_oracle"] = float(np.linalg.norm(Ug - Uo) / np.linalg.norm(Uo))
        res["max_abs_ratio_vs_oracle"] = float(np.abs(Ug - Uo).max() / np.abs(Uo).max())
    del ws, U, F
    torch.cuda.empty_cache()
    return res


def bench_adjoint(fps, workloads, torch, tol, n=2048, batch=16, steps=3, check=True, tight=True):
    """Differentiation form: one forward and one backward pass of the autograd
    solve over a batch of 16 right-hand sides at n = 2048, for the quadratic
    loss ||U(F) - U*||^2 (U* the solution for a fixed target right-hand side).
    The backward pass is the adjoint solve (the transposed products in reverse
    order); nothing is stored from the forward pass."""
    import numpy as np
    F_host, Fstar, _ = workloads.adjoint_case(n, batch, n_dirs=1)
    p = fps.plan(n, tol=tol, tight=tight)
    Ustar = fps.solve(p, torch.from_numpy(Fstar).cuda())
    F = torch.from_numpy(F_host).cuda().requires_grad_(True)

    def step():
        F.grad = None
        U = fps.solve_fn(F, p)
        loss = ((U - Ustar) ** 2).sum()
        loss.backward()
        return U

    step()
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps):
        U = step()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    dof = float(batch) * n * n
    flops = 2.0 * batch * sum(product_flops(n))  # eight product launches
    res = {"n": n, "batch": batch, "J": p.J, "ms_per_fwd_bwd": ms,
           "dof_per_s": dof / (ms * 1e-3),
           "product_flops": flops,
           "product_TFLOPs_whole_step": round(flops / (ms * 1e-3) / 1e12, 2),
           "method": "autograd Function over one fps_batch: forward fps_batch_solve, backward "
                     "fps_batch_solve_adjoint (the products of all problems in one launch per "
                     "stage)"}
    if check:
        from oracle import adjoint
        Ub = (2.0 * (U[0] - Ustar)).detach().cpu().numpy()
        ref = adjoint.vjp_square(Ub, np.asarray(p.shifts(), dtype=float))
        got = F.grad[0].cpu().numpy()
        res["rel_err_vs_oracle_vjp_problem0"] = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    del F, U, Ustar
    torch.cuda.empty_cache()
    return res


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--n", type=int, default=4096)
    ap.add_argument("--tol", type=float, default=1e-13)
    ap.add_argument("--enclosure", choices=["tight", "lemma"], default="tight",
                    help="shift intervals: computed spectrum (default) or the Lemma B.1 enclosure")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-check", action="store_true")
    ap.add_argument("--no-forms", action="store_true",
                    help="skip the FP32-refined, batched, cube, rectangle and cylinder timings")
    ap.add_argument("--only", choices=["fp32_refined", "batched", "cube", "cube_zeig",
                                       "rect_dirichlet", "cylinder", "adjoint", "square_n10000"],
                    help="run only this form and print its figures (profiling)")
    ap.add_argument("--copy-calib-mib", type=int, default=0,
                    help="run one device-to-device copy of this size first (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "the solver runs on one GPU; sharding across GPUs is not "
                                   "implemented"}))
        return 2

    import numpy as np
    import torch

    import paper_1710_11259_amd as fps
    import workloads

    n = args.n
    dev = torch.device("cuda:0")
    if args.only in ("batched", "cube", "cube_zeig", "rect_dirichlet", "cylinder", "adjoint",
                     "square_n10000"):
        if args.copy_calib_mib:
            calibration_copy(torch, dev, args.copy_calib_mib)
        tight = args.enclosure == "tight"
        if args.only == "batched":
            res = bench_batch(fps, workloads, torch, args.tol, tight=tight)
        elif args.only == "cube":
            res = bench_cube(fps, workloads, torch, args.tol, steps=max(1, args.steps),
                             check=not args.no_check, tight=tight)
        elif args.only == "cylinder":
            res = bench_cylinder(fps, workloads, torch, steps=max(1, args.steps),
                                 check=not args.no_check)
        elif args.only == "rect_dirichlet":
            res = bench_rect_dirichlet(fps, workloads, torch, args.tol, n=n,
                                       steps=max(1, args.steps), check=not args.no_check,
                                       tight=tight)
        elif args.only == "adjoint":
            res = bench_adjoint(fps, workloads, torch, args.tol, steps=max(1, args.steps),
                                check=not args.no_check, tight=tight)
        elif args.only == "square_n10000":
            res = bench_square_large(fps, workloads, torch, args.tol, steps=max(1, args.steps),
                                     check=not args.no_check, tight=tight)
        else:
            res = bench_cube_zeig(fps, workloads, torch, args.tol, steps=max(1, args.steps),
                                  check=not args.no_check, tight=tight)
        print(json.dumps({"form": args.only, **res}), flush=True)
        return 0
    F_host = workloads.square_rhs(n, seed=0)
    F = torch.from_numpy(F_host).to(dev)
    tight = args.enclosure == "tight"
    plan = fps.plan(n, tol=args.tol, tight=tight)
    ws = fps.workspace(plan, dev)
    U = torch.empty(plan.out_shape(), dtype=torch.float64, device=dev)
    print(f"# plan n={n} J={plan.J} ws={plan.workspace_bytes / 2**20:.1f} MiB", file=sys.stderr,
          flush=True)

    if args.copy_calib_mib:
        calibration_copy(torch, dev, args.copy_calib_mib)

    for _ in range(args.warmup):
        fps.solve(plan, F, out=U, ws=ws)
    torch.cuda.synchronize()

    stream = torch.cuda.current_stream(dev)
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    # Timed region: exactly `steps` solves, no instrumentation.
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(args.steps):
        fps.solve(plan, F, out=U, ws=ws)
    e1.record(stream)
    torch.cuda.synchronize()
    total_ms = e0.elapsed_time(e1)
    # Roofline pass: the same solves again, every product launch carrying a HIP
    # event pair that records the dispatch's own start and end.
    plan.set_sweep_timing(4 * args.steps)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(args.steps):
        fps.solve(plan, F, out=U, ws=ws)
    e1.record(stream)
    torch.cuda.synchronize()
    instr_ms = e0.elapsed_time(e1)
    products = plan.sweep_time()
    plan.set_sweep_timing(0)
    ms_per_step = total_ms / args.steps
    dof = float(n) * float(n)
    value = dof / (ms_per_step * 1e-3)
    J = plan.J
    roofline = product_roofline(n, products)
    roofline["share_of_step"] = round(sum(products) / instr_ms, 4)
    # the stage entry point's half-sweeps (HBM bound) and the streaming rate
    ceiling = stream_rate(fps, torch, dev)
    roofline["copy_kernel_GBs"] = round(copy_rate(torch, dev), 1)
    roofline["stream_kernel"] = ceiling
    sw = bench_sweeps(fps, torch, plan, F, ws)
    sw["frac_of_stream_kernel"] = round(sw["achieved_GBs"] / ceiling["GBs"], 4)
    roofline["adi_native_sweeps"] = sw

    out = {"metric": METRIC, "value": value, "unit": "dof/s", "n_gpus": 1,
           "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
           "data": "synthetic",
           "config": {"workload": f"square [-1,1]^2 Poisson, zero Dirichlet, n={n} "
                                  f"({n}x{n} Chebyshev coefficients of f, "
                                  f"N(0,1)(1+j)^-2(1+k)^-2, seed 0), FP64, tol {args.tol:g}, "
                                  f"J={J} (shift intervals: "
                                  f"{'computed spectrum of A~' if tight else 'Lemma B.1 enclosure'}), "
                                  "one right-hand side",
                      "n": n, "J": J, "tol": args.tol,
                      "enclosure": "computed spectrum" if tight else "Lemma B.1"},
           "roofline": roofline}

    forms = {}
    if not args.no_forms or args.only == "fp32_refined":
        po = fps.plan(n, tol=args.tol, tight=not tight)
        wso = fps.workspace(po, dev)
        Uo_ = torch.empty(po.out_shape(), dtype=torch.float64, device=dev)
        fps.solve(po, F, out=Uo_, ws=wso)
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(args.steps):
            fps.solve(po, F, out=Uo_, ws=wso)
        e1.record(stream)
        torch.cuda.synchronize()
        ms_o = e0.elapsed_time(e1) / args.steps
        forms["lemma_enclosure" if tight else "computed_spectrum"] = {
            "ms_per_step": ms_o, "dof_per_s": dof / (ms_o * 1e-3), "J": po.J}
        del wso, Uo_
        # Precision form: the iterate of the refinement's rounds (in float64), same workload and tol.
        pr = fps.plan(n, tol=args.tol, precision="fp32_refined", tight=tight)
        wsr = fps.workspace(pr, dev)
        Ur = torch.empty(pr.out_shape(), dtype=torch.float64, device=dev)
        fps.solve(pr, F, out=Ur, ws=wsr)
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(args.steps):
            fps.solve(pr, F, out=Ur, ws=wsr)
        e1.record(stream)
        torch.cuda.synchronize()
        ms_r = e0.elapsed_time(e1) / args.steps
        rsteps, rtols = pr.round_steps()
        forms["fp32_refined"] = {"ms_per_step": ms_r, "dof_per_s": dof / (ms_r * 1e-3),
                                 "speedup_vs_fp64": ms_per_step / ms_r,
                                 "rounds": pr.rounds, "round_steps": rsteps, "round_tols": rtols,
                                 "fp64_J": J}
        del wsr
        if args.only is None:
            forms["batched"] = bench_batch(fps, workloads, torch, args.tol, tight=tight)
            forms["cube"] = bench_cube(fps, workloads, torch, args.tol, check=not args.no_check,
                                       tight=tight)
            forms["cube_zeig"] = bench_cube_zeig(fps, workloads, torch, args.tol,
                                                 check=not args.no_check, tight=tight)
            forms["rect_dirichlet"] = bench_rect_dirichlet(fps, workloads, torch, args.tol, n=n,
                                                           check=not args.no_check, tight=tight)
            forms["cylinder"] = bench_cylinder(fps, workloads, torch, check=not args.no_check)
            forms["adjoint"] = bench_adjoint(fps, workloads, torch, args.tol,
                                             check=not args.no_check, tight=tight)
            forms["square_n10000"] = bench_square_large(fps, workloads, torch, args.tol,
                                                        check=not args.no_check, tight=tight)
    if forms:
        out["forms"] = forms

    Ug = U.cpu().numpy()
    if not args.no_cpu_baseline or not args.no_check:
        from oracle import square

        def oracle_solve():
            # the oracle's square solve (poisson_square), keeping its native X
            Xo_ = square.solve_native(square.rhs_ct(F_host))
            return Xo_, square.to_chebyshev(Xo_)

        if args.no_cpu_baseline:
            Xo, Uo = oracle_solve()
        else:
            t_cpu, t_all, (Xo, Uo) = time_oracle(oracle_solve)
        err = float(np.linalg.norm(Ug - Uo) / np.linalg.norm(Uo))
        # the same comparison on X (a native-output plan, outside the timing)
        pn = fps.plan(n, tol=args.tol, out="native", tight=tight)
        Xg = fps.solve(pn, F).cpu().numpy()
        del pn
        out["accuracy"] = {"rel_frobenius_err_vs_oracle": err,
                           "max_abs_ratio_vs_oracle": float(np.abs(Ug - Uo).max() / np.abs(Uo).max()),
                           "native_X": {"rel_frobenius": float(np.linalg.norm(Xg - Xo)
                                                               / np.linalg.norm(Xo)),
                                        "max_abs_ratio": float(np.abs(Xg - Xo).max()
                                                               / np.abs(Xo).max())},
                           "bound": 1e-12, "ok": bool(err <= 1e-12)}
        if "fp32_refined" in forms:
            er = float(np.linalg.norm(Ur.cpu().numpy() - Uo) / np.linalg.norm(Uo))
            forms["fp32_refined"]["rel_frobenius_err_vs_oracle"] = er
        if not args.no_cpu_baseline:
            hi = host_info()
            out["cpu_baseline"] = {
                "value": dof / t_cpu, "unit": "dof/s", "cores": hi["blas_threads"],
                "kind": "oracle",
                "sample": f"full n={n} solves by the FP64 eigen-decomposition oracle "
                          f"(numpy/scipy/OpenBLAS), one warm-up then the median of "
                          f"{len(t_all)}: " + ", ".join(f"{t:.2f}" for t in t_all) + " s",
                "host": hi}
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
