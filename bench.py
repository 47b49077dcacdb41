#!/usr/bin/env python3
"""Throughput of the MI355X absolute-value preconditioned MINRES solver.

Workload (one "step"): the batched-shift configuration -- 64 complex-shifted
2-D systems (K + lambda_j I) z_j = f_j, 16 each on grids n = 63, 127, 255,
511, coefficient a = 1 + 0.5 sin(2 pi x) sin(2 pi y), shifts of an
alpha-circulant all-at-once time discretisation (tau = 1/64, gamma = 1e-2),
right-hand sides N(0,1) + i N(0,1), zero initial guess, stop at relative
residual 1e-8.  The step solves all 64 systems with one replay of a captured
hipGraph of the persistent solver kernel, FP32 sine transforms and mode
scaling in the preconditioner, FP64 everywhere else.  Inputs are resident in
HBM before timing starts.

Also measured (reported beside the main figure): the same 64 systems solved
one after another by the plain FP64 solver (one persistent launch each), the
HBM roofline fraction of the solver kernel, and the CPU oracle on a bounded
sample of the systems.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "MINRES solves/s at relres 1e-8: batched mixed-precision vs plain FP64, 1 GPU"
PEAK_HBM_GBS = 8000.0
# Algorithmic HBM bytes per grid point per MINRES iteration: what the method
# streams with one read of each operand and one write of each result per
# step: stencil 40 (z 16 in, a 8, A z 16 out) + Lanczos recurrence and w / x
# updates 160 (seven 16-byte reads, three writes) + p sine-transform passes
# of 4 s bytes (read + write of a complex value of s-byte parts; s = 8 FP64,
# 4 FP32 preconditioner).  p = 3 in 2-D and in 3-D with the plane phase (the
# plane of the two leading axes transformed in one pass), 5 in 3-D otherwise:
#   2-D FP64 296, 2-D FP32 248, 3-D plane FP64 296 and FP32 248,
#   3-D five-pass FP64 360 and FP32 280.


def bytes_model(d: int, fp32: bool, plane: bool = False) -> float:
    p = 3 if d == 2 or plane else 5
    return 200.0 + p * 4.0 * (4 if fp32 else 8)


# The same model with the w / x updates of two consecutive steps sharing one
# pass (what the solver does): 32 bytes less per iteration.
def bytes_model_paired(d: int, fp32: bool, plane: bool = False) -> float:
    return bytes_model(d, fp32, plane) - 32.0


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--plain-reps", type=int, default=2)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-sample", type=int, default=48,
                    help="systems of the batch timed with the CPU oracle")
    ap.add_argument("--count", type=int, default=64)
    ap.add_argument("--no-extra", action="store_true",
                    help="skip the other workloads (c1, c2, c3, adjoint)")
    ap.add_argument("--no-tune", action="store_true",
                    help="keep the creation-time batch schedule")
    ap.add_argument("--tile-points", type=int, default=0,
                    help="fix the batch schedule's tile size (skips the tuner)")
    ap.add_argument("--lds-bytes", type=int, default=0,
                    help="fix the batch schedule's LDS budget (skips the tuner)")
    ap.add_argument("--block-threads", type=int, default=0,
                    help="fix the batch solver's workgroup size, 256 or 512 (skips the tuner)")
    ap.add_argument("--batch-only", action="store_true",
                    help="time only the batched solve (for profiler runs)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run device-to-device copies of 1 GiB, the reference for the "
                         "HBM byte counters")
    ap.add_argument("--hbm-rates", action="store_true",
                    help="time plain device copies, fills and sums of 1 and 4 GiB: the HBM "
                         "rates that simple streaming kernels reach on this GPU")
    return ap.parse_args()


def copy_calibration():
    """Three device copies of 1 GiB (1 GiB read + 1 GiB written each): the
    reference that scales the FETCH_SIZE / WRITE_SIZE counters to bytes."""
    import torch
    n = (1 << 30) // 8
    src = torch.ones(n, dtype=torch.float64, device="cuda")
    dst = torch.empty_like(src)
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_read": 1 << 30, "copy_bytes_written": 1 << 30, "copies": 3}))


def hbm_rates():
    """HBM rates of plain streaming work (torch's own kernels, FP64 vectors of
    1 and 4 GiB, 20 timed calls each after 3 untimed): a copy (read + write), a
    fill (write only) and a sum (read only).  The scale against which the
    solver's measured traffic rate is read: 8 TB/s is the published peak, not
    what a streaming kernel reaches."""
    import torch
    out = {}
    for gib in (1, 4):
        n = (gib << 30) // 8
        a = torch.ones(n, dtype=torch.float64, device="cuda")
        b = torch.empty_like(a)
        cases = (("copy", lambda: b.copy_(a), 2 * n * 8), ("fill", lambda: b.fill_(1.5), n * 8),
                 ("sum", lambda: a.sum(), n * 8))
        for name, fn, nbytes in cases:
            for _ in range(3):
                fn()
            torch.cuda.synchronize()
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            reps = 20
            e0.record()
            for _ in range(reps):
                fn()
            e1.record()
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1) / reps
            tbs = nbytes / ms / 1e9
            out[f"{name}_{gib}GiB"] = {"ms": round(ms, 4), "TB/s": round(tbs, 3),
                                       "frac_of_8TBs": round(tbs * 1e3 / PEAK_HBM_GBS, 3)}
        del a, b
        torch.cuda.empty_cache()
    print(json.dumps(out))


KERNEL_SOURCES = ["paper_2408_00488_amd/csrc/csl_kernels.hip",
                  "paper_2408_00488_amd/csrc/csl_kernels_wg256h.hip",
                  "paper_2408_00488_amd/csrc/csl_kernels_wg512.hip",
                  "paper_2408_00488_amd/csrc/csl_kernels_wg512x.hip",
                  "paper_2408_00488_amd/csrc/csl_kernels_wg1024p.hip",
                  "paper_2408_00488_amd/csrc/csl_kernels_wg512p.hip",
                  "paper_2408_00488_amd/csrc/csl_team.hpp",
                  "paper_2408_00488_amd/csrc/csl_device.hpp",
                  "paper_2408_00488_amd/csrc/csl_common.hpp"]
TRAFFIC_FILE = "profiles/solve_kernel_batch64_hbm_traffic.txt"


def kernel_source_hash() -> str:
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def measured_traffic():
    """HBM bytes per launch from the committed rocprofv3 counter summary, if
    it was taken on the kernel source as it is now (else None)."""
    path = os.path.join(ROOT, TRAFFIC_FILE)
    if not os.path.exists(path):
        return None
    vals = {}
    for line in open(path):
        if ":" in line:
            k, v = line.split(":", 1)
            vals[k.strip()] = v.strip()
    if vals.get("kernel_source_sha256") != kernel_source_hash():
        return None
    try:
        return float(vals["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_threads() -> int:
    """Threads the oracle may use here: the cores this process may run on,
    at most 16 (the host share of one GPU on the measurement machines)."""
    return max(1, min(16, len(os.sched_getaffinity(0))))


def cpu_baseline(workload, systems_idx, gpu_solutions, threads):
    """Time the CPU oracle (NumPy/SciPy FP64) on a sample of the batch; the
    sample keeps the batch's mix of grid sizes.  threads = 1 holds every
    thread pool (BLAS, OpenMP, SciPy's FFT) to one thread; otherwise the
    pools and SciPy's FFT get `threads` workers."""
    import scipy.fft as sfft
    from threadpoolctl import threadpool_limits
    from oracle import csl_oracle as O
    t_total = 0.0
    errs = []
    iters = []
    with threadpool_limits(limits=threads), sfft.set_workers(threads):
        for j in systems_idx:
            s = workload.systems[j]
            t0 = time.perf_counter()
            po = O.Problem(s.a, s.lam.real, s.lam.imag)
            zo, io = po.solve(s.f, tol=1e-8)
            t_total += time.perf_counter() - t0
            iters.append(io["iters"])
            zg = gpu_solutions[j]
            errs.append(float(np.linalg.norm(zg - zo) / np.linalg.norm(zo)))
    return t_total, errs, iters


def time_solve(C, p, f, z, reps):
    import torch
    C.minres_solve(p, f, z, want_info=False)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        C.minres_solve(p, f, z, want_info=False)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) / reps * 1e3
    _, info = C.minres_solve(p, f, z)
    return ms, info


def other_configs(C, WL, dev):
    """The other workloads, each on its own (not part of the timed step):
    plain FP64 solves of the 2-D cases, the 3-D case with the FP64 and the
    FP32 preconditioner, and the adjoint workload (solve + adjoint of every
    shift)."""
    import torch
    out = {}
    for name, fp32s in (("c1", (False,)), ("c2", (False,)), ("c2_const", (False,)),
                        ("c3", (False, True))):
        s = WL.workload(name).systems[0]
        a = torch.from_numpy(s.a).to(dev)
        f = torch.from_numpy(s.f).to(dev)
        z = torch.empty_like(f)
        for fp32 in fp32s:
            p = C.Problem(a, s.lam.real, s.lam.imag, pinv_fp32=fp32)
            sched = p.tune(f, z)
            reps = 20 if s.a.size < 100000 else 3
            ms, info = time_solve(C, p, f, z, reps)
            bpp = bytes_model(s.a.ndim, fp32, sched["block_threads"] == 1024)
            out[f"{name}_{'fp32p' if fp32 else 'fp64'}"] = {
                "points": int(s.a.size), "ms_per_solve": ms, "iters": info["iters"],
                "relres_true": info["relres_true"], "status": info["status_name"],
                "alg_GBps": info["iters"] * s.a.size * bpp / ms / 1e6,
                "alg_frac_of_8TBps": info["iters"] * s.a.size * bpp / ms / 1e6 / PEAK_HBM_GBS,
                "bytes_per_point_iter": bpp,
                "schedule": {"tile_points": sched["tile_points"],
                             "lds_bytes": sched["lds_bytes"],
                             "block_threads": sched["block_threads"]}}
    if "c3_fp64" in out and "c3_fp32p" in out:
        out["c3_speedup_fp32p_vs_fp64"] = out["c3_fp64"]["ms_per_solve"] / out["c3_fp32p"]["ms_per_solve"]
    # adjoint workload: 16 shifts sharing one coefficient, loss sum ||z - zt||^2
    w = WL.workload("c5")
    at = torch.from_numpy(w.systems[0].a).to(dev)
    probs = [C.Problem(at, s.lam.real, s.lam.imag) for s in w.systems]
    fs = [torch.from_numpy(s.f).to(dev) for s in w.systems]
    zts = [torch.from_numpy(s.z_target).to(dev) for s in w.systems]

    def run():
        ga = torch.zeros_like(at)
        worst = 0.0
        for p, f, zt in zip(probs, fs, zts):
            z, info = C.minres_solve(p, f)
            g, ainfo = C.minres_adjoint(p, z, 2.0 * (z - zt), ga=ga)
            worst = max(worst, info["relres_true"], ainfo["relres_true"])
        return worst

    run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    worst = run()
    torch.cuda.synchronize()
    ms_seq = (time.perf_counter() - t0) * 1e3
    # the same work as one batched forward solve and one batched adjoint
    # (two persistent launches for the 16 systems)
    b = C.Batch(probs)
    b.tune(fs)
    zs = [torch.empty_like(f) for f in fs]

    def run_batched():
        ga = torch.zeros_like(at)
        _, infos = b.solve(fs, zs, want_info=False)
        gzs = [2.0 * (z - zt) for z, zt in zip(zs, zts)]
        b.adjoint(zs, gzs, ga=ga, want_info=False)
        return ga

    run_batched()
    torch.cuda.synchronize()
    reps = 5
    t0 = time.perf_counter()
    for _ in range(reps):
        run_batched()
    torch.cuda.synchronize()
    ms_batched = (time.perf_counter() - t0) / reps * 1e3
    _, finfos = b.solve(fs, zs)
    _, ainfos = b.adjoint(zs, [2.0 * (z - zt) for z, zt in zip(zs, zts)])
    b.close()
    out["c5_adjoint"] = {"systems": len(w.systems), "points_each": int(w.systems[0].a.size),
                         "ms_forward_plus_adjoint_all": ms_seq,
                         "ms_batched_forward_plus_adjoint": ms_batched,
                         "speedup_batched_vs_sequential": ms_seq / ms_batched,
                         "max_relres": worst,
                         "max_relres_batched": max(i["relres_true"] for i in finfos + ainfos)}
    out["paradiag"] = paradiag_config(C, WL, dev)
    out["many_rhs"] = many_rhs_config(C, WL, dev)
    out["paper_table2a"] = table2a_config(C, WL, dev)
    out["paper_table1a"] = table1a_config(C, WL, dev)
    return out


# The paper's Octave times per solve with a = 1 (the preconditioner is then
# |A| itself, two steps) at the shift -100 + 100i (Table 1(a)): context.
PAPER_TABLE1A_S = {63: 0.0073, 255: 0.054, 1023: 0.83}


def table1a_config(C, WL, dev, alpha=-100.0, beta=100.0):
    """Example 1 of the paper: a = 1, FP64, tol 1e-8, at the sizes of Table
    1(a) that the grids admit: one tuned single solve each."""
    import torch
    out = {"shift": [alpha, beta], "paper_octave_s_per_solve": PAPER_TABLE1A_S}
    g = WL.rng(9)
    for n in (63, 255, 1023):
        a = torch.ones((n, n), dtype=torch.float64, device=dev)
        f = torch.from_numpy(WL.complex_normal(g, (n, n))).to(dev)
        z = torch.empty_like(f)
        p = C.Problem(a, alpha, beta)
        p.tune(f, z)
        ms, info = time_solve(C, p, f, z, 10)
        out[str(n)] = {"ms_per_solve": ms, "iters": info["iters"],
                       "relres_true": info["relres_true"],
                       "paper_time_over_gpu_time": PAPER_TABLE1A_S[n] * 1e3 / ms}
        p.close()
    return out


# The paper's Octave times per solve for Example 2 at the shift -100 + 100i
# (Table 2(a); GNU Octave 8.2 on two 16-core Xeon Gold 6246R, FP64): context
# for the same workload here, not a target.
PAPER_TABLE2A_S = {63: 0.028, 255: 0.25, 1023: 4.47}


def table2a_config(C, WL, dev, alpha=-100.0, beta=100.0):
    """Example 2 of the paper (a = (20 + x^2)(20 + y^2) on the unit square,
    abar = sqrt(a_min a_max), FP64, tol 1e-8) at the sizes of Table 2(a)
    that the grids admit: one tuned single solve each."""
    import torch
    out = {"shift": [alpha, beta], "paper_octave_s_per_solve": PAPER_TABLE2A_S}
    g = WL.rng(8)
    for n in (63, 255, 1023):
        a = torch.from_numpy(WL.coef_paper_ex2(n)).to(dev)
        f = torch.from_numpy(WL.complex_normal(g, (n, n))).to(dev)
        z = torch.empty_like(f)
        p = C.Problem(a, alpha, beta, abar_rule="geomean")
        p.tune(f, z)
        ms, info = time_solve(C, p, f, z, 10)
        out[str(n)] = {"ms_per_solve": ms, "iters": info["iters"],
                       "relres_true": info["relres_true"],
                       "paper_time_over_gpu_time": PAPER_TABLE2A_S[n] * 1e3 / ms}
        p.close()
    return out


def many_rhs_config(C, WL, dev, n=255, count=64):
    """64 right-hand sides of one shifted system (c1's coefficient and shift
    on a 2-D n = 255 grid, FP64): one batch of the problem and 63 clones
    against 64 single solves of the problem."""
    import torch
    s = WL.workload("c1", n_override=n).systems[0]
    a = torch.from_numpy(s.a).to(dev)
    g = WL.rng(7)
    fs = [torch.from_numpy(WL.complex_normal(g, (n, n))).to(dev) for _ in range(count)]
    zs = [torch.empty_like(f) for f in fs]
    p = C.Problem(a, s.lam.real, s.lam.imag)
    p.tune(fs[0], zs[0])
    probs = [p] + [p.clone() for _ in range(count - 1)]
    b = C.Batch(probs)
    sched = b.tune(fs, zs)
    _, infos = b.solve(fs, zs)
    torch.cuda.synchronize()
    reps = 5
    t0 = time.perf_counter()
    for _ in range(reps):
        b.solve(fs, zs, want_info=False)
    torch.cuda.synchronize()
    ms_batch = (time.perf_counter() - t0) / reps * 1e3
    for f, z in zip(fs, zs):
        C.minres_solve(p, f, z, want_info=False)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for f, z in zip(fs, zs):
        C.minres_solve(p, f, z, want_info=False)
    torch.cuda.synchronize()
    ms_single = (time.perf_counter() - t0) * 1e3
    out = {"rhs": count, "points": n * n, "ms_batch": ms_batch, "ms_64_single_solves": ms_single,
           "solves_per_s_batch": count / ms_batch * 1e3,
           "solves_per_s_single": count / ms_single * 1e3,
           "speedup": ms_single / ms_batch,
           "iters_min": min(i["iters"] for i in infos), "iters_max": max(i["iters"] for i in infos),
           "all_converged": all(i["status"] == 0 for i in infos),
           "schedule": {"tile_points": sched["tile_points"], "lds_bytes": sched["lds_bytes"],
                        "block_threads": sched["block_threads"]}}
    b.close()
    for q in probs:
        q.close()
    return out


def paradiag_config(C, WL, dev, n=255, steps=64, tau=1.0 / 64, alpha_c=1e-2):
    """The alpha-circulant all-at-once layer: 64 implicit-Euler steps on a
    2-D n = 255 grid (a as c1, FP32 preconditioner, tol 1e-8): one solve =
    step transform, batched solve of the 64 shifted systems, inverse
    transform.  The step transform's rate is from HIP events around 20
    forward + inverse pairs (32 bytes per point and step each)."""
    import torch
    a = torch.from_numpy(WL.coef_c1(n)).to(dev)
    R = torch.from_numpy(WL.complex_normal(WL.rng(6), (steps, n, n))).to(dev)
    pd = C.ParaDiag(a, steps, tau, alpha_c, pinv_fp32=True)
    sched = pd.tune(R)
    U = torch.empty_like(R)
    _, infos = pd.solve(R, U)
    torch.cuda.synchronize()
    reps = 5
    t0 = time.perf_counter()
    for _ in range(reps):
        pd.solve(R, U, want_info=False)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) / reps * 1e3
    Y = torch.empty_like(R)
    pd.transform(R, Y)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(20):
        pd.transform(R, Y)
        pd.transform(Y, U, inverse=True)
    e1.record()
    torch.cuda.synchronize()
    tms = e0.elapsed_time(e1) / 40
    M = n * n
    its = [i["iters"] for i in infos]
    out = {"steps": steps, "points_per_step": M, "tau": tau, "alpha_c": alpha_c,
           "ms_per_all_at_once_solve": ms, "mode_solves_per_s": steps / ms * 1e3,
           "iters_min": min(its), "iters_max": max(its),
           "all_converged": all(i["status"] == 0 for i in infos),
           "max_relres_true": max(i["relres_true"] for i in infos),
           "step_transform_ms": tms,
           "step_transform_GBps": steps * M * 32.0 / tms / 1e6,
           "step_transform_frac_of_8TBps": steps * M * 32.0 / tms / 1e6 / 8000.0,
           "schedule": {"tile_points": sched["tile_points"], "lds_bytes": sched["lds_bytes"],
                        "block_threads": sched["block_threads"]}}
    pd.close()
    return out


def main():
    args = parse()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU; several GPUs would each "
                                   "solve their own share of the batch, which is not implemented"}))
        sys.exit(2)
    import torch
    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU available"}))
        sys.exit(1)
    if args.copy_calibration:
        copy_calibration()
        return
    if args.hbm_rates:
        hbm_rates()
        return
    import paper_2408_00488_amd as C
    from paper_2408_00488_amd import workloads as WL
    C.load_library()
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)

    w = WL.workload("c4", count_override=args.count)
    log(WL.describe(w))
    A = [torch.from_numpy(s.a).to(dev) for s in w.systems]
    F = [torch.from_numpy(s.f).to(dev) for s in w.systems]
    points = int(sum(s.a.size for s in w.systems))

    # ---------------- batched mixed precision (the measured step)
    probs32 = [C.Problem(a, s.lam.real, s.lam.imag, pinv_fp32=True) for a, s in zip(A, w.systems)]
    fixed = args.no_tune or args.tile_points > 0 or args.lds_bytes > 0 or args.block_threads > 0
    batch = C.Batch(probs32, tol=1e-8, maxit=1000, check_true=True, use_graph=True,
                    tile_points=args.tile_points, lds_bytes=args.lds_bytes,
                    block_threads=args.block_threads)
    Z = [torch.empty_like(f) for f in F]
    stream = torch.cuda.current_stream()
    # schedule (tile size, LDS budget, workgroup size) chosen by the batch autotuner, outside
    # the timed region
    tuning = batch.tune(F, Z) if not fixed else dict(batch.schedule, fixed=True)
    log("schedule:", tuning)
    zs, infos = batch.solve(F, Z)
    log("batch iters:", [i["iters"] for i in infos])
    for _ in range(args.warmup):
        batch.solve(F, Z, want_info=False)
    torch.cuda.synchronize()
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(args.steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        ev[k][0].record(stream)
        batch.solve(F, Z, want_info=False)
        ev[k][1].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    launch_ms = [a.elapsed_time(b) for a, b in ev]
    ms_per_step = wall * 1e3 / args.steps
    value = len(w.systems) * args.steps / wall
    zs, infos = batch.solve(F, Z)
    iters = [i["iters"] for i in infos]
    if args.batch_only:
        log(f"batched: {ms_per_step:.2f} ms per solve of {len(w.systems)} systems, "
            f"{value:.0f} solves/s, iterations {sum(iters)}")
        return
    relres = [i["relres_true"] for i in infos]
    statuses = [i["status"] for i in infos]
    Zcpu = [z.cpu().numpy() for z in Z]

    # algorithmic bytes of one launch (per-iteration model x iterations)
    alg_bytes = sum(it * s.a.size * bytes_model(2, True) for it, s in zip(iters, w.systems))
    alg_bytes_paired = sum(it * s.a.size * bytes_model_paired(2, True)
                           for it, s in zip(iters, w.systems))
    avg_launch_s = float(np.mean(launch_ms)) * 1e-3
    achieved = alg_bytes / avg_launch_s / 1e9

    # ---------------- plain FP64, one solve after another
    probs64 = [C.Problem(a, s.lam.real, s.lam.imag, pinv_fp32=False)
               for a, s in zip(A, w.systems)]
    Z64 = [torch.empty_like(f) for f in F]
    # every problem's single-solve schedule (tile size, LDS budget, workgroup
    # size, chunk size, and the engines where they were chosen automatically)
    # from the problem autotuner on its own right-hand side
    plain_sched = {}
    for p, f, z, s in zip(probs64, F, Z64, w.systems):
        t = p.tune(f, z)
        plain_sched.setdefault(str(s.n), []).append(
            (t["tile_points"], t["lds_bytes"], t["block_threads"], t["tile_elems"]))
    for p, f, z in zip(probs64, F, Z64):
        C.minres_solve(p, f, z, want_info=False)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.plain_reps):
        for p, f, z in zip(probs64, F, Z64):
            C.minres_solve(p, f, z, want_info=False)
    torch.cuda.synchronize()
    plain_wall = (time.perf_counter() - t0) / args.plain_reps
    plain_value = len(w.systems) / plain_wall
    iters64 = []
    for p, f, z in zip(probs64, F, Z64):
        _, inf = C.minres_solve(p, f, z)
        iters64.append(inf["iters"])

    # ---------------- batched plain FP64 (one tuned graph replay): splits the
    # speed-up over the plain solver into batching and precision
    batch64 = C.Batch(probs64, tol=1e-8, maxit=1000, check_true=True, use_graph=True)
    tuning64 = batch64.tune(F, Z64)
    _, infos_b64 = batch64.solve(F, Z64)
    for _ in range(max(1, args.warmup)):
        batch64.solve(F, Z64, want_info=False)
    torch.cuda.synchronize()
    reps64 = max(3, args.steps // 2)
    t0 = time.perf_counter()
    for _ in range(reps64):
        batch64.solve(F, Z64, want_info=False)
    torch.cuda.synchronize()
    b64_wall = (time.perf_counter() - t0) / reps64
    b64_value = len(w.systems) / b64_wall
    batch64.close()

    # ---------------- CPU oracle on a bounded sample
    cpu = None
    err_vs_oracle = None
    if not args.no_cpu_baseline:
        k = max(4, min(args.cpu_sample, len(w.systems)))
        idx = list(range(k))
        nthr = cpu_threads()
        model = cpu_model()
        t_cpu, errs, it_o = cpu_baseline(w, idx, Zcpu, nthr)
        t_cpu1, errs1, _ = cpu_baseline(w, idx, Zcpu, 1)
        sample = (f"first {k} systems of the batch (n = 63,127,255,511 in turn), FP64 "
                  f"NumPy/SciPy, on {model}")
        cpu = {"value": k / t_cpu, "unit": "solves/s", "cores": nthr, "kind": "oracle",
               "sample": f"{sample}, thread pools and SciPy's FFT given {nthr} threads, "
                         f"{t_cpu:.1f} s",
               "cpu_model": model, "affinity_cores": len(os.sched_getaffinity(0)),
               "single_thread": {"value": k / t_cpu1, "unit": "solves/s", "cores": 1,
                                 "sample": f"{sample}, every thread pool held to one thread, "
                                           f"{t_cpu1:.1f} s"}}
        err_vs_oracle = max(errs + errs1)
        log("oracle iters", it_o, "gpu", iters[:k], "max rel err vs oracle", err_vs_oracle)

    extra = None if args.no_extra else other_configs(C, WL, dev)
    out = {
        "metric": METRIC,
        "value": value,
        "unit": "solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64+f32",
        "data": "synthetic",
        "config": {"workload": "batched shifts: 64 2-D systems, n in {63,127,255,511} "
                               "(16 each), a=1+0.5 sin(2 pi x) sin(2 pi y), alpha-circulant "
                               "shifts tau=1/64 gamma=1e-2, FP32 preconditioner, tol 1e-8, "
                               "one hipGraph replay",
                   "systems": len(w.systems), "points": points,
                   "schedule": tuning},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                     "frac": achieved / PEAK_HBM_GBS, "traffic": measured_traffic(),
                     "kernel": "solve_kernel", "avg_launch_ms": avg_launch_s * 1e3,
                     "alg_bytes_per_launch": alg_bytes,
                     "bytes_per_point_iter": bytes_model(2, True),
                     "paired_update_model": {
                         "bytes_per_point_iter": bytes_model_paired(2, True),
                         "alg_bytes_per_launch": alg_bytes_paired,
                         "achieved": alg_bytes_paired / avg_launch_s / 1e9,
                         "frac": alg_bytes_paired / avg_launch_s / 1e9 / PEAK_HBM_GBS}},
        "cpu_baseline": cpu,
        "plain_fp64": {"value": plain_value, "unit": "solves/s",
                       "ms_per_64": plain_wall * 1e3,
                       "iters_min": min(iters64), "iters_max": max(iters64),
                       "schedules": plain_sched},
        "batched_fp64": {"value": b64_value, "unit": "solves/s", "ms_per_64": b64_wall * 1e3,
                         "iters_max": max(i["iters"] for i in infos_b64),
                         "all_converged": all(i["status"] == 0 for i in infos_b64),
                         "schedule": tuning64},
        "speedup_vs_plain_fp64": value / plain_value,
        "speedup_split": {"batching_fp64": b64_value / plain_value,
                          "precision_batched": value / b64_value},
        "iters": {"min": min(iters), "max": max(iters), "sum": int(sum(iters))},
        "max_relres_true": max(relres),
        "all_converged": all(s == 0 for s in statuses),
        "max_rel_err_vs_fp64_oracle": err_vs_oracle,
        "other_configs": extra,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
