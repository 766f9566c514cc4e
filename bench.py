#!/usr/bin/env python3
"""Benchmark: CGO solves per second at N = 1024 on one MI355X (the spectral D-bar method, Klein & McLaughlin).

A step is one pass of the whole hot path over one batch of synthetic input: solve A(S) = b (GMRES on the real 2N^2
form of the regularised integral equation) for all 16 spectral parameters k of the N = 1024 workload and produce S and
m = h(S) for each, with Q, S and m resident in device memory.  The headline path is the batched mixed-precision solver
(FP32 transforms and Krylov basis, FP64 residuals / moments / Hessenberg, refined to ||b - A S|| <= 1e-12 ||b|| in
FP64); it is reported only if every S agrees with the FP64 solver's S to <= 1e-10 (relative L-infinity), otherwise
the FP64 batched path is the headline.

Prints one JSON line.  Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload plain_n1024]
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, HERE)

METRIC = "solves/s at N=1024, err≤1e-10 vs FP64; FFT/matvec HBM GB/s; p50/p99 latency"
HBM_PEAK_GBS = 8000.0


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="plain_n1024")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-context", action="store_true", help="skip the FP64 batched / plain path timings")
    ap.add_argument("--headline", choices=["auto", "mixed", "fp64"], default="auto")
    ap.add_argument("--no-serving", action="store_true", help="skip the request-stream (p50/p99 latency) leg")
    ap.add_argument("--serving-requests", type=int, default=48)
    ap.add_argument("--no-configs", action="store_true",
                    help="skip the N = 512 batched and N = 4096 mixed-precision context legs")
    ap.add_argument("--no-autotune", action="store_true",
                    help="keep the default column-tile widths (skip the library's tuner before the timed region)")
    ap.add_argument("--no-rows-f", action="store_true",
                    help="skip the iterated-solver (Section 5.3) and DS II round-trip (Section 6) legs")
    ap.add_argument("--traffic-from", nargs=2, metavar=("FETCH_DIR", "WRITE_DIR"), default=None,
                    help="no GPU: turn the FETCH_SIZE / WRITE_SIZE counter CSVs of two `--probe` runs into "
                         "profiles/traffic_<workload>.json (bytes per launch per stage, scaled by the calibration "
                         "copy)")
    ap.add_argument("--probe", choices=["mixed", "fp64"], default=None,
                    help="counter-collection mode: two steps of the given path, then a 256 MiB device copy of known "
                         "size (the calibration kernel for FETCH_SIZE / WRITE_SIZE) and two grid transforms whose "
                         "column and row launches move known bytes with the line kernels' access patterns (a check "
                         "of that calibration); prints one JSON line")
    ap.add_argument("--batch", type=int, default=0,
                    help="entries per launch of the timed path (0: every k of the workload in one batch)")
    return ap.parse_args()


# sources that neither define, launch nor drive the solver's line kernels (serving, the DS II wrappers, the
# allocation-free entry point, the stage timer): a change there leaves stored counter measurements valid
_NOT_KERNEL_SOURCES = {"dbar_serve.hip", "dbar_scatter.hip", "dbar_noalloc.hip", "dbar_timer.hip"}


def kernel_source_hash() -> str:
    """sha256 over the HIP sources of the line kernels and the solver that launches them: a stored counter
    measurement is only valid for the kernels it was taken on."""
    import glob
    import hashlib
    h = hashlib.sha256()
    for f in sorted(glob.glob(os.path.join(HERE, "paper_1508_02363_amd", "csrc", "*"))):
        if os.path.basename(f) in _NOT_KERNEL_SOURCES:
            continue
        h.update(os.path.basename(f).encode())
        h.update(open(f, "rb").read())
    return h.hexdigest()


def stored_traffic(kernel: str, workload: str = "plain_n1024", entries: int = 0) -> dict:
    """Of `kernel`, from the PMC runs recorded in profiles/traffic_<workload>.json: `traffic`, the HBM bytes per launch
    scaled from the entries per launch of those runs (`traffic_entries`) to `entries`; None if none was recorded for it
    or the kernels changed since."""
    none = {"traffic": None, "traffic_entries": None}
    path = traffic_path(workload)
    if not os.path.exists(path):
        return none
    rec = json.load(open(path))
    ent = rec.get("kernels", {}).get(kernel)
    measured = rec.get("entries_per_launch")
    if rec.get("source_sha256") != kernel_source_hash() or ent is None or not measured:
        return none
    return {"traffic": ent["bytes_per_launch"] * (entries or measured) / measured, "traffic_entries": measured}


def stage_of_kernel(name: str):
    """Stage name (as reported by the library's launch timer) of a demangled kernel name from rocprofv3."""
    ops = {"OpRowsInvScaled": "RowsInvScaled", "OpColsInvMoments": "ColsInvMoments", "OpRowsInvRegular":
           "RowsInvRegular", "OpRowsFwdEpilogue": "RowsFwdEpilogue", "OpColsFwdPotential": "ColsFwdPotential",
           "OpRowsFwdMoments": "RowsFwdMoments", "OpColsFwdRegInv": "ColsFwdRegularInv",
           "OpRowsInvTailEpi": "RowsInvTailEpilogue"}
    prec = "f32" if "<float" in name else "f64"
    if "k_lines" in name:
        if "OpColsInvTail" in name:
            return f"lines.{'ColsInvTail' if 'true>' in name.split('OpColsInvTail')[1] else 'ColsInvTailFwd'}.{prec}"
        for k, v in ops.items():
            if k in name:
                return f"lines.{v}.{prec}"
    for k in ("dots", "update"):
        if f"k_{k}<" in name:
            return f"krylov.{k}.{prec}"
    return None


def traffic_path(workload: str) -> str:
    return os.path.join(HERE, "profiles", f"traffic_{workload}.json")


def traffic_from(fetch_dir: str, write_dir: str, workload: str, entries: int) -> dict:
    import csv
    import glob

    def load(d):
        out = {}
        for f in glob.glob(os.path.join(d, "*counter_collection.csv")):
            for r in csv.DictReader(open(f)):
                out.setdefault(r["Kernel_Name"], []).append((float(r["Counter_Value"]), int(r["Grid_Size"])))
        return out
    F, Wt = load(fetch_dir), load(write_dir)
    cal = "__amd_rocclr_copyBuffer"
    big = max(g for _, g in F[cal])
    kib = 256 * 1024  # the probe's calibration copy: 256 MiB read and written
    ff = kib / [v for v, g in F[cal] if g == big][-1]
    fw = kib / [v for v, g in Wt[cal] if g == big][-1]
    kernels, check = {}, {}
    for name, vals in F.items():
        if name not in Wt:
            continue
        f = sum(v for v, _ in vals) / len(vals) * ff * 1024
        wv = sum(v for v, _ in Wt[name]) / len(Wt[name]) * fw * 1024
        # the probe's transform: its column and row launches read one N x N array and write one
        for tag, op in (("cols", "OpColsPlain<"), ("rows", "OpRowsFwdEpilogue<")):
            if op in name:
                import re
                m = re.search(r"k_lines<(float|double), (\d+),", name)
                es, n = (8 if m.group(1) == "float" else 16), int(m.group(2))
                check[f"{tag}.{m.group(1)}.N{n}"] = {"expected_bytes": 2.0 * n * n * es, "measured_bytes": f + wv,
                                                     "ratio": (f + wv) / (2.0 * n * n * es)}
        st = stage_of_kernel(name)
        if st is None or "OpColsPlain<" in name or "OpRowsFwdEpilogue<" in name:
            continue
        kernels[st] = {"bytes_per_launch": f + wv, "fetch_bytes_per_launch": f, "write_bytes_per_launch": wv,
                       "launches": len(vals)}
    rec = {"source_sha256": kernel_source_hash(), "workload": workload, "entries_per_launch": entries,
           "fetch_scale": ff, "write_scale": fw, "calibration_check": check, "kernels": kernels}
    json.dump(rec, open(traffic_path(workload), "w"), indent=1)
    return rec


def rel_linf(a, b):
    return float(np.max(np.abs(a - b)) / max(float(np.max(np.abs(b))), 1e-300))


# ----------------------------------------------------------------------------------------------------------------
# CPU baseline: the oracle, as it is, in worker processes on the host cores (one single-threaded NumPy process per
# core: the parallelisation over k that the outlook of the paper proposes)
# ----------------------------------------------------------------------------------------------------------------
_OM = {}


def _oracle_worker(args):
    """One oracle solve of workload `name`, k index j (run in a spawned worker; single-threaded BLAS/FFT)."""
    name, j, want = args
    from threadpoolctl import threadpool_limits

    import dbar_workloads as W
    from oracle import dbar_oracle as O
    w = W.workload(name)
    with threadpool_limits(limits=1):
        t0 = time.perf_counter()
        key = (w.N, w.L, w.M)
        if key not in _OM:
            g = O.make_grid(w.N, w.L)
            _OM.clear()
            _OM[key] = (g, O.omega_table(g, w.M))
        g, om = _OM[key]
        ref = O.solve(g, w.Q, w.ks[j], tol=1e-13, M=w.M, om=om)
        dt = time.perf_counter() - t0
    return j, dt, ref.iters, ref.rel_residual, (ref.S if want else None), (ref.m if want else None)


def host_description() -> dict:
    import platform

    import scipy
    cpu = platform.processor() or "?"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                cpu = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    return {"cpu_model": cpu, "host_cores_visible": len(os.sched_getaffinity(0)), "numpy": np.__version__,
            "scipy": scipy.__version__, "fft_backend": "numpy.fft (pocketfft, C, single-threaded)",
            "python": platform.python_version()}


def oracle_pool(workers: int):
    import concurrent.futures as cf
    import multiprocessing as mp
    for v in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS"):
        os.environ[v] = "1"
    return cf.ProcessPoolExecutor(max_workers=workers, mp_context=mp.get_context("spawn"))


def cpu_baseline_leg(w, S, m, subset_n512=None) -> tuple[dict, dict]:
    """The oracle timed on the host: (i) one solve in one process (k index 0), (ii) all 16 k of the benchmark workload
    over one single-threaded worker per core (at most 16, a one-GPU host's CPU share), as solves/s; the same for the
    small-grid workload (1 k) and a seeded 64-k subset of the N = 512 batched workload.  Returns (cpu_baseline,
    accuracy): the GPU results of every benchmark k against the oracle's."""
    workers = max(1, min(16, len(os.sched_getaffinity(0))))
    nk = len(w.ks)
    acc = {}
    with oracle_pool(workers) as ex:
        # (i) one process, one solve (the pool's first worker: warm interpreter, cold caches)
        t0 = time.perf_counter()
        j0, dt0, it0, res0, S0, m0 = ex.submit(_oracle_worker, (w.name, 0, True)).result()
        single = time.perf_counter() - t0
        # (ii) every k, one worker per core
        t0 = time.perf_counter()
        out = list(ex.map(_oracle_worker, [(w.name, j, True) for j in range(nk)]))
        wall = time.perf_counter() - t0
        errS = max(rel_linf(S[j].cpu().numpy(), Sj) for j, _, _, _, Sj, _ in out)
        errm = max(rel_linf(m[j].cpu().numpy(), mj) for j, _, _, _, _, mj in out)
        acc = {"err_S_vs_oracle_max": errS, "err_m_vs_oracle_max": errm, "oracle_k": nk,
               "oracle_rel_residual_max": max(o[3] for o in out), "oracle_iters": [o[2] for o in out]}
        others = {}
        # the small-grid workload: N = 128, one k
        t0 = time.perf_counter()
        r = ex.submit(_oracle_worker, ("plain_n128", 0, False)).result()
        others["plain_n128"] = {"solves_per_s_one_core": 1.0 / r[1], "seconds": r[1]}
        if subset_n512 is not None:
            t0 = time.perf_counter()
            res = list(ex.map(_oracle_worker, [("batched_n512", int(j), False) for j in subset_n512]))
            dt = time.perf_counter() - t0
            others["batched_n512_subset"] = {"n_k": len(subset_n512), "solves_per_s": len(subset_n512) / dt,
                                             "seconds": dt, "mean_iters": float(np.mean([x[2] for x in res]))}
    base = {
        "value": nk / wall, "unit": "solves/s", "cores": workers, "kind": "oracle",
        "sample": f"all {nk} k of the benchmark workload (N={w.N}), one oracle solve each (NumPy FP64, GMRES to 1e-13, "
                  f"W_n tables included) over {workers} single-threaded worker processes, {wall:.1f} s wall",
        "single_core_solves_per_s": 1.0 / dt0, "single_core_seconds_per_solve": dt0,
        "single_core_sample": f"k index 0 in one worker process ({dt0:.1f} s; {single:.1f} s with process start)",
        "other_configs": others, "host": host_description(),
    }
    return base, acc


def serving_leg(D, W, n_req: int) -> dict:
    """Poisson request stream over grids N in {256, 512, 1024, 2048} (k uniform in |k| <= 6, Gaussian-sum or sech^2
    potentials with |A| <= 2, mixed precision to 1e-10).  The saturated capacity is measured first with a burst of
    requests; the stream then arrives at 0.8 x that rate.  Latency = submit -> result on the host."""
    import threading

    burst = W.serving_stream(32, rate=1.0, seed=50)
    stream = W.serving_stream(n_req, rate=1.0, seed=5)
    with D.Session(max_slots=64) as s:
        # the first burst warms the session (grid-class workspaces, pinned staging blocks); the second one measures
        for rep in range(2):
            t0 = time.perf_counter()
            tk = [s.submit(r.Q, r.k, r.L, tol=r.tol) for r in burst]
            for t in tk:
                s.wait(t)
            capacity = len(burst) / (time.perf_counter() - t0)
        rate = 0.8 * capacity
        # rescale the unit-rate arrival times to the target rate
        arrivals = [r.t_arrival / rate for r in stream]
        lat, infos, done_at = {}, {}, {}
        lock = threading.Lock()
        pending = []
        stop = [False]

        def poller():
            while True:
                with lock:
                    todo = list(pending)
                for t in todo:
                    res = s.poll(t)
                    if res is not None:
                        with lock:
                            pending.remove(t)
                        lat[t], infos[t], done_at[t] = res[3], res[2], time.perf_counter()
                if stop[0] and not todo:
                    return
                time.sleep(0.0005)

        th = threading.Thread(target=poller)
        th.start()
        t_start = time.perf_counter()
        for r, ta in zip(stream, arrivals):
            dt = t_start + ta - time.perf_counter()
            if dt > 0:
                time.sleep(dt)
            t = s.submit(r.Q, r.k, r.L, tol=r.tol)
            with lock:
                pending.append(t)
        stop[0] = True
        th.join()
        t_end = max(done_at.values())
        stats = s.stats()
    L_ms = np.array([v * 1e3 for v in lat.values()])
    by_n = {}
    for r, t in zip(stream, sorted(lat)):
        by_n.setdefault(r.N, []).append(lat[t] * 1e3)
    return {
        "requests": n_req, "grid_sizes": [256, 512, 1024, 2048], "precision": "mixed", "tol": 1e-10,
        "saturated_capacity_solves_per_s": capacity, "arrival_rate_per_s": rate,
        "solves_per_s": n_req / (t_end - t_start),
        "p50_latency_ms": float(np.percentile(L_ms, 50)), "p99_latency_ms": float(np.percentile(L_ms, 99)),
        "p50_latency_ms_by_N": {int(k): float(np.percentile(v, 50)) for k, v in sorted(by_n.items())},
        "max_rel_residual": max(i.rel_residual for i in infos.values()),
        "max_err_estimate": max(i.err_estimate for i in infos.values()),
        "all_converged": all(i.status == 0 for i in infos.values()),
        "session_stats": stats,
    }


def iterated_leg(D, Qd, L: float, M: int, tol: float) -> dict:
    """The Section 5.3 iterated solver on the benchmark's potential and grid: 16 k with 2kL integer (a 4 x 4 grid over
    {-2, -0.6, 0.6, 2}^2), batched; the mixed path's S is checked against the FP64 path's."""
    import torch
    ks = np.array([complex(a, b) for b in (-2.0, -0.6, 0.6, 2.0) for a in (-2.0, -0.6, 0.6, 2.0)])

    def run(prec):
        return D.solve_device(Qd, ks, L, tol=tol, M=M, batch=len(ks), method=D.DBAR_METHOD_ITERATED, precision=prec)

    out = {"n_k": len(ks), "k_set": "{-2, -0.6, 0.6, 2}^2"}
    res = {}
    for name, prec in (("mixed", D.DBAR_MIXED), ("fp64", D.DBAR_FP64)):
        run(prec)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        res[name] = run(prec)
        torch.cuda.synchronize()
        out[f"{name}_solves_per_s"] = len(ks) / (time.perf_counter() - t0)
        out[f"{name}_iters"] = [i.iters for i in res[name][2]]
    S64 = res["fp64"][0].cpu().numpy()
    out["mixed_err_S_vs_fp64"] = max(rel_linf(res["mixed"][0][j].cpu().numpy(), S64[j]) for j in range(len(ks)))
    return out


def stage_summary(stages: list) -> dict:
    """Roofline of the dominant stage of one timed pass (the stage with the largest total time: its algorithmic bytes
    per launch over its average launch duration, HIP events on the stream the kernels run on), the per-stage GB/s,
    and the stages whose algorithmic rate would exceed the HBM peak (a byte-model error, reported, never hidden).
    `bound` is what limits that stage: vector issue for the column stage of the x-space operator in FP32 (0.59 to 0.74 of
    its time by the SQ counters, where its bytes take 0.2 to 0.4 of it), else memory; achieved and peak are HBM rates
    either way."""
    dom = max(stages, key=lambda s: s["total_ms"])
    achieved = dom["bytes"] / (dom["total_ms"] * 1e-3) / 1e9
    fft = [s for s in stages if s["name"].startswith("lines.")]
    fft_ms = sum(s["total_ms"] for s in fft)
    per = {s["name"]: {"ms": round(s["total_ms"], 4), "launches": s["launches"],
                       "GB/s": round(s["bytes"] / max(s["total_ms"], 1e-9) / 1e6, 1)} for s in stages}
    return {
        "roofline": {"bound": "valu" if dom["name"] == "lines.ColsFwdRegularInv.f32" else "hbm",
                     "kernel": dom["name"], "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "launches": dom["launches"],
                     "avg_launch_us": dom["total_ms"] * 1e3 / dom["launches"],
                     "bytes_per_launch": dom["bytes"] / dom["launches"]},
        "stages": per,
        "fft_matvec_GBs": sum(s["bytes"] for s in fft) / (fft_ms * 1e-3) / 1e9 if fft_ms > 0 else 0.0,
        "stages_above_peak": [k for k, v in per.items() if v["GB/s"] > HBM_PEAK_GBS],
        "total_stage_ms": sum(s["total_ms"] for s in stages),
    }


def configs_leg(D, W) -> dict:
    """The other full-size workloads, one timed pass each after a warm-up: the batched N = 512 workload (all 1024 k
    of the 32 x 32 grid, FP64, column tiles and batch tuned first) and the N = 4096 mixed-precision workload (64 k),
    whose S is checked against the FP64 path for four sampled k."""
    import torch
    out = {}
    w = W.workload("batched_n512")
    tune = D.autotune(w.N, w.L, precision=D.DBAR_FP64, batch=64, M=w.M)
    Qd = torch.from_numpy(w.Q).to("cuda:0")
    D.solve_device(Qd, w.ks[:64], w.L, tol=w.tol, M=w.M, precision=D.DBAR_FP64, want_m=False)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    _, _, info = D.solve_device(Qd, w.ks, w.L, tol=w.tol, M=w.M, precision=D.DBAR_FP64)
    torch.cuda.synchronize()
    out["batched_n512"] = {"n_k": len(w.ks), "precision": "fp64", "solves_per_s": len(w.ks) / (time.perf_counter() - t0),
                           "batch": tune["batch"], "fp64_tile_columns": tune["fp64"]["chosen_columns"],
                           "all_converged": all(i.status == 0 for i in info),
                           "mean_iters": float(np.mean([i.iters for i in info]))}
    D.set_tile(w.N, D.DBAR_FP64, 0)
    del Qd
    w = W.workload("mixed_n4096")
    # column tiles for this grid (FP32 and FP64 operators), outside the timed region like every warm-up
    tune4096 = D.autotune(w.N, w.L, precision=D.DBAR_MIXED, batch=16, M=w.M)
    Qd = torch.from_numpy(w.Q).to("cuda:0")
    # warm-up on the same k set: the same batch size, so the timed call replays the captured Krylov graphs
    D.solve_device(Qd, w.ks, w.L, tol=w.tol, M=w.M, precision=D.DBAR_MIXED, want_m=False)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    S, _, info = D.solve_device(Qd, w.ks, w.L, tol=w.tol, M=w.M, precision=D.DBAR_MIXED, want_m=False)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    sample = [0, 21, 42, 63]
    S64, _, _ = D.solve_device(Qd, w.ks[sample], w.L, tol=w.tol, M=w.M, precision=D.DBAR_FP64, want_m=False)
    err = max(rel_linf(S[j].cpu().numpy(), S64[i].cpu().numpy()) for i, j in enumerate(sample))
    del S, S64
    # per-stage timing of one more pass: here one FP32 vector is 128 MiB and a launch over the batch streams
    # gigabytes, far beyond the 256 MB Infinity Cache, so the rates are HBM rates
    D.timer_enable(True)
    D.solve_device(Qd, w.ks, w.L, tol=w.tol, M=w.M, precision=D.DBAR_MIXED, want_m=False)
    torch.cuda.synchronize()
    D.timer_enable(False)
    summ = stage_summary(D.timer_stages())
    out["mixed_n4096"] = {"n_k": len(w.ks), "precision": "mixed", "solves_per_s": len(w.ks) / dt,
                          "all_converged": all(i.status == 0 for i in info),
                          "max_rel_residual": max(i.rel_residual for i in info),
                          "max_err_estimate": max(i.err_estimate for i in info),
                          "max_cond_estimate": max(i.cond_estimate for i in info),
                          "err_S_vs_fp64_sampled": err, "sampled_k": sample,
                          "roofline": dict(summ["roofline"], **stored_traffic(summ["roofline"]["kernel"], "mixed_n4096",
                                                                              tune4096["batch"])),
                          "stages": summ["stages"],
                          "fft_matvec_GBs": summ["fft_matvec_GBs"], "stages_above_peak": summ["stages_above_peak"],
                          "tuning": tune4096}
    D.set_tile(w.N, D.DBAR_FP64, 0)
    D.set_tile(w.N, D.DBAR_FP32, 0)
    return out


def ds2_leg(D, W, N: int = 128, L: float = 3.2) -> dict:
    """DS II round trip of Section 6.2 (reconstruction table row N = 2^7, L = 3.2, M = 11; the paper's error is
    2.40e-13): r(k) for q0 = e^{-x^2-y^2} at every k of the xi grid, then q from r at every z of the x grid, FP64."""
    q0 = W.potential_gaussian(N, L, 1.0)
    ks = W.k_xi_grid(N, L)
    t0 = time.perf_counter()
    r, info_r = D.reflection(q0, ks.ravel(), L, tol=1e-12)
    t_r = time.perf_counter() - t0
    t0 = time.perf_counter()
    q, info_q = D.reconstruct(r.reshape(N, N), L, tol=1e-12, want_info=True)
    t_q = time.perf_counter() - t0
    return {
        "N": N, "L": L, "M": 11, "precision": "fp64", "solves": 2 * N * N,
        "reflection_solves_per_s": N * N / t_r, "reconstruction_solves_per_s": N * N / t_q,
        "round_trip_s": t_r + t_q, "err_q_vs_q0": float(np.max(np.abs(q - q0))), "paper_err": 2.40e-13,
        "mean_iters": float(np.mean([i.iters for i in info_r] + [i.iters for i in info_q])),
        "all_converged": all(i.status == 0 for i in info_r) and all(i.status == 0 for i in info_q),
    }


def entries_per_launch(batch: int) -> tuple[int, int]:
    """(lanes, entries per launch of each): the library splits a batch of 16 or more into two concurrent lanes of half the
    entries each."""
    lanes = 2 if batch >= 16 else 1
    return lanes, -(-batch // lanes)


def main():
    args = parse()
    if args.traffic_from:
        import dbar_workloads as W
        rec = traffic_from(*args.traffic_from, args.workload,
                           entries_per_launch(args.batch if args.batch > 0 else len(W.workload(args.workload).ks))[1])
        print(json.dumps({"traffic_stages": len(rec["kernels"]), "fetch_scale": rec["fetch_scale"],
                          "write_scale": rec["write_scale"], "calibration_check": rec["calibration_check"]}))
        return
    if args.gpus != 1:
        print(json.dumps({"error": "one GPU only: --gpus must be 1 (sharding the k values over several GPUs is "
                          "not built)"}))
        sys.exit(2)
    import torch

    import dbar_workloads as W
    from paper_1508_02363_amd import dbar as D

    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU visible"}))
        sys.exit(1)
    dev = torch.device("cuda:0")
    w = W.workload(args.workload)
    N, L, nk = w.N, w.L, len(w.ks)
    Qd = torch.from_numpy(w.Q).to(dev)
    torch.cuda.synchronize()

    batch = args.batch if args.batch > 0 else nk
    lanes, lane_batch = entries_per_launch(batch)

    def step(**kw):
        kw.setdefault("batch", batch)
        return D.solve_device(Qd, w.ks, L, tol=w.tol, M=w.M, **kw)

    # the library's tuner picks the column-tile widths for this grid at the entries per launch of one lane (outside
    # the timed region, like the warm-up)
    tuning = None if args.no_autotune or args.probe else D.autotune(N, L, precision=D.DBAR_MIXED, batch=lane_batch,
                                                                    M=w.M)

    paths = {
        "mixed": dict(precision=D.DBAR_MIXED),
        "fp64": dict(precision=D.DBAR_FP64),
        "plain": dict(precision=D.DBAR_FP64, mode=D.DBAR_MODE_PLAIN),
        "mixed_xi": dict(precision=D.DBAR_MIXED, space=D.DBAR_SPACE_XI),
    }

    if args.probe:
        # one lane at the lanes' entries per launch: the launches of the timed step, timed one at a time
        kw = dict(paths[args.probe], batch=lane_batch, lanes=1)
        step(**kw)
        torch.cuda.synchronize()
        step(**kw)
        # a third step under the library's launch timer: the algorithmic bytes per launch of each stage, for the
        # counter runs' measured bytes to be set against (the same launches, so the per-launch averages agree)
        D.timer_enable(True)
        step(**kw)
        torch.cuda.synchronize()
        algo = {s["name"]: s["bytes"] / s["launches"] for s in D.timer_stages() if s["launches"]}
        D.timer_enable(False)
        src = torch.ones(16 * 2 ** 20, dtype=torch.complex128, device=dev)  # 256 MiB
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
        # the transform check: a column launch (FFT of every column) and a row launch (FFT of every row), each
        # reading one N x N array and writing one
        f = np.random.default_rng(1).standard_normal((N, N)) + 0j
        D.transform(f, L, precision=D.DBAR_FP64 if args.probe == "fp64" else D.DBAR_FP32)
        torch.cuda.synchronize()
        print(json.dumps({"probe": args.probe, "workload": w.name, "copy_bytes_read": 256 * 2 ** 20,
                          "copy_bytes_written": 256 * 2 ** 20, "algorithmic_bytes_per_launch": algo}))
        return

    def timed(kw, steps, warmup):
        out = None
        for _ in range(warmup):
            out = step(**kw)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            out = step(**kw)
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / steps, out

    # reference FP64 batched results (also the accuracy yardstick of the mixed path)
    t_fp64, (S64, m64, info64) = timed(paths["fp64"], 1, 1)
    S64h, m64h = S64.cpu().numpy(), m64.cpu().numpy()
    t_mix, (Smx, mmx, infomx) = timed(paths["mixed"], 1, 1)
    err_mixed = max(rel_linf(Smx[j].cpu().numpy(), S64h[j]) for j in range(nk))
    err_mixed_m = max(rel_linf(mmx[j].cpu().numpy(), m64h[j]) for j in range(nk))
    headline = args.headline
    if headline == "auto":
        headline = "mixed" if (err_mixed <= 1e-10 and all(i.status == 0 for i in infomx)) else "fp64"
    kw = paths[headline]

    # the timed region
    sec, (S, m, info) = timed(kw, args.steps, args.warmup)
    value = nk / sec

    # per-stage launch timing with HIP events (one more pass of the same step).  The timer runs one lane at a time
    # (its events time each launch on its own), so this pass solves the lanes' parts one after the other: the same
    # launches, with the entries per launch of one lane
    D.timer_enable(True)
    step(**dict(kw, batch=lane_batch, lanes=1))
    torch.cuda.synchronize()
    D.timer_enable(False)
    summ = stage_summary(D.timer_stages())
    roof = summ["roofline"]
    roof.update(stored_traffic(roof["kernel"], w.name, lane_batch))

    context = {}
    if not args.no_context:
        context["fp64_batched_solves_per_s"] = nk / t_fp64
        t_plain, (Sp, mp, infop) = timed(paths["plain"], 1, 0)
        context["plain_fp64_solves_per_s"] = nk / t_plain
        context["speedup_vs_plain_fp64"] = value / context["plain_fp64_solves_per_s"]
        context["plain_err_vs_fp64_batched"] = max(rel_linf(Sp[j].cpu().numpy(), S64h[j]) for j in range(nk))
        # the same mixed solver with GMRES on S itself (the paper's form) instead of s = F^{-1} S
        t_xi, (Sq, _, _) = timed(paths["mixed_xi"], 2, 1)
        context["mixed_xi_space_solves_per_s"] = nk / t_xi
        context["mixed_xi_space_err_vs_fp64"] = max(rel_linf(Sq[j].cpu().numpy(), S64h[j]) for j in range(nk))
        # one lane at the full batch, Krylov iterations replayed from captured HIP graphs
        t_1l, (S1l, _, _) = timed(dict(kw, lanes=1, use_graph=1), 2, 1)
        context["one_lane_graph_solves_per_s"] = nk / t_1l
        context["one_lane_graph_err_vs_headline"] = max(rel_linf(S1l[j].cpu().numpy(), S[j].cpu().numpy())
                                                        for j in range(nk))
        # the same solvers with full orthogonalisation (classical GMRES, no Gram-Schmidt window)
        for name in ("mixed", "fp64"):
            t_full, (Sf, _, infof) = timed(dict(paths[name], orth_window=0), 2, 1)
            context[f"{name}_full_gmres_solves_per_s"] = nk / t_full
            context[f"{name}_full_gmres_iters"] = [i.iters for i in infof]
            context[f"{name}_full_gmres_err_vs_fp64"] = max(rel_linf(Sf[j].cpu().numpy(), S64h[j]) for j in range(nk))

    result = {
        "metric": METRIC,
        "value": value,
        "unit": "solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": sec * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32+f64" if headline == "mixed" else "f64",
        "data": "synthetic",
        "config": {
            "workload": f"{w.name}: N={N}, L={L}, Q=(0.8+0.6i)exp(-(x^2+y^2)), {nk} k on a 4x4 grid in [-2,2]^2, "
                        f"M={w.M}, tol {w.tol:g}, batched {headline}",
            "N": N, "L": L, "n_k": nk, "M": w.M, "tol": w.tol, "path": headline, "batch": batch, "lanes": lanes,
            "entries_per_launch": lane_batch,
        },
        "accuracy": {
            "mixed_err_S_vs_fp64": err_mixed, "mixed_err_m_vs_fp64": err_mixed_m,
            "max_rel_residual": max(i.rel_residual for i in info),
            "iters": [i.iters for i in info], "outer": [i.outer for i in info],
            "cond_estimate": [round(i.cond_estimate, 3) for i in info],
            "max_err_estimate": max(i.err_estimate for i in info),
        },
        "roofline": roof,
        "stages": summ["stages"],
        "stages_above_peak": summ["stages_above_peak"],
        "fft_matvec_GBs": summ["fft_matvec_GBs"],
        # the timer pass runs the lanes' parts one after the other: its stages' total above ms_per_step is the time
        # the overlapped lanes save
        "timer_pass_stage_ms": summ["total_stage_ms"],
        "context": context,
        "tuning": tuning,
    }

    if not args.no_serving:
        result["serving"] = serving_leg(D, W, args.serving_requests)
    if not args.no_rows_f:
        result["iterated"] = iterated_leg(D, Qd, L, w.M, w.tol)
        result["ds2"] = ds2_leg(D, W)
    if not args.no_configs:
        result["other_configs"] = configs_leg(D, W)

    if not args.no_cpu_baseline:
        subset = np.sort(np.random.default_rng(3).choice(1024, 64, replace=False))
        base, acc = cpu_baseline_leg(w, S, m, subset)
        result["cpu_baseline"] = base
        result["accuracy"].update(acc)
    print(json.dumps(result))


if __name__ == "__main__":
    main()
