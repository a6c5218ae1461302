#!/usr/bin/env python3
"""Throughput of exact hypercube-grid DBSCAN on one MI355X.

One step = one full clustering call (bounding box, cube keys and radix sort,
cube tables, neighbour-group lists, core points, representatives, merging,
border points, canonical labels) over one synthetic workload whose points are
already resident in HBM.  Default workload: 2-D, 1M points.  Prints one JSON
line.  The CPU oracle (the paper's grid method run on the host) is timed on a
bounded sample beside it as a reported baseline.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import statistics
import sys
import time
from pathlib import Path

ROOT = Path(__file__).resolve().parent
sys.path.insert(0, str(ROOT))

METRIC = "points clustered/s (2-D 1M, 8-D 500k) vs HBM roofline; served p50/p99 latency"
HBM_PEAK_GBS = 8000.0
# int32 VALU lane-ops: 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz = 39.3e12 /s
ALU_PEAK_TOPS = 256 * 64 * 2.4e9 / 1e12
# int8 matrix ops (a multiply-add counts as two): 256 CUs x 8192 x 2.4 GHz
MFMA_PEAK_TOPS = 256 * 8192 * 2.4e9 / 1e12
WORKLOADS = {"2d": 2, "8d": 3, "small": 1, "batch": 4, "served": 5, "54d": 54}
# 54d: the shape of the paper's largest data set (PAMAP2, Table 1), 54 axes
HIGH_N = 3_850_505
HBM_PHASES = ("bbox", "sort", "cells", "labels")
ALU_PHASES = {"core": "tests_core", "intra": "tests_intra", "merge": "tests_merge",
              "border": "tests_border"}
SMALL_CALL = 16384      # most points that the library's path for small calls takes
PHASE_KERNELS = {
    "bbox": ["k_bbox", "k_bbox_check"], "sort": ["k_keys_hist", "k_onesweep"], "cells": ["k_cells", "k_table_clear", "k_table"],
    "lists": ["k_group_prep", "k_group_box", "k_nbr_lists", "k_nbr_bscan", "k_nbr_back"],
    "core": ["k_core", "k_core_chunks", "k_core_flat", "k_core_lanes", "k_core_deferred", "k_core_list_lanes",
             "k_core_list_deferred", "k_core_group_lanes", "k_core_group_rest", "k_core_cubes"],
    "reps": ["k_reps_init", "k_reps", "k_reps_small", "k_reps_big"],
    "intra": ["k_link_recorded", "k_link_listed", "k_core_box", "k_merge_tiles", "k_merge_big", "k_merge_unify"],
    "merge": ["k_merge_near", "k_merge_open", "k_merge_rep", "k_merge_cubes", "k_merge_exact", "k_merge_inter",
              "k_merge_pairs", "k_flatten", "k_compress"],
    "border": ["k_border", "k_border_chunks", "k_border_rec", "k_border_list", "k_border_walk_list"],
    "labels": ["k_label_marks", "k_label_scan", "k_label_cubes", "k_label_write", "k_label_bin", "k_label_fill"],
}
# more than 8 axes: the kernels of each phase
PHASE_KERNELS_HIGH = {
    "bbox": ["k_hd_bbox"], "sort": ["k_hd_keys_hist", "k_onesweep", "k_hd_gather"],
    "cells": ["k_cells", "k_table"], "lists": ["k_hd_group_init", "k_hd_group_box", "k_hd_lists", "k_nbr_bscan", "k_nbr_back"],
    "core": ["k_hd_planes", "k_hd_runs", "k_hd_core_tiles", "k_hd_left", "k_hd_core", "k_hd_core_rest", "k_hd_gcore"],
    "merge": ["k_link_recorded", "k_hd_unify", "k_hd_need", "k_hd_merge", "k_compress"],
    "border": ["k_hd_border_rec", "k_hd_border"],
    "labels": PHASE_KERNELS["labels"],
}


def algorithmic_bytes(phase: str, n: int, d: int, key_bytes: int, passes: int, cells: int) -> float:
    """Bytes a phase must move per call whatever the kernels do (per point and
    per cube figures times the counts)."""
    if phase == "bbox":
        return 4.0 * d * n                                   # read the points
    if phase == "sort":
        kv = key_bytes + 4
        # keys: read points, write (key, index); each pass reads and writes
        # (key, index); the last pass gathers the points into cube order
        return n * (4.0 * d + kv + 2.0 * passes * kv + 8.0 * d)
    if phase == "cells":
        return n * (key_bytes + 4.0) + cells * 16.0           # read keys, write cube ids + tables
    if phase == "labels":
        # core flag, cube or owner, input index read; label written; + per cube
        return n * (1.0 + 4.0 + 4.0 + 4.0) + cells * 16.0
    return 0.0


def kernel_source_digest() -> str:
    h = hashlib.sha256()
    for f in sorted((ROOT / "paper_1912_00323_amd" / "csrc").glob("*.*")):
        if f.suffix in (".hip", ".h", ".cpp"):
            h.update(f.read_bytes())
    return h.hexdigest()[:16]


def measured_traffic(phase: str, workload: str):
    """HBM bytes per call of a phase from the committed rocprofv3 PMC summary,
    if it was taken on the current kernel sources; else None."""
    f = ROOT / "profiles" / "pmc_traffic.json"
    if not f.exists():
        return None
    try:
        data = json.loads(f.read_text())
    except ValueError:
        return None
    e = data.get("entries", {}).get(f"{workload}:{phase}")
    if not e or e.get("source_digest") != kernel_source_digest():
        return None
    return e.get("bytes_per_call")


def cpu_model() -> str:
    """The host CPU's model string (as lscpu prints it), from /proc/cpuinfo."""
    try:
        for line in Path("/proc/cpuinfo").read_text().splitlines():
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def host_threads() -> int:
    return len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()


def cpu_baseline(w, budget_s: float = 12.0) -> dict:
    """The oracle on the host cores with OpenMP over all of them, and on one
    thread; each leg takes about budget_s seconds."""
    threads = host_threads()
    multi = cpu_oracle_rate(w, threads, budget_s)
    single = cpu_oracle_rate(w, 1, budget_s)
    return {"value": multi["value"], "unit": "points/s", "cores": threads, "kind": "oracle",
            "sample": multi["sample"],
            "single_thread": {"value": single["value"], "unit": "points/s", "cores": 1,
                              "sample": single["sample"]},
            "cpu_model": cpu_model(), "host_threads": threads}


def cpu_oracle_rate(w, threads: int, budget_s: float) -> dict:
    """The oracle on `threads` host threads (its grid method up to 8 axes, the
    definition above that), on the whole workload when it finishes within
    the budget, else on the first m points of the input (which is in random
    order), m doubling from 20k while runs stay short."""
    import oracle
    if w.d > 8:
        def run(p):
            oracle.dbscan(p, w.eps, w.min_pts, threads=threads)
        method = ("DBSCAN from its definition in plain C (oracle/dbscan_def.c: points visited in order "
                  "of axis 0, OpenMP over points; the grid method's stencil is out of reach past 8 axes)")
    else:
        def run(p):
            oracle.hca_grid(p, w.eps, w.min_pts, threads=threads)
        method = ("the paper's hypercube method in plain C (oracle/hca_grid.c: OpenMP over points for "
                  "core marking and borders, sequential depth-first merge)")
    t_all = time.perf_counter()
    m = min(w.n, 20_000)
    while True:
        t0 = time.perf_counter()
        run(w.points[:m])
        t = time.perf_counter() - t0
        # the cost grows at least linearly in m: stop before overrunning
        if m == w.n or t * 4 > budget_s - (time.perf_counter() - t_all):
            break
        m = min(w.n, 2 * m)
    times = [t]
    while len(times) < 3 and time.perf_counter() - t_all + t < budget_s:
        t0 = time.perf_counter()
        run(w.points[:m])
        times.append(time.perf_counter() - t0)
    t = statistics.median(times)
    what = (f"the whole {w.name} workload (n={w.n})" if m == w.n else
            f"the first {m} of the {w.n} points of {w.name} (same eps and minPts; lower density "
            f"than the whole set, so the per-point rate flatters the CPU)")
    return {"value": m / t, "unit": "points/s", "cores": threads, "kind": "oracle",
            "sample": f"{what}; {method}, {threads} thread(s), median of {len(times)} run(s)"}


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", choices=sorted(WORKLOADS), default="2d")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--requests", type=int, default=10_000, help="served workload: distinct requests")
    ap.add_argument("--slo-ms", type=float, default=250.0, help="served workload: p99 latency objective")
    ap.add_argument("--loads", default="0.7,1.0,1.3",
                    help="served workload: arrival rates as multiples of the plain path's sustained rate")
    ap.add_argument("--saturated", action="store_true", help="served workload: also every request at once")
    ap.add_argument("--batch-ms", type=float, default=4.0,
                    help="served workload: estimated device time a batch may gather")
    ap.add_argument("--no-second", action="store_true",
                    help="2d workload: skip the 8-D 500k workload that is measured beside it")
    ap.add_argument("--merge", choices=("exact", "representatives"), default="exact",
                    help="representatives: the paper's merge test on cube representatives alone "
                         "(approximate; cubes as search groups only)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}); the multi-GPU form of "
              f"this path is a design, not a measured mode", file=sys.stderr)
        return 2

    if args.workload == "batch":
        return bench_batch(args)
    if args.workload == "served":
        return bench_served(args)

    from paper_1912_00323_amd.datagen import make_config, make_high

    w = make_high(54, HIGH_N) if args.workload == "54d" else make_config(WORKLOADS[args.workload])
    res = measure(w, args.steps, args.warmup, args.merge, not args.no_cpu_baseline)
    line = {
        "metric": METRIC,
        "value": res["value"],
        "unit": "points/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": res["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "i32",
        "data": "synthetic",
        "config": {"workload": w.name, "n": w.n, "d": w.d, "eps": w.eps, "min_pts": w.min_pts,
                   "fixed_point_bits": w.q, "parallelism": "single-gpu", "merge": args.merge},
    }
    line.update({k: v for k, v in res.items() if k not in ("value", "ms_per_step")})
    if args.workload == "2d" and args.merge == "exact" and not args.no_second:
        # the metric's second workload (8-D, 500k points), measured the same way
        w8 = make_config(WORKLOADS["8d"])
        r8 = measure(w8, args.steps, args.warmup, "exact", not args.no_cpu_baseline)
        line["blobs8d_500k"] = {"config": {"workload": w8.name, "n": w8.n, "d": w8.d, "eps": w8.eps,
                                           "min_pts": w8.min_pts, "fixed_point_bits": w8.q}, **r8}
    print(json.dumps(line), flush=True)
    return 0


def measure(w, steps: int, warmup: int, merge: str, with_cpu: bool) -> dict:
    """Time `steps` whole clustering calls on workload w (points resident in
    HBM) and derive the dominant phase's roofline; optionally time the CPU
    oracle beside it."""
    import torch
    from paper_1912_00323_amd import hca

    dev = torch.device("cuda:0")
    pts = torch.from_numpy(w.points).to(dev)
    labels = torch.empty(w.n, dtype=torch.int32, device=dev)
    ctx = hca.Context(0)
    stream = torch.cuda.current_stream(dev)
    ctx.set_stream(stream.cuda_stream)
    approx = None
    if merge == "representatives":
        exact_labels = ctx.cluster(pts, w.eps, w.min_pts).cpu().numpy()
        ctx.set_exact(False)
        approx = disagreement(exact_labels, ctx.cluster(pts, w.eps, w.min_pts).cpu().numpy())

    for _ in range(warmup):
        ctx.cluster(pts, w.eps, w.min_pts, out=labels)

    # per-phase breakdown and pair-test counts (HIP events on the library's
    # stream around every phase), outside the timed region
    ctx.set_profiling("all")
    acc = {p: [] for p in hca.PHASES}
    tests = {k: [] for k in ALU_PHASES.values()}
    stats = None
    for _ in range(max(3, min(steps, 10))):
        _, stats = ctx.cluster(pts, w.eps, w.min_pts, out=labels, stats=True)
        for p, v in ctx.phase_times().items():
            acc[p].append(v)
        for k in tests:
            tests[k].append(stats[k])
    phase_ms = {p: statistics.mean(v) for p, v in acc.items()}
    dominant = max(phase_ms, key=phase_ms.get)

    # timed region: K whole clustering calls, inputs resident in HBM; only the
    # dominant phase is bracketed by HIP events (two per call).  Small calls
    # are timed without: they have no phases of their own, and a call under
    # profiling takes the general path in their place, so the phase figures
    # are those of profiled calls after the timed ones
    plain = w.n <= SMALL_CALL
    ctx.set_profiling(None if plain else dominant)
    dom_ix = hca.PHASES.index(dominant)
    dom_ms = []
    reuse0 = ctx.plan_reuse_counts()
    # the timed calls go through the C ABI with their arguments checked and
    # marshalled once (the binding's per-call checks stay out of the loop)
    call = ctx.prepared(pts, w.eps, w.min_pts, labels)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        call()
        if not plain:
            dom_ms.append(ctx.phase_time(dom_ix))
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    reuse1 = ctx.plan_reuse_counts()
    if plain:
        ctx.set_profiling(dominant)
        for _ in range(max(3, min(steps, 10))):
            call()
            dom_ms.append(ctx.phase_time(dom_ix))
    ctx.set_profiling(None)
    # for reference, outside the timed region: the same calls with plan reuse
    # off, each waiting for its own bounding box before the rest is launched
    ctx.set_plan_reuse(False)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(steps):
        call()
    torch.cuda.synchronize()
    dt_off = time.perf_counter() - t1
    ctx.set_plan_reuse(True)
    ms_per_step = dt * 1e3 / steps
    dom = statistics.mean(dom_ms)
    key_bytes = 8 if stats["key_bits"] > 32 or w.d > 8 else 4
    kernels = PHASE_KERNELS_HIGH if w.d > 8 else PHASE_KERNELS

    def traffic(phase):
        t = measured_traffic(phase, w.name)
        return t, ("profiles/pmc_traffic.json, taken on the current kernel sources" if t is not None else
                   "no PMC run of the current kernel sources for this phase and workload")

    def hbm_roofline(phase, ms):
        ab = algorithmic_bytes(phase, w.n, w.d, key_bytes, stats["sort_passes"], stats["n_cells"])
        achieved = ab / (ms * 1e-3) / 1e9
        t, src = traffic(phase)
        return {"bound": "hbm", "phase": phase, "kernels": kernels[phase],
                "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": t, "traffic_source": src,
                "algorithmic_bytes": ab, "phase_ms": round(ms, 4)}

    def alu_roofline(phase, ms):
        n_tests = statistics.mean(tests[ALU_PHASES[phase]])
        if phase == "core" and stats["packed_rows"]:
            # byte planes on the matrix units: four products over the axes
            # padded to a multiple of 32
            per_test = 4 * 2 * (-(-w.d // 32) * 32)
            achieved = per_test * n_tests / (ms * 1e-3) / 1e12
            return {"bound": "mfma", "phase": phase, "kernels": kernels[phase],
                    "achieved": round(achieved, 1), "peak": round(MFMA_PEAK_TOPS, 1),
                    "unit": "Tops/s (int8 matrix ops)", "frac": round(achieved / MFMA_PEAK_TOPS, 5),
                    "traffic": traffic(phase)[0], "traffic_source": traffic(phase)[1], "pair_tests": n_tests,
                    "ops_per_test": per_test, "phase_ms": round(ms, 4)}
        ops = 3.0 * w.d * n_tests                        # d sub + d mul + (d-1) add + compare
        achieved = ops / (ms * 1e-3) / 1e12
        t, src = traffic(phase)
        return {"bound": "alu", "phase": phase, "kernels": kernels[phase],
                "achieved": round(achieved, 4), "peak": round(ALU_PEAK_TOPS, 2),
                "unit": "Tops/s (int32 lane-ops)", "frac": round(achieved / ALU_PEAK_TOPS, 5),
                "traffic": t, "traffic_source": src, "pair_tests": n_tests,
                "ops_per_test": 3 * w.d, "phase_ms": round(ms, 4)}

    if dominant in ALU_PHASES:
        roofline = alu_roofline(dominant, dom)
    elif dominant in HBM_PHASES:
        roofline = hbm_roofline(dominant, dom)
    else:
        t, src = traffic(dominant)
        roofline = {"bound": "alu", "phase": dominant, "kernels": kernels[dominant],
                    "achieved": None, "peak": round(ALU_PEAK_TOPS, 2), "unit": "Tops/s (int32 lane-ops)",
                    "frac": None, "traffic": t, "traffic_source": src, "phase_ms": round(dom, 4)}
    out = {
        "value": w.n * steps / dt,
        "ms_per_step": round(ms_per_step, 4),
        "roofline": roofline,
        "roofline_binning_sort": hbm_roofline("sort", phase_ms["sort"]),
        "phase_ms": {p: round(v, 4) for p, v in phase_ms.items() if v > 0},
        "stats": stats,
        "plan_reuse": {"timed_calls_planned_ahead": reuse1[0] - reuse0[0],
                       "timed_calls_run_again": reuse1[1] - reuse0[1],
                       "ms_per_step_without": round(dt_off * 1e3 / steps, 4),
                       "note": "every call computes its bounding box; a call planned from the previous "
                               "calls' box has it compared on the device and runs again if it differs"},
    }
    if plain:
        out["phase_note"] = ("the timed calls take the path for small calls; phases, stats and roofline are those of "
                             "profiled calls, which take the general path")
    if approx is not None:
        out["approximate"] = approx
    ctx.close()
    if with_cpu and approx is None:
        out["cpu_baseline"] = cpu_baseline(w)
    return out


def disagreement(exact, approx) -> dict:
    """How far labels from the representative-only merge are from exact DBSCAN.
    Core points and noise are the same in both, and a representative-only merge
    implies an exact one, so each exact cluster falls apart into fragments; a
    point disagrees when it lies outside the largest fragment of its cluster."""
    import numpy as np
    noise_diff = int(np.count_nonzero((exact < 0) != (approx < 0)))
    m = (exact >= 0) & (approx >= 0)
    e, a = exact[m].astype(np.int64), approx[m].astype(np.int64)
    pair, cnt = np.unique(e * (int(a.max(initial=0)) + 1) + a, return_counts=True)
    owner = pair // (int(a.max(initial=0)) + 1)
    best = np.zeros(int(e.max(initial=-1)) + 1, np.int64)
    np.maximum.at(best, owner, cnt)
    frags = np.bincount(owner, minlength=best.size)
    differ = int(m.sum() - best.sum()) + noise_diff
    return {"points_differing": differ, "fraction": differ / max(1, exact.size),
            "clusters_exact": int(best.size), "clusters_approx": int(np.unique(a).size),
            "exact_clusters_split": int(np.count_nonzero(frags > 1)), "noise_differing": noise_diff}


def bench_batch(args) -> int:
    """The batched workload: 256 independent data sets (n log-uniform in
    [1e3, 2e5], d in {2, 3, 4}, per-set eps and minPts).  One step = one
    batch through a batch handle: a graph launch of the plan captured (and
    tuned) on the handle's first run.  Timed beside it on the same data: the
    same handle with default knobs, the host-planned batch call
    (hca_cluster_batch) and the plain path (one hca_cluster call per set)."""
    import tempfile
    import torch
    import numpy as np
    from paper_1912_00323_amd import hca
    from paper_1912_00323_amd.datagen import make_batch

    jobs = make_batch(seed=4, count=256)
    total = sum(j.n for j in jobs)
    dev = torch.device("cuda:0")
    rows = [j.n for j in jobs]
    dims = [j.d for j in jobs]
    eps = [j.eps for j in jobs]
    mps = [j.min_pts for j in jobs]
    sets = [torch.from_numpy(j.points).to(dev) for j in jobs]
    outs = [torch.empty(j.n, dtype=torch.int32, device=dev) for j in jobs]
    ctx = hca.Context(0)
    ctx.set_stream(torch.cuda.current_stream(dev).cuda_stream)

    def timed(fn, steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / steps

    # the tuned handle (a fresh cache, so the tuning is measured every run)
    cache = tempfile.NamedTemporaryFile(prefix="hca_tune_", suffix=".json", delete=False).name
    os.environ["HCA_TUNE_CACHE"] = cache
    tuned = hca.Batch(ctx, rows, dims, eps, mps, tune=2)
    t_first = timed(lambda: tuned.run(sets, outs), 1)        # plan + tune + capture
    for _ in range(args.warmup):
        tuned.run(sets, outs)
    dt = timed(lambda: tuned.run(sets, outs), args.steps)
    graph_labels = [o.clone() for o in outs]
    st = tuned.stats()
    default = hca.Batch(ctx, rows, dims, eps, mps, tune=0)
    default.run(sets, outs)
    dt_default = timed(lambda: default.run(sets, outs), max(3, args.steps // 2))
    same_default = all(torch.equal(a, b) for a, b in zip(graph_labels, outs))
    # the host-planned batch call (phase times of its groups for the roofline)
    flat = torch.from_numpy(np.concatenate([j.points.reshape(-1) for j in jobs])).to(dev)
    labels = torch.empty(total, dtype=torch.int32, device=dev)
    ctx.cluster_batch(flat, rows, dims, eps, mps, out=labels)
    dt_planned = timed(lambda: ctx.cluster_batch(flat, rows, dims, eps, mps, out=labels), max(3, args.steps // 2))
    same_planned = bool(torch.equal(torch.cat(graph_labels), labels))
    ctx.set_profiling("all")
    ctx.cluster_batch(flat, rows, dims, eps, mps, out=labels)
    phase_ms = ctx.phase_times()
    ctx.set_profiling(None)
    # the plain path on the same data: one call per data set, inputs resident
    for x, o, j in zip(sets, outs, jobs):
        ctx.cluster(x, j.eps, j.min_pts, out=o)
    dt_plain = timed(lambda: [ctx.cluster(x, j.eps, j.min_pts, out=o) for x, o, j in zip(sets, outs, jobs)],
                     max(1, min(3, args.steps)))
    same_plain = all(torch.equal(a, b) for a, b in zip(graph_labels, outs))

    # binning and sort bytes of every group from its plan's key width and
    # passes, against the sort phase of the host-planned call
    ab = 0.0
    for g in st["groups"]:
        kb = 8 if g["key_bits"] > 32 else 4
        ab += algorithmic_bytes("sort", g["rows"], g["d"], kb, g["sort_passes"], 0)
    sort_ms = phase_ms["sort"]
    achieved = ab / (sort_ms * 1e-3) / 1e9 if sort_ms > 0 else None
    ms = dt * 1e3
    line = {
        "metric": METRIC,
        "value": total / dt,
        "unit": "points/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "i32",
        "data": "synthetic",
        "config": {"workload": "batch256_mixed", "jobs": len(jobs), "points": total,
                   "d": sorted(set(dims)), "parallelism": "single-gpu", "form": "batch handle, one graph launch"},
        "graph": {"replays": st["graph_replays"], "plans": st["plans"], "first_run_ms": round(t_first * 1e3, 2),
                  "groups": st["groups"]},
        "default_knobs": {"ms_per_batch": round(dt_default * 1e3, 3), "labels_identical": same_default},
        "tuned_vs_default": round(dt_default / dt, 3),
        "host_planned_batch": {"ms_per_batch": round(dt_planned * 1e3, 3), "labels_identical": same_planned},
        "plain_path": {"value": total / dt_plain, "unit": "points/s", "ms_per_batch": round(dt_plain * 1e3, 3),
                       "calls": len(jobs), "labels_identical": same_plain},
        "speedup_vs_plain": round(dt_plain / dt, 3),
        "phase_ms": {p: round(v, 4) for p, v in phase_ms.items() if v > 0},
        "roofline": {"bound": "hbm", "phase": "sort (all groups, host-planned call)",
                     "kernels": PHASE_KERNELS["sort"], "achieved": round(achieved, 1) if achieved else None,
                     "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4) if achieved else None, "traffic": None,
                     "traffic_source": "no PMC run of the batched sequence",
                     "algorithmic_bytes": ab, "phase_ms": round(sort_ms, 4)},
    }
    tuned.close()
    default.close()
    if not args.no_cpu_baseline:
        import oracle
        threads = host_threads()
        done, pts_done, t_start = 0, 0, time.perf_counter()
        while done < len(jobs) and time.perf_counter() - t_start < 20.0:
            j = jobs[done]
            oracle.hca_grid(j.points, j.eps, j.min_pts, threads=threads)
            done += 1
            pts_done += j.n
        tcpu = time.perf_counter() - t_start
        line["cpu_baseline"] = {"value": pts_done / tcpu, "unit": "points/s", "cores": threads, "kind": "oracle",
                                "sample": f"the first {done} of the {len(jobs)} data sets ({pts_done} points), "
                                          f"one oracle.hca_grid call each", "cpu_model": cpu_model()}
    print(json.dumps(line), flush=True)
    ctx.close()
    try:
        os.unlink(cache)
    except OSError:
        pass
    return 0


def bench_served(args, workers: int = 2) -> int:
    """The served workload: Poisson arrivals of --requests distinct clustering
    requests (n log-uniform in [1e4, 2e6], d in {2, 3, 5}, per-request eps and
    minPts; points drawn on the device from a seeded torch generator) at
    several loads, given as multiples of the request rate the plain sequential
    path sustains.  The request loop (hca_server: continuous batching over
    `workers` workers, batches bounded by estimated device time) and the
    plain path (one hca_cluster call at a time, in arrival order) replay the
    same arrival trace; latency = completion - arrival.  Each path's
    throughput is compared at the highest load whose p99 stays within the
    SLO (--slo-ms)."""
    import torch
    import numpy as np
    from paper_1912_00323_amd import hca
    from paper_1912_00323_amd.datagen import device_request, poisson_arrivals, served_requests

    loads = tuple(float(v) for v in args.loads.split(","))
    reqs = served_requests(seed=5, count=args.requests)
    dev = torch.device("cuda:0")

    def note(msg):
        print(f"[served] {msg}", file=sys.stderr, flush=True)

    xs = []
    for k, r in enumerate(reqs):
        xs.append(device_request(r, dev))
        if k % 1000 == 999:
            note(f"drew {k + 1} requests")
    outs = [torch.empty(r["n"], dtype=torch.int32, device=dev) for r in reqs]
    points = sum(r["n"] for r in reqs)
    ctx = hca.Context(0)
    ctx.set_stream(torch.cuda.current_stream(dev).cuda_stream)
    # reference labels and the plain path's sustained rate (one pass, warm)
    ref = [ctx.cluster(x, r["eps"], r["min_pts"]) for x, r in zip(xs[:64], reqs[:64])]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ref = []
    for k, (x, r) in enumerate(zip(xs, reqs)):
        ref.append(ctx.cluster(x, r["eps"], r["min_pts"]))
        if k % 1000 == 999:
            note(f"plain reference pass: {k + 1} requests")
    torch.cuda.synchronize()
    plain_rate = len(reqs) / (time.perf_counter() - t0)
    note(f"plain path sustains {plain_rate:.1f} requests/s")
    srv = hca.Server(0, workers=workers, budget_bytes=48 << 30, max_batch=64, batch_ms=args.batch_ms)
    same = True
    count = len(reqs)

    def plain(arr):
        lat = []
        start = hca.clock() + 0.02
        for k, r in enumerate(reqs):
            while hca.clock() < start + arr[k]:
                pass
            ctx.cluster(xs[k], r["eps"], r["min_pts"], out=outs[k])
            lat.append(hca.clock() - (start + arr[k]))
            if k % 2000 == 1999:
                note(f"plain: {k + 1} requests")
        return lat, hca.clock() - start

    def served(arr):
        nonlocal same
        for o in outs:
            o.fill_(-9)
        done = {}
        start = hca.clock() + 0.02
        for k, r in enumerate(reqs):
            while hca.clock() < start + arr[k]:
                for t, st, td in srv.poll():
                    done[t] = (st, td)
            srv.submit(xs[k], r["eps"], r["min_pts"], outs[k], tag=k)
            if k % 2000 == 1999:
                note(f"served: {k + 1} requests submitted")
        srv.drain()
        for t, st, td in srv.poll(1 << 20):
            done[t] = (st, td)
        same = same and all(done[k][0] == 0 and torch.equal(outs[k], ref[k]) for k in range(count))
        lat = [done[k][1] - (start + arr[k]) for k in range(count)]
        return lat, max(done[k][1] for k in range(count)) - start

    def summary(lat, span):
        v = np.asarray(lat) * 1e3
        return {"p50_ms": round(float(np.percentile(v, 50)), 3), "p99_ms": round(float(np.percentile(v, 99)), 3),
                "points_per_s": points / span}

    sweep = {}
    for load in loads:
        arr = poisson_arrivals(5, count, load * plain_rate)
        sweep[str(load)] = {"arrival_rate_per_s": round(load * plain_rate, 2),
                            "served": summary(*served(arr)), "plain_sequential": summary(*plain(arr))}
        print(f"[load {load}] {json.dumps(sweep[str(load)])}", file=sys.stderr, flush=True)
    saturated = None
    if args.saturated:
        zero = np.zeros(count)
        saturated = {"served": summary(*served(zero)), "plain_sequential": summary(*plain(zero))}
    srv.close()
    ctx.close()

    def at_slo(path):
        ok = [float(l) for l in sweep if sweep[l][path]["p99_ms"] <= args.slo_ms]
        if not ok:
            return None
        best = str(max(ok))
        return {"load": float(best), "points_per_s": sweep[best][path]["points_per_s"],
                "p99_ms": sweep[best][path]["p99_ms"]}

    slo = {"slo_ms": args.slo_ms, "served": at_slo("served"), "plain_sequential": at_slo("plain_sequential")}
    main = max(sweep, key=lambda l: (sweep[l]["served"]["p99_ms"] <= args.slo_ms, float(l)))
    line = {
        "metric": METRIC,
        "value": sweep[main]["served"]["points_per_s"],
        "unit": "points/s",
        "n_gpus": 1,
        "steps": count,
        "warmup": 64,
        "ms_per_step": round(points / sweep[main]["served"]["points_per_s"] * 1e3 / count, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "i32",
        "data": "synthetic (drawn on the device from a seeded torch generator)",
        "config": {"workload": "served_poisson", "requests": count, "load_vs_plain": float(main),
                   "arrival_rate_per_s": round(float(main) * plain_rate, 3), "points": points,
                   "d": sorted(set(r["d"] for r in reqs)), "workers": workers, "batch_ms": args.batch_ms,
                   "parallelism": "single-gpu"},
        "served": sweep[main]["served"],
        "plain_sequential": sweep[main]["plain_sequential"] | {"sustained_requests_per_s": round(plain_rate, 3)},
        "throughput_at_slo": slo,
        "load_sweep": sweep,
        "saturated": saturated,
        "labels_identical": bool(same),
        "roofline": {"bound": None, "phase": None, "achieved": None, "peak": None, "unit": None, "frac": None,
                     "traffic": None,
                     "reason": "requests of 2, 3 and 5 axes run different launch sequences side by side; the "
                               "roofline of each is that of the plain path at its shape (the 2-D and 8-D lines)"},
    }
    print(json.dumps(line), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
