"""Throughput of the PrefixPlace planner hot path on one MI355X.

One step = one full plan (standalone scores, WorkerGreedy, coordinate
refinement until no sweep improves, best start) of the tree50k workload
(n = 50,000 chunks, M = 16 workers, k = 4,096 each, 8 order-diverse starts,
source-dependent fetch costs) through the device-resident C-ABI entry point,
inputs already in HBM.  Prints one JSON line.  After the timed region:
  configs      the other four synthetic workloads (tiny, tree2k, rag10k,
               chat50k), each planned on the GPU and checked against the
               oracle's stored plan, the small ones also timed on the
               oracle (full plans, one thread and one thread per start)
  replan       epoch re-planning after a 50% routing shift (host arrays)
  f64          the same workload in the paper's units, as doubles
  paper_config the paper's own timing configuration (k = 128)
  cpu_baseline the oracle on a bounded sample of the headline workload
--no-configs, --no-replan, --no-f64, --no-paper-config and
--no-cpu-baseline skip them.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME]
"""

from __future__ import annotations

import argparse
import hashlib
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# The rooted-tree DP sweep (k_dp) keeps its rows on chip: per cell it moves
# about one byte of HBM traffic (choice bits and stage-boundary words) and
# executes a fixed number of vector instructions, so the bound that applies
# is vector instruction issue.  MI355X: 256 CUs x 4 SIMDs x 16 lanes at
# 2.4 GHz = 39.32e12 32-bit lane operations per second.
VALU_PEAK_TOPS = 256 * 4 * 16 * 2.4e9 / 1e12
# LDS: 128 bytes per clock per CU.
LDS_PEAK_GBS = 256 * 128 * 2.4e9 / 1e9
HBM_PEAK_GBS = 8000.0
# Algorithmic bytes per DP cell in the table formulation of Theorem 1 (8 B
# write of D[i][j], 8 B read of D[next(i)][j], one choice bit): the model
# the HBM fraction of the metric is quoted on.  k_dp does not move these
# bytes, so the model fraction exceeds 1; it is reported under its own name.
TABLE_BYTES_PER_CELL = 16.125
# Gains bytes per (worker, chunk) and per chunk of one update (k_gains:
# demand, recompute and fetch as int64, top-1, top-2 and holder; profit).
GAIN_BYTES_PER_MN, GAIN_BYTES_PER_N = 41, 8
# Eq. 9 per cell, as 32-bit integer operations: the take operand's 64-bit
# add (two), the 64-bit comparison and the two selects of the maximum, and
# the choice bit shifted into its word.
ALGO_OPS_PER_CELL = 6
METRIC = ("full PrefixPlace plans/sec and tree-DP cells/sec "
          "(n·k·updates/s), 1 GPU")
# Paper context: n = 50,000, M = 16 solved in 12.29 s on one EPYC 9V74 with
# k = 128 (Sec. V, RQ5) -- a different capacity, so not a like-for-like
# baseline.
PAPER_CONTEXT = "n=50,000, M=16, k=128: 12.29 s per plan on one EPYC 9V74"

# HBM traffic of the DP sweep as measured by hardware counters (FETCH_SIZE
# and WRITE_SIZE per dispatch, each scaled by what the same counter reads for
# a device copy of known size).  The summary records a digest of the sources
# that decide the kernel and its launch; a different digest means the
# counters describe another kernel and the figure is not reported.
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "k_dp_hbm_traffic.md")
KERNEL_SOURCES = ("paper_2608_01655_amd/csrc/pp_kernels.hip",
                  "paper_2608_01655_amd/csrc/pp_internal.h",
                  "paper_2608_01655_amd/csrc/pp_host.cpp")


def dp_valu_per_step(cells, fmax, f64):
    """Vector instructions the DP sweep's compute wave issues per row step
    (64 * cells cells): two row addresses; cell 0's take operand (a DPP
    64-bit add, or for doubles two DPP moves and an add); with several
    cells per lane the profit moved into lane 0 (two DPP moves) and the
    other cells' take operands (one 64-bit add each); per cell the choice
    bit (compare, add with carry), the skip operand (two bit selects) and
    the maximum (one v_max_f64, or a compare and two selects).  The SQ
    counters of one cell per lane and the compiled code of every width
    agree (profiles/)."""
    return (2 + (3 if f64 else 2) + (2 + (cells - 1) if cells > 1 else 0)
            + cells * (4 + (1 if fmax else 3)))


def dp_lds_bytes_per_cell(cells):
    """LDS bytes per DP cell: the compute wave's step record (16 B per
    lane), row store and skip row read (8 B per cell each), one gathered
    column per group of sink rows; the I/O wave's staging (two 16-byte views
    for 33 lanes per 32-step batch)."""
    sink = 16 if cells == 1 else 4
    per_step = 64 * 16 + 2 * 64 * cells * 8 + 64 * 8 / sink + 2 * 16 * 33 / 32
    return per_step / (64 * cells)


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def kernel_sources_digest():
    h = hashlib.sha256()
    for rel in KERNEL_SOURCES:
        with open(os.path.join(ROOT, rel), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def measured_traffic(workload):
    """HBM bytes per DP-sweep launch from the committed counter summary, or
    None if there is none for this workload and these kernel sources."""
    try:
        with open(TRAFFIC_FILE) as fh:
            text = fh.read()
    except OSError:
        return None
    for m in re.finditer(r"<!-- traffic (\{.*?\}) -->", text):
        rec = json.loads(m.group(1))
        if rec.get("workload") == workload and \
                rec.get("sources_sha256") == kernel_sources_digest():
            return float(rec["bytes_per_launch"])
    return None


def copy_probe(mib):
    """A device-to-device copy of known size, for calibrating the HBM byte
    counters (run under rocprofv3 --pmc)."""
    import torch

    n = mib * 2 ** 20 // 8
    a = torch.arange(n, dtype=torch.int64, device="cuda")
    b = torch.empty_like(a)
    torch.cuda.synchronize()
    for _ in range(3):
        b.copy_(a)
    torch.cuda.synchronize()
    ok = bool(torch.equal(a, b))
    print(json.dumps({"copy_bytes": n * 8, "copies": 3, "equal": ok}),
          flush=True)
    return 0 if ok else 1


def host_description():
    """CPU model (the full /proc/cpuinfo identification: model name, family,
    model and stepping), logical CPUs, CPUs this process may run on, and
    memory of the machine the bench runs on."""
    info, mem_kib = {}, None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                key, _, val = line.partition(":")
                key = key.strip()
                if key in ("model name", "cpu family", "model", "stepping",
                           "vendor_id", "cpu MHz") and key not in info:
                    info[key] = val.strip()
                if not line.strip() and info:
                    break
        with open("/proc/meminfo") as fh:
            for line in fh:
                if line.startswith("MemTotal"):
                    mem_kib = int(line.split()[1])
                    break
    except OSError:
        pass
    try:
        usable = len(os.sched_getaffinity(0))
    except (AttributeError, OSError):
        usable = os.cpu_count()
    model = info.get("model name")
    if model and "family" not in model:
        model = (f"{model} (vendor {info.get('vendor_id')}, family "
                 f"{info.get('cpu family')}, model {info.get('model')}, "
                 f"stepping {info.get('stepping')}, {info.get('cpu MHz')} MHz)")
    return {"cpu_model": model, "host_cpus": os.cpu_count(),
            "usable_cpus": usable,
            "mem_gib": round(mem_kib / 2 ** 20, 1) if mem_kib else None}


def oracle_threads(starts):
    """One oracle thread per start, at most the CPUs this process may use."""
    try:
        usable = len(os.sched_getaffinity(0))
    except (AttributeError, OSError):
        usable = os.cpu_count() or 1
    return max(1, min(starts, usable))


def cpu_baseline(inst, plan_cells, threads):
    """The oracle as it stands, on a bounded sample of the same workload:
    Algorithm 1 with the sweep cap set to one -- the standalone pass, the
    greedy pass and the first refinement sweep of every start, every cell
    of every DP table computed and the objective recomputed from scratch at
    every acceptance test -- one thread per start.  plans/s = the sample's
    DP cells per second / the DP cells of one full plan (Algorithm 1's
    count, as the GPU reports it)."""
    import oracle

    oracle.lib()
    t0 = time.perf_counter()
    res = oracle.plan_instance(inst, max_rounds=1, threads=threads)
    dt = time.perf_counter() - t0
    cps = res.dp_cells / dt
    return {
        "value": cps / plan_cells,
        "unit": "plans/s",
        "cells_per_s": cps,
        "cores": threads,
        "kind": "oracle",
        "sample": (f"{inst.name} with the refinement sweeps capped at one: "
                   f"standalone, greedy and first refinement sweep of all "
                   f"{inst.n_starts} starts ({res.updates} worker updates, "
                   f"{res.dp_cells:.3e} DP cells) in {dt:.1f} s on "
                   f"{threads} threads; plans/s = cells/s / "
                   f"{plan_cells:.4e} cells of one full plan"),
        "sample_seconds": dt,
        **host_description(),
    }


def plan_timing(B, ctx, inst, lam, w, f, tgt, steps, warmup, plan_flags=0):
    """Plans of `inst` through the device entry point (inputs in HBM);
    returns the per-plan wall times, the last plan and the kernel totals."""
    import torch

    def step(flags=0):
        return ctx.pp_plan_device(inst.parent, lam, w, f, inst.cap, tgt,
                                  n_starts=inst.n_starts,
                                  max_rounds=inst.max_rounds,
                                  order_seed=inst.order_seed,
                                  flags=flags | plan_flags)

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    plans, marks = [], []
    for _ in range(steps):
        plans.append(step(B.PP_F_TIME_KERNELS))
        marks.append(time.perf_counter())  # the call returns after its stream drained
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    step_ms = sorted((b - a) * 1e3 for a, b in zip([t0] + marks[:-1], marks))
    return dt, step_ms, plans


# a reduced solve reads per node: its profit (8), key (4) and parent link (2)
SOLVE_BYTES_PER_N = 14


def all_swept(B, ctx, inst, lam, w, f, tgt, p, plan_flags=0):
    """Whether every solve of plan `p` was a DP sweep: one ran, and a plan
    with the reduced solve switched off takes the same launches for the same
    cells."""
    if p.dp_lane_cells == 0:
        return False
    before = os.environ.get("PP_REDUCE_MIN_N")
    os.environ["PP_REDUCE_MIN_N"] = str(1 << 30)
    try:
        q = ctx.pp_plan_device(inst.parent, lam, w, f, inst.cap, tgt,
                               n_starts=inst.n_starts, max_rounds=inst.max_rounds,
                               order_seed=inst.order_seed,
                               flags=B.PP_F_TIME_KERNELS | plan_flags)
    finally:
        if before is None:
            del os.environ["PP_REDUCE_MIN_N"]
        else:
            os.environ["PP_REDUCE_MIN_N"] = before
    return (q.dp_launches, q.dp_cells_executed) == (p.dp_launches, p.dp_cells_executed)


def dp_figures(inst, plans, dt, swept):
    """Throughput and roofline figures of a series of plans: plan-level
    cells per second (Algorithm 1's count, and that of the updates solved:
    n * k each, whether a sweep visits them or a reduced solve proves them
    away), the same per second inside the solve launches and, where every
    solve is a sweep (`swept`), its fraction of the vector-issue ceiling, of
    the LDS peak and, under the table model, of HBM."""
    p = plans[-1]
    steps = len(plans)
    exec_cells = sum(q.dp_cells_executed for q in plans)
    dp_ms = sum(q.dp_kernel_ms for q in plans)
    launches = sum(q.dp_launches for q in plans)
    kernel_cps = exec_cells / (dp_ms / 1e3) if dp_ms > 0 else 0.0
    c = max(1, p.dp_lane_cells)
    solved = exec_cells / (inst.n * max(1.0, float(inst.cap.clip(max=inst.n).mean())))
    valu = dp_valu_per_step(c, p.dp_fmax, isinstance(p.objective, float))
    issue_ceiling = VALU_PEAK_TOPS * 1e12 * c / valu  # cells/s
    lds_b = dp_lds_bytes_per_cell(c)
    plan_bytes_table = (exec_cells / steps * TABLE_BYTES_PER_CELL
                        + p.updates * (GAIN_BYTES_PER_MN * inst.m * inst.n
                                       + GAIN_BYTES_PER_N * inst.n))
    return {
        "plans_per_s": steps / dt,
        "ms_per_plan": dt / steps * 1e3,
        "dp_cells_per_s_algorithm1": p.dp_cells * steps / dt,
        "dp_cells_per_s_solved": exec_cells / dt,
        "dp_cells_per_plan_algorithm1": p.dp_cells,
        "dp_cells_per_plan_solved": exec_cells // steps,
        "updates_per_plan": p.updates,
        "dp_lane_cells": p.dp_lane_cells,
        "solves_per_plan": solved / steps,
        # a solve has to read the profits and the tree once
        "solve_hbm_gbs": solved * SOLVE_BYTES_PER_N * inst.n / (dp_ms / 1e3) / 1e9
        if dp_ms > 0 else None,
        "dp_launches_per_plan": launches // steps,
        "dp_avg_launch_ms": dp_ms / launches if launches else None,
        "dp_share_of_plan_time": dp_ms / 1e3 / dt,
        "dp_cells_per_s_in_kernel": kernel_cps,
        "dp_issue_frac": kernel_cps / issue_ceiling if swept else None,
        "dp_valu_per_row_step": valu,
        "dp_lds_frac": kernel_cps * lds_b / (LDS_PEAK_GBS * 1e9) if swept else None,
        "dp_table_model_hbm_frac": kernel_cps * TABLE_BYTES_PER_CELL
        / (HBM_PEAK_GBS * 1e9) if swept else None,
        "plan_table_model_hbm_frac": plan_bytes_table * steps / dt
        / (HBM_PEAK_GBS * 1e9) if swept else None,
        "plan_issue_frac": exec_cells / dt / issue_ceiling if swept else None,
        "sweeps_per_start": p.start_sweeps.tolist(),
    }


def golden_plan(name):
    gold_path = os.path.join(ROOT, "tests", "golden", "plans.json")
    if not os.path.exists(gold_path):
        return None
    with open(gold_path) as fh:
        return json.load(fh).get(name)


def configs_leg(B, W, ctx, names, with_oracle):
    """Every other synthetic workload: plans on the GPU (inputs in HBM; a
    number of plans sized to about a second of GPU time), checked against
    the oracle's stored plan; for the small workloads also full oracle plans
    (one thread, and one thread per start) on the host cores."""
    import numpy as np
    import torch

    out = {}
    dev = torch.device("cuda:0")
    for name in names:
        inst = W.make_workload(name)
        log(f"[bench] config {name}: n={inst.n} m={inst.m} S={inst.n_starts}")
        lam = torch.from_numpy(inst.demand).to(dev)
        w = torch.from_numpy(inst.recompute_cost).to(dev)
        f = torch.from_numpy(inst.fetch_cost).to(dev)
        tgt = torch.zeros((inst.m, inst.n), dtype=torch.uint8, device=dev)
        # one timed plan to size the run
        t1, _, _ = plan_timing(B, ctx, inst, lam, w, f, tgt, 1, 1)
        steps = int(max(3, min(200, 1.0 / max(t1, 1e-4))))
        dt, step_ms, plans = plan_timing(B, ctx, inst, lam, w, f, tgt, steps, 0)
        swept = all_swept(B, ctx, inst, lam, w, f, tgt, plans[-1])
        fig = dp_figures(inst, plans, dt, swept)
        fig["steps"] = steps
        fig["ms_per_plan_median"] = step_ms[len(step_ms) // 2]
        fig["ms_per_plan_min"] = step_ms[0]
        gold = golden_plan(name)
        if gold:
            import hashlib as _h

            target = tgt.cpu().numpy()
            rows = [_h.sha256(np.ascontiguousarray(target[h]).tobytes()).hexdigest()
                    for h in range(inst.m)]
            fig["parity_vs_golden"] = (
                all(q.objective == gold["objective"] for q in plans)
                and plans[-1].start_sweeps.tolist() == gold["start_sweeps"]
                and rows == gold["target_row_sha256"])
        if with_oracle and inst.n * int(inst.cap.max()) <= 2 * 10 ** 7:
            import oracle

            oracle.lib()
            reps = 5 if inst.n <= 2000 else 1
            T = oracle_threads(inst.n_starts)
            o = {}
            for threads in sorted({1, T}):
                t0 = time.perf_counter()
                for _ in range(reps):
                    res = oracle.plan_instance(inst, threads=threads)
                sec = (time.perf_counter() - t0) / reps
                o[f"threads_{threads}"] = {
                    "s_per_plan": sec, "plans_per_s": 1.0 / sec,
                    "dp_cells_per_s": res.dp_cells / sec, "repetitions": reps}
            o["same_objective"] = res.objective == plans[-1].objective
            fig["oracle_full_plan"] = o
        out[name] = fig
    return out


def replan_leg(B, W, inst, steps, warmup):
    """Epoch re-planning (Sec. IV-D) after a 50% routing shift, the incumbent
    being the first k_h preorder chunks of every worker, horizon 1,000
    epochs: the host-array entry point, so the time includes the PCIe copies
    of the inputs and outputs (inputs: demand, costs and incumbent; outputs:
    target and proposal)."""
    lam = W.shift_routing(inst.parent, inst.demand, 1, 2)
    inc = W.prefix_incumbent(inst.n, inst.cap)
    horizon = 1000

    def call():
        return B.pp_replan(inst.parent, lam, inst.recompute_cost,
                           inst.fetch_cost, inst.cap, inc, horizon,
                           n_starts=inst.n_starts, max_rounds=inst.max_rounds,
                           order_seed=inst.order_seed)

    for _ in range(warmup):
        call()
    t0 = time.perf_counter()
    for _ in range(steps):
        r = call()
    dt = (time.perf_counter() - t0) / steps
    out = {"ms_per_replan": dt * 1e3, "includes_pcie": True,
           "shift": "50% routing shift", "horizon": horizon,
           "adopt": r.adopt, "incumbent_objective": r.incumbent_objective,
           "proposal_objective": r.proposal_objective,
           "materialization_cost": r.materialization_cost}
    gain = r.proposal_objective - r.incumbent_objective
    if gain > 0:
        out["break_even_epochs"] = r.materialization_cost // gain + 1
    gold_path = os.path.join(ROOT, "tests", "golden", "replans.json")
    if os.path.exists(gold_path):
        with open(gold_path) as fh:
            gold = json.load(fh).get(f"{inst.name}-shift50")
        if gold:
            out["parity_vs_golden"] = (
                r.adopt == gold["adopt"]
                and r.proposal_objective == gold["proposal_objective"]
                and r.incumbent_objective == gold["incumbent_objective"]
                and r.materialization_cost == gold["materialization_cost"])
    return out


def f64_leg(B, W, inst, ctx, steps, warmup):
    """The same workload in the paper's own units, as doubles (requests per
    epoch and milliseconds, each entry jittered), planned through the
    real-valued device entry point with epsilon = 1e-9 of sum(demand *
    recompute cost); inputs already in HBM."""
    import numpy as np
    import torch

    lam, w, f = W.real_valued(inst, 1)
    eps = 1e-9 * float(np.sum(lam * w))
    dev = torch.device("cuda:0")
    tl = torch.from_numpy(lam).to(dev)
    tw = torch.from_numpy(w).to(dev)
    tf = torch.from_numpy(f).to(dev)
    tgt = torch.zeros((inst.m, inst.n), dtype=torch.uint8, device=dev)

    def call(flags=0):
        return ctx.pp_plan_f64_device(inst.parent, tl, tw, tf, inst.cap, tgt,
                                      epsilon=eps, n_starts=inst.n_starts,
                                      max_rounds=inst.max_rounds,
                                      order_seed=inst.order_seed, flags=flags)

    for _ in range(warmup):
        call()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    plans = [call(B.PP_F_TIME_KERNELS) for _ in range(steps)]
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / steps
    p = plans[-1]
    dp_ms = sum(q.dp_kernel_ms for q in plans)
    launches = sum(q.dp_launches for q in plans)
    out = {"plans_per_s": 1.0 / dt, "ms_per_plan": dt * 1e3,
           "dp_avg_launch_ms": dp_ms / launches,
           "dp_launches_per_plan": launches // steps,
           "dp_cells_per_s_in_kernel":
               sum(q.dp_cells_executed for q in plans) / (dp_ms / 1e3),
           "objective": p.objective, "epsilon": eps,
           "sweeps_per_start": p.start_sweeps.tolist(),
           "units": "requests/epoch and ms, per-entry jitter U[0.75, 1.25]"}
    gold_path = os.path.join(ROOT, "tests", "golden", "plans_f64.json")
    if os.path.exists(gold_path):
        with open(gold_path) as fh:
            gold = json.load(fh).get(inst.name)
        if gold:
            out["parity_vs_golden"] = all(
                q.best_start == gold["best_start"]
                and q.start_sweeps.tolist() == gold["start_sweeps"]
                and q.objective == float.fromhex(gold["objective"]) for q in plans)
    return out


def _runtime_point(B, W, ctx, inst, steps, with_oracle):
    """One of the paper's solver-runtime configurations: the instance in
    requests per epoch and milliseconds as doubles (epsilon = 1e-9 of the
    sum of demand x recompute cost), planned through the real-valued device
    entry point with the instance's start set and refinement to
    convergence; with `with_oracle`, the CPU oracle (one thread, the full DP
    table) on the same inputs."""
    import numpy as np
    import torch

    lam, w, f = W.real_valued(inst, 1)
    eps = 1e-9 * float(np.sum(lam * w))
    dev = torch.device("cuda:0")
    tl = torch.from_numpy(lam).to(dev)
    tw = torch.from_numpy(w).to(dev)
    tf = torch.from_numpy(f).to(dev)
    tgt = torch.zeros((inst.m, inst.n), dtype=torch.uint8, device=dev)
    kw = dict(epsilon=eps, n_starts=inst.n_starts, max_rounds=inst.max_rounds,
              order_seed=inst.order_seed)
    ctx.pp_plan_f64_device(inst.parent, tl, tw, tf, inst.cap, tgt, **kw)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        p = ctx.pp_plan_f64_device(inst.parent, tl, tw, tf, inst.cap, tgt, **kw)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / steps
    out = {"ms_per_plan": dt * 1e3, "starts": int(p.n_starts), "updates_per_plan": p.updates,
           "sweeps_per_start": p.start_sweeps.tolist(), "objective": p.objective}
    if with_oracle:
        import oracle

        oracle.lib()
        t1 = time.perf_counter()
        o = oracle.plan_f64(inst.parent, lam, w, f, inst.cap, **kw)
        out["oracle_s_per_plan_1_thread"] = time.perf_counter() - t1
        out["same_as_oracle"] = (
            bool(np.array_equal(o.target, tgt.cpu().numpy()))
            and o.objective == p.objective)
    return out, dt


def paper_config_leg(B, W, ctx, steps, with_oracle):
    """The configurations of the paper's own solver timing (k = 128 per
    worker): n = 50,000 with M = 16 -- the tree50k tree and demand with every
    capacity set to 128, 8 starts -- and n = 10,000 with M = 4, 8 and 16 --
    the RAG-shaped tree and demand of rag10k split over M workers, the
    paper's default start set (every order for M = 4) -- all real-valued,
    refinement to convergence.  The paper reports 12.29 s and 0.41, 1.12,
    2.35 s per plan on one EPYC 9V74 for its own inputs of these sizes
    (context: other inputs and hardware); the CPU oracle (one thread) is
    timed on the same inputs as a second point of reference."""
    import dataclasses

    import numpy as np

    inst = W.make_workload("tree50k")
    inst = dataclasses.replace(inst, cap=np.full(inst.m, 128, np.int32))
    pt, dt = _runtime_point(B, W, ctx, inst, steps, with_oracle)
    out = {"workload": "tree50k tree and demand, k = 128 for all 16 workers, "
                       "real-valued (requests, ms)",
           **pt, "paper_s_per_plan": 12.29, "paper_hardware": "one EPYC 9V74",
           "ratio_paper_time_to_this": 12.29 / dt}
    points = []
    for m, paper_s in ((4, 0.41), (8, 1.12), (16, 2.35)):
        pt, dt = _runtime_point(B, W, ctx, W.runtime_instance(m), max(steps, 3), with_oracle)
        points.append({"n": 10_000, "workers": m, "k": 128, **pt, "paper_s_per_plan": paper_s,
                       "ratio_paper_time_to_this": paper_s / dt})
    out["n10k_points"] = points
    out["n10k_workload"] = ("rag10k tree and demand split over M workers, k = 128, "
                            "the paper's default start set, real-valued (requests, ms)")
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="tree50k")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--safeguards", action="store_true",
                    help="requester-side variant of the workload (each "
                         "requester's fetch cost taken from one source) "
                         "planned with the comparator safeguards")
    ap.add_argument("--no-configs", action="store_true",
                    help="skip the other synthetic workloads")
    ap.add_argument("--configs", default="tiny,tree2k,rag10k,chat50k",
                    help="comma-separated workloads of the configs object")
    ap.add_argument("--no-replan", action="store_true",
                    help="skip the re-planning leg")
    ap.add_argument("--no-host-plan", action="store_true",
                    help="skip the timing of the host-array entry point")
    ap.add_argument("--no-f64", action="store_true",
                    help="skip the real-valued leg")
    ap.add_argument("--no-paper-config", action="store_true",
                    help="skip the leg at the paper's own timing configuration")
    ap.add_argument("--paper-config-only", action="store_true",
                    help="only the leg at the paper's own timing configuration "
                         "(prints its object; for kernel traces of that leg)")
    ap.add_argument("--oracle-full", action="store_true",
                    help="also time one full oracle plan of the workload "
                         "(minutes at 50,000 chunks)")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="MIB",
                    help="only copy MIB MiB device to device (counter "
                         "calibration) and exit")
    args = ap.parse_args()
    if args.copy_probe:
        sys.exit(copy_probe(args.copy_probe))
    if args.gpus != 1:
        print("bench.py runs on exactly one GPU: the planner's starts would "
              "shard across GPUs with one exchange of (objective, start) "
              "pairs, which this implementation does not run", file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_2608_01655_amd import binding as B
    from paper_2608_01655_amd import workloads as W

    if not os.path.exists(B.LIB_PATH):
        from paper_2608_01655_amd import build

        build.build()
    if args.paper_config_only:
        ctx = B.Context(0)
        out = paper_config_leg(B, W, ctx, max(1, min(args.steps, 3)),
                               not args.no_cpu_baseline)
        ctx.close()
        print(json.dumps({"paper_config": out}), flush=True)
        return
    inst = W.make_workload(args.workload)
    plan_flags = 0
    if args.safeguards:
        import dataclasses

        f_req = inst.fetch_cost.copy()
        for dst in range(inst.m):
            src0 = 1 if dst == 0 else 0
            for src in range(inst.m):
                if src != dst and inst.m > 1:
                    f_req[src, dst] = inst.fetch_cost[src0, dst]
        inst = dataclasses.replace(inst, name=inst.name + "-requester-side",
                                   fetch_cost=f_req)
        plan_flags = B.PP_F_SAFEGUARDS
    log(f"[bench] workload {inst.name}: n={inst.n} m={inst.m} "
        f"k={int(inst.cap.min())}..{int(inst.cap.max())} S={inst.n_starts}")
    dev = torch.device("cuda:0")
    lam = torch.from_numpy(inst.demand).to(dev)
    w = torch.from_numpy(inst.recompute_cost).to(dev)
    f = torch.from_numpy(inst.fetch_cost).to(dev)
    tgt = torch.zeros((inst.m, inst.n), dtype=torch.uint8, device=dev)
    ctx = B.Context(0)

    dt, step_ms, plans = plan_timing(B, ctx, inst, lam, w, f, tgt, args.steps,
                                     args.warmup, plan_flags)
    for i, q in enumerate(plans):
        log(f"[bench] step {i}: objective {q.objective} dp {q.dp_kernel_ms:.1f} ms")
    p = plans[-1]
    objectives = {q.objective for q in plans}
    gold = golden_plan(inst.name)
    gold_ok = (objectives == {gold["objective"]}) if gold else None
    swept = all_swept(B, ctx, inst, lam, w, f, tgt, p, plan_flags)
    fig = dp_figures(inst, plans, dt, swept)
    exec_cells = sum(q.dp_cells_executed for q in plans)
    dp_ms = sum(q.dp_kernel_ms for q in plans)
    launches = sum(q.dp_launches for q in plans)
    avg_launch_s = dp_ms / launches / 1e3
    cells_per_launch = exec_cells / launches
    c = max(1, p.dp_lane_cells)
    valu = fig["dp_valu_per_row_step"]
    # lane operations one launch issues for the DP (VALU instructions per
    # row step x 64 lanes per 64*C cells), over its measured duration
    achieved = cells_per_launch * valu / c / avg_launch_s / 1e12
    traffic = measured_traffic(inst.name)
    real = "true" if isinstance(p.objective, float) else "false"
    if swept:
        roofline = {
            "bound": "alu",
            "kernel": f"k_dp<{c}, {'true' if p.dp_fmax else 'false'}, false> "
                      "(rooted-tree DP sweep)",
            "achieved": achieved,
            "peak": VALU_PEAK_TOPS,
            "unit": "T lane-ops/s (32-bit vector)",
            "frac": achieved / VALU_PEAK_TOPS,
            "traffic": traffic,
            "ops_basis": (f"{valu} vector instructions per row step of "
                          f"{64 * c} cells (compute wave; SQ_INSTS_VALU), "
                          f"each one 32-bit op per lane"),
            "cells_per_launch": cells_per_launch,
            "dp_launches_per_plan": launches // args.steps,
            "avg_launch_ms": avg_launch_s * 1e3,
            "dp_cells_per_s_in_kernel": fig["dp_cells_per_s_in_kernel"],
            "dp_share_of_plan_time": fig["dp_share_of_plan_time"],
            # Eq. 9's own arithmetic (6 ops per cell) against the same peak
            "algorithmic_frac": fig["dp_cells_per_s_in_kernel"]
            * ALGO_OPS_PER_CELL / (VALU_PEAK_TOPS * 1e12),
            "lds": {"bytes_per_cell": dp_lds_bytes_per_cell(c),
                    "achieved_gbs": fig["dp_cells_per_s_in_kernel"]
                    * dp_lds_bytes_per_cell(c) / 1e9,
                    "peak_gbs": LDS_PEAK_GBS,
                    "frac": fig["dp_lds_frac"]},
            "hbm_measured": ({"gbs": traffic / avg_launch_s / 1e9,
                              "frac": traffic / avg_launch_s / 1e9 / HBM_PEAK_GBS,
                              "bytes_per_cell": traffic / cells_per_launch}
                             if traffic else None),
            # Theorem 1's table formulation (16.125 B per cell) against HBM
            # peak: above 1 because the sweep keeps the table on chip
            "hbm_table_model": {"bytes_per_cell": TABLE_BYTES_PER_CELL,
                                "achieved_gbs": fig["dp_cells_per_s_in_kernel"]
                                * TABLE_BYTES_PER_CELL / 1e9,
                                "frac": fig["dp_table_model_hbm_frac"]},
        }
    else:
        # the reduced solve: one block a chain, bound by the serial chain of
        # its phases; against HBM, the bytes its solves cannot do without
        roofline = {
            "bound": "hbm",
            "kernel": f"k_ladder<{real}> + k_reduce<{real}> (reduced exact tree solve)"
                      + (", k_dp where it leaves a chain" if p.dp_lane_cells else ""),
            "achieved": fig["solve_hbm_gbs"],
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": fig["solve_hbm_gbs"] / HBM_PEAK_GBS,
            "traffic": None,
            "bytes_basis": f"{SOLVE_BYTES_PER_N} bytes a node and solve (profit, key, link)",
            "cells_per_launch": cells_per_launch,
            "dp_launches_per_plan": launches // args.steps,
            "avg_launch_ms": avg_launch_s * 1e3,
            "dp_cells_per_s_in_kernel": fig["dp_cells_per_s_in_kernel"],
            "dp_share_of_plan_time": fig["dp_share_of_plan_time"],
        }
    out = {
        "metric": METRIC,
        "value": args.steps / dt,
        "unit": "plans/s",
        # Algorithm 1's cells (every update n * min(k_h, n)) per second
        "dp_cells_per_s": fig["dp_cells_per_s_algorithm1"],
        # n * k of the updates solved, by a reduced solve or a sweep (updates of
        # workers whose inputs did not change need none; discarded
        # speculative updates add theirs)
        "dp_cells_executed_per_s": fig["dp_cells_per_s_solved"],
        "dp_cells_per_s_frac_issue_roofline": fig["plan_issue_frac"],
        "dp_cells_per_s_frac_hbm_table_model": fig["dp_cells_per_s_solved"]
        * TABLE_BYTES_PER_CELL / (HBM_PEAK_GBS * 1e9) if swept else None,
        "plans_per_s_frac_hbm_table_model": fig["plan_table_model_hbm_frac"],
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": dt / args.steps * 1e3,
        "ms_per_step_median": step_ms[len(step_ms) // 2],
        "ms_per_step_min": step_ms[0],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int64",
        "data": "synthetic",
        "config": {
            "workload": inst.name, "n": inst.n, "workers": inst.m,
            "k": [int(x) for x in sorted(set(inst.cap.tolist()))],
            "starts": inst.n_starts, "max_rounds": inst.max_rounds,
            "updates_per_plan": p.updates, "dp_cells_per_plan": p.dp_cells,
            "dp_cells_executed_per_plan": exec_cells // args.steps,
            "sweeps_per_start": p.start_sweeps.tolist(),
        },
        "roofline": roofline,
        "parity_vs_golden": gold_ok,
        **({"safeguards": {"run": p.safeguards_run, "returned": p.best_start,
                           "objectives": list(p.safeguard_objective)}}
           if args.safeguards else {}),
        "paper_context": PAPER_CONTEXT,
    }
    # the host-array entry point on the same inputs: PCIe copies of the
    # inputs and the placement inside the call
    host_ms = []
    for _ in range(0 if args.no_host_plan else 2):
        t1 = time.perf_counter()
        hp = B.pp_plan(inst.parent, inst.demand, inst.recompute_cost,
                       inst.fetch_cost, inst.cap, n_starts=inst.n_starts,
                       max_rounds=inst.max_rounds, order_seed=inst.order_seed,
                       flags=plan_flags)
        host_ms.append((time.perf_counter() - t1) * 1e3)
    if host_ms:
        out["host_pp_plan_ms"] = min(host_ms)
        out["host_pp_plan_same_objective"] = hp.objective == p.objective
    if not args.no_configs and not args.safeguards:
        names = [x for x in args.configs.split(",") if x and x != inst.name]
        out["configs"] = configs_leg(B, W, ctx, names, not args.no_cpu_baseline)
    if not args.no_replan and not args.safeguards:
        log("[bench] re-planning leg")
        out["replan"] = replan_leg(B, W, inst, max(1, min(args.steps, 3)),
                                   min(args.warmup, 1))
    if not args.no_f64 and not args.safeguards:
        log("[bench] real-valued leg")
        out["f64"] = f64_leg(B, W, inst, ctx, max(1, min(args.steps, 3)),
                             min(args.warmup, 1))
    if not args.no_paper_config and not args.safeguards:
        log("[bench] paper-configuration leg (k = 128)")
        out["paper_config"] = paper_config_leg(B, W, ctx, max(1, min(args.steps, 3)),
                                                not args.no_cpu_baseline)
    if not args.no_cpu_baseline:
        threads = oracle_threads(inst.n_starts)
        log(f"[bench] timing the CPU oracle on a bounded sample ({threads} threads)")
        out["cpu_baseline"] = cpu_baseline(inst, p.dp_cells, threads)
    if args.oracle_full:
        import oracle

        threads = oracle_threads(inst.n_starts)
        log(f"[bench] timing one full oracle plan ({threads} threads)")
        oracle.lib()
        t1 = time.perf_counter()
        res = oracle.plan_instance(inst, threads=threads)
        sec = time.perf_counter() - t1
        out["oracle_full_plan"] = {"s_per_plan": sec, "plans_per_s": 1.0 / sec,
                                   "threads": threads,
                                   "dp_cells_per_s": res.dp_cells / sec,
                                   "same_objective": res.objective == p.objective}
    ctx.close()
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
