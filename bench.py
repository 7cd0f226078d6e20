#!/usr/bin/env python3
"""Benchmark of the per-time-step core update (arXiv 2504.13750, JANC) on one MI355X.

Workload (default): the 2-D 9-species reacting front on a 3-level block-structured
AMR hierarchy -- 1024 x 512 base cells in 64 x 64 blocks, ratio-2 levels of 8x8 ..
64x64 blocks, 637 valid blocks, 1,975,360 cells; synthetic 9-species / 19-reaction
reversible mechanism (seed 13750); WENO5 + Lax-Friedrichs + SSP-RK3, Newton for T,
point-implicit chemistry, synchronous advance with restriction; FP64.

Metric: FP64 cell-stage updates/s = (cells of valid blocks, ring cells included)
x 3 RK stages x steps / wall time of the timed region, inputs resident in HBM.
Reported beside it: the same update in the per-block launch form (one launch per
block and stage), the stage kernel's roofline position (FP64 VALU bound)
from HIP events, and the CPU oracle on a bounded sample.

python bench.py [--gpus 1] [--steps K] [--warmup W]
"""

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "FP64 cell-stage updates/s (2D 9-species AMR) vs per-block form; adjoint/fwd cost"

PEAK_FP64_VALU_TFLOPS = 78.6   # MI355X FP64 vector, FMA counted as 2 flops
PEAK_HBM_GBS = 8000.0

# Algorithmic FP64 flops of one owned cell and one RK stage in the fused stage
# kernel, counted from its formulas (an FMA is two flops, a division or square
# root one): a WENO5 reconstruction is 67 flops (three candidate stencils,
# three smoothness indicators, the weighted average with one division); an
# interface flux is two reconstructions plus their sum (135); per component and
# direction a cell also forms its split fluxes (6.2 on average), the flux
# difference (2) and the RK combination (4 on average over the three stages).
WENO = 67.0
IFACE = 2 * WENO + 1


def stage_flops(model, nU, twod):
    dirs = 2 if twod else 1
    per_comp = dirs * (IFACE + 6.2 + 2.0) + 4.0 + (1.0 if twod else 0.0)
    if model == 2:      # NASA-7: primitives 26, Newton (coefficients + ~2 iterations + cv, c) 200
        extra = 26 + 200
    elif model == 1:    # one-step: primitives 14, T and sound speed 15, explicit source 6
        extra = 14 + 15 + 6
    else:
        extra = 12 + 12
    return nU * per_comp + extra + 6.0   # + wave-speed maxima


def stage_bytes(nU):
    """Algorithmic HBM bytes per cell and stage: read U^(s-1) and T, read U^n in
    stages 2 and 3, write U^(s) and T (average over the three stages)."""
    return 8.0 * ((nU + 1 + nU + 1) + 2 * (nU + 1 + nU + nU + 1)) / 3.0


def log(msg):
    print(msg, file=sys.stderr, flush=True)


STAGE_SOURCES = ("csrc/janc_device.h", "csrc/janc_internal.h", "csrc/janc_kernels.h",
                 "csrc/janc_species.hip", "build.py")


def kernel_source_hash():
    """sha256[:16] of the sources and build flags the stage kernel is compiled from."""
    import hashlib
    h = hashlib.sha256()
    for f in STAGE_SOURCES:
        with open(os.path.join(ROOT, "paper_2504_13750_amd", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(width, linear):
    """HBM bytes per stage-kernel launch of the schedule (tile width, workgroup order) from
    the committed FETCH_SIZE / WRITE_SIZE counter passes (profiles/, one line per
    schedule: source hash, width, order, bytes), or None when the kernel sources changed
    since or the schedule was not measured."""
    path = os.path.join(ROOT, "profiles", "stage_kernel_traffic.txt")
    order = "linear" if linear else "xcd"
    try:
        with open(path) as fh:
            for line in fh:
                f = line.split()
                if len(f) == 4 and f[0] == kernel_source_hash() and int(f[1]) == width \
                        and f[2] == order:
                    return float(f[3])
    except (OSError, ValueError):
        return None
    return None


def optional(name, fn):
    """Run an optional section of the benchmark: a failure is logged and recorded in its
    place, and the headline measurement is still printed."""
    try:
        return fn()
    except Exception as e:  # noqa: BLE001
        log(f"[bench] {name} failed: {type(e).__name__}: {e}")
        return {"error": f"{type(e).__name__}: {e}"}


def host_cpu():
    """Model name and logical CPU count of the host that runs the oracle."""
    model = None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"model": model, "logical_cpus": os.cpu_count(),
            "affinity_cpus": len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity")
            else None}


def cpu_baseline(case, steps, target_s=10.0, max_steps=20):
    """The oracle on the same workload: `steps` steps, extended to about target_s of work."""
    import oracle
    U, T = oracle.block_state(case)
    t0 = time.perf_counter()
    U, T, t, _, _ = oracle.step_blocks(case, U, T, steps)
    el = time.perf_counter() - t0
    if el < 0.8 * target_s:
        more = min(max_steps - steps, int(math.ceil(target_s / (el / steps))) - steps)
        if more > 0:
            t1 = time.perf_counter()
            oracle.step_blocks(case, U, T, more, t=t)
            el += time.perf_counter() - t1
            steps += more
    cells = case.valid_cells()
    out = {"value": cells * 3 * steps / el, "unit": "cell-stage/s",
           "cores": oracle.max_threads(), "kind": "oracle", "host": host_cpu(),
           "sample": f"{steps} step(s) of the same {len(case.blocks)}-block AMR workload "
                     f"({cells} cells), OpenMP over all host threads, {el:.1f} s"}
    # the same oracle on one host thread, one step
    nthreads = oracle.max_threads()
    oracle.set_threads(1)
    try:
        U1, T1 = oracle.block_state(case)
        t0 = time.perf_counter()
        oracle.step_blocks(case, U1, T1, 1)
        el1 = time.perf_counter() - t0
    finally:
        oracle.set_threads(nthreads)
    out["one_thread"] = {"value": cells * 3 / el1, "unit": "cell-stage/s",
                         "sample": f"1 step of the same workload on 1 thread, {el1:.1f} s"}
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=40)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--per-block-steps", type=int, default=8)
    ap.add_argument("--kernel-reps", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-per-block", action="store_true")
    ap.add_argument("--no-adjoint", action="store_true")
    ap.add_argument("--no-crossover", action="store_true")
    ap.add_argument("--no-regrid", action="store_true")
    ap.add_argument("--no-ensemble", action="store_true")
    ap.add_argument("--cpu-steps", type=int, default=1)
    ap.add_argument("--paper-shape", action="store_true",
                    help="also time the uniform 9-species path on a 4000 x 1000 grid, the shape "
                         "of the paper's single-GPU core-solver run (context only)")
    ap.add_argument("--schedule", default=None, metavar="WIDTH/ORDER",
                    help="fix the stage launch shape instead of autotuning it, e.g. 32/xcd or "
                         "16/linear (counter passes)")
    ap.add_argument("--calibrate-copy-mib", type=int, default=0,
                    help="run one device copy of this size first (HBM counter calibration)")
    args = ap.parse_args()
    fixed = None
    if args.schedule is not None:
        w, _, o = args.schedule.partition("/")
        if w not in ("16", "32", "64") or o not in ("xcd", "linear"):
            ap.error("--schedule takes WIDTH/ORDER with WIDTH 16, 32 or 64 and ORDER xcd or linear")
        fixed = (int(w), int(o == "linear"))
    if args.gpus != 1:
        print("bench.py measures one GPU: this build has no multi-GPU path "
              "(run with --gpus 1).", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import paper_2504_13750_amd as janc
    from cases import amr_case

    dev = torch.device("cuda:0")
    torch.cuda.init()
    if args.calibrate_copy_mib > 0:
        n = args.calibrate_copy_mib * 1024 * 1024 // 8
        a = torch.ones(n, dtype=torch.float64, device=dev)
        b = torch.empty_like(a)
        b.copy_(a)
        torch.cuda.synchronize()
        del a, b

    log("[bench] generating the AMR workload")
    case = amr_case()
    nU = case.nU
    cells = case.valid_cells()
    ctx = janc.Context(janc.DETAILED, case.mech)
    domains = janc.domains_of(case)
    tm = janc.time_of(case)

    def fresh_state():
        W = torch.tensor(case.W, dtype=torch.float64, device=dev)
        U = torch.empty_like(W)
        T = torch.empty(case.pool_cells, dtype=torch.float64, device=dev)
        dom = case.domains[0]
        u, tt = ctx.init_state(janc.physics_of(dom), W)
        U.copy_(u)
        T.copy_(tt)
        return U, T, torch.zeros(1, dtype=torch.float64, device=dev)

    def timed_run(plan, steps, warmup, sim=None):
        U, T, t = fresh_state()
        if warmup:
            ctx.step_blocks(plan, tm, U, T, warmup, t)
        ctx.sync_status()
        t_start = float(t[0].item())
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        w0 = time.perf_counter()
        e0.record()
        ctx.step_blocks(plan, tm, U, T, steps, t)
        e1.record()
        torch.cuda.synchronize()
        wall = time.perf_counter() - w0
        ctx.sync_status()
        if sim is not None:
            sim.append(float(t[0].item()) - t_start)   # simulated time of the timed steps
        return e0.elapsed_time(e1) / 1e3, wall, (U, T, t)

    # ------------------------------------------------------------ fused batched form
    log(f"[bench] fused batched step: {len(case.blocks)} blocks, {cells} cells, "
        f"{args.warmup} warm-up + {args.steps} timed steps")
    # default launch shape (16 x 16 tiles, XCD-contiguous tile runs), then the shape the
    # autotuner picks on the workload's own state; the headline is the tuned plan
    dplan = ctx.plan(domains, case.blocks, case.pool_cells, janc.PLAN_DEFAULT)
    d_s, _, _ = timed_run(dplan, args.steps, args.warmup)
    dplan.close()
    default_value = cells * 3 * args.steps / d_s
    log(f"[bench] default shape: {1e3 * d_s / args.steps:.3f} ms/step, {default_value:.4e} cell-stage/s")
    plan = ctx.plan(domains, case.blocks, case.pool_cells, janc.PLAN_DEFAULT)
    if fixed is None:
        U0, T0, _ = fresh_state()
        choice, cand_ms = plan.autotune(tm, U0, T0, reps=5)
        del U0, T0
        log(f"[bench] autotuner: tile width {choice[0]}, "
            f"{'linear' if choice[1] else 'XCD-contiguous'} order; candidates (median ms per "
            f"stage triple) "
            + ", ".join(f"{w}/{'lin' if l else 'xcd'} {v:.3f}" for (w, l), v in cand_ms.items()))
    else:
        choice, cand_ms = fixed, {}
        plan.set_schedule(*fixed)
        log(f"[bench] fixed schedule: tile width {fixed[0]}, "
            f"{'linear' if fixed[1] else 'XCD-contiguous'} order")
    sim_sync = []
    gpu_s, wall_s, (U, T, t) = timed_run(plan, args.steps, args.warmup, sim_sync)
    value = cells * 3 * args.steps / gpu_s
    ms_step = 1e3 * gpu_s / args.steps
    log(f"[bench] {ms_step:.3f} ms/step, {value:.4e} cell-stage/s (wall {wall_s:.3f} s)")
    autotune = {"tile_width": choice[0], "order": "linear" if choice[1] else "xcd-contiguous",
                "fixed": fixed is not None,
                "candidates_ms": {f"{w}/{'linear' if l else 'xcd'}": v for (w, l), v in cand_ms.items()},
                "default_shape_value": default_value, "gain_over_default": value / default_value}

    # ------------------------------------------------------------ per-kernel timing (HIP events)
    stage_ms, chem_ms, restr_ms, ring_ms = [], [], [], []
    for _ in range(args.kernel_reps):
        ms = ctx.profile_step(plan, tm, U, T, t)
        stage_ms += ms[0:3]
        chem_ms.append(ms[3])
        restr_ms.append(ms[4])
        ring_ms.append(ms[5])
    # the chemistry kernel specialised to the mechanism's structure (the default) against
    # the generic one, same state and plan
    chem_kernel = "specialized" if ctx.chem_kernel == janc.CHEM_SPECIALIZED else "generic"
    chem_generic_ms = None
    if chem_kernel == "specialized":
        ctx.chem_kernel = janc.CHEM_GENERIC
        chem_generic_ms = float(np.mean([ctx.profile_step(plan, tm, U, T, t)[3]
                                         for _ in range(args.kernel_reps)]))
        ctx.chem_kernel = janc.CHEM_SPECIALIZED
    ctx.sync_status()
    stage_avg = sum(stage_ms) / len(stage_ms)
    pst = plan.stats()
    ring_cells = int(pst["ring_cells"])
    assert pst["cells"] == cells
    solved = cells - ring_cells
    flops = stage_flops(2, nU, True) * solved
    achieved_tf = flops / (stage_avg * 1e-3) / 1e12
    bytes_launch = stage_bytes(nU) * solved
    achieved_gbs = bytes_launch / (stage_avg * 1e-3) / 1e9
    log(f"[bench] stage kernel {stage_avg:.3f} ms avg: {achieved_tf:.2f} TFLOP/s FP64, "
        f"{achieved_gbs:.0f} GB/s algorithmic; chemistry {np.mean(chem_ms):.3f} ms, "
        f"restriction {np.mean(restr_ms):.3f} ms, ring {np.mean(ring_ms):.3f} ms")
    if chem_generic_ms is not None:
        log(f"[bench] chemistry kernel specialised to the mechanism {np.mean(chem_ms):.3f} ms, "
            f"generic {chem_generic_ms:.3f} ms")

    # ------------------------------------------------------------ per-block launch form
    def _per_block():
        per_block = None
        pplan = ctx.plan(domains, case.blocks, case.pool_cells,
                         janc.PLAN_PER_BLOCK | janc.PLAN_NO_GRAPH)
        pb_s, _, _ = timed_run(pplan, args.per_block_steps, 1)
        pb_value = cells * 3 * args.per_block_steps / pb_s
        per_block = {"value": pb_value, "unit": "cell-stage/s",
                     "ms_per_step": 1e3 * pb_s / args.per_block_steps,
                     "steps": args.per_block_steps,
                     "speedup_of_fused": value / pb_value,
                     "form": "one launch per block and RK stage"}
        log(f"[bench] per-block form {per_block['ms_per_step']:.3f} ms/step "
            f"-> fused speed-up {value / pb_value:.2f}x")
        pplan.close()
        # the paper's structure: one batched launch per refinement level and stage
        lplan = ctx.plan(domains, case.blocks, case.pool_cells, janc.PLAN_PER_LEVEL)
        pl_s, _, _ = timed_run(lplan, args.steps, args.warmup)
        pl_value = cells * 3 * args.steps / pl_s
        per_block["per_level"] = {"value": pl_value, "unit": "cell-stage/s",
                                  "ms_per_step": 1e3 * pl_s / args.steps, "steps": args.steps,
                                  "speedup_of_fused": value / pl_value,
                                  "form": "one launch per refinement level and RK stage "
                                          "(per-level batching, Alg. 2)"}
        log(f"[bench] per-level form {per_block['per_level']['ms_per_step']:.3f} ms/step "
            f"-> fused speed-up {value / pl_value:.2f}x")
        lplan.close()
        return per_block
    per_block = None if args.no_per_block else optional("per_block", _per_block)

    # ------------------------------------------------------------ crossover advance
    def _crossover():
        crossover = None
        xplan = ctx.plan(domains, case.blocks, case.pool_cells, janc.PLAN_CROSSOVER)
        xsteps = max(1, args.steps // 4)
        sim_x = []
        x_s, _, _ = timed_run(xplan, xsteps, 1, sim_x)
        lev_cells = {}
        for b in case.blocks:
            if b["valid"]:
                lev_cells[int(b["level"])] = lev_cells.get(int(b["level"]), 0) + int(b["nx"] * b["ny"])
        x_updates = sum(n * (1 << l) for l, n in lev_cells.items()) * 3 * xsteps
        rate_x = sim_x[0] / x_s
        rate_s = sim_sync[0] / gpu_s
        crossover = {"ms_per_step": 1e3 * x_s / xsteps, "steps": xsteps,
                     "cell_stage_per_s": x_updates / x_s,
                     "simulated_time_per_s": rate_x,
                     "synchronous_simulated_time_per_s": rate_s,
                     "speedup_vs_synchronous": rate_x / rate_s,
                     "form": "Fig. 2a: per level dt_0/2^l, deepest level first"}
        log(f"[bench] crossover advance {crossover['ms_per_step']:.3f} ms per level-0 step, "
            f"{rate_x / rate_s:.2f}x the synchronous advance in simulated time per second")
        xplan.close()
        return crossover
    crossover = None if args.no_crossover else optional("crossover", _crossover)

    # ------------------------------------------------------------ layer update (regridding)
    def _regrid():
        regrid = None
        thr, buf, sub, every = 0.05, 4, 8, 40
        U0, T0, t0 = fresh_state()
        ctx.step_blocks(plan, tm, U0, T0, 2, t0)

        def one_update():
            torch.cuda.synchronize()
            w0 = time.perf_counter()
            blocks, pool = ctx.regrid(plan, U0, thr, buf, sub)
            w1 = time.perf_counter()
            nplan = ctx.plan(domains, blocks, pool, janc.PLAN_DEFAULT)
            w2 = time.perf_counter()
            Un, Tn = ctx.regrid_fill(plan, U0, T0, nplan)
            torch.cuda.synchronize()
            w3 = time.perf_counter()
            return (w1 - w0, w2 - w1, w3 - w2), blocks, nplan, Un, Tn

        one_update()[2].close()                    # warm-up
        reps = [one_update() for _ in range(3)]
        best = min(reps, key=lambda r: sum(r[0]))
        for r in reps:
            if r is not best:
                r[2].close()
        (t_flag, t_plan, t_fill), nblocks, nplan, Un, Tn = best
        total = t_flag + t_plan + t_fill
        ncells = int(np.sum(nblocks["nx"].astype(np.int64) * nblocks["ny"]))
        # the step on the updated hierarchy
        tn = t0.clone()
        ctx.step_blocks(nplan, tm, Un, Tn, 2, tn)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        rsteps = max(1, args.steps // 4)
        torch.cuda.synchronize()
        e0.record()
        ctx.step_blocks(nplan, tm, Un, Tn, rsteps, tn)
        e1.record()
        torch.cuda.synchronize()
        ctx.sync_status()
        r_s = e0.elapsed_time(e1) / 1e3
        regrid = {"criterion": f"density gradient, threshold {thr}, buffer {buf}, subregion {sub}",
                  "blocks_before": int(len(case.blocks)), "blocks_after": int(len(nblocks)),
                  "cells_after": ncells,
                  "levels_after": [int(x) for x in np.bincount(nblocks["level"])],
                  "regrid_ms": 1e3 * t_flag, "plan_ms": 1e3 * t_plan, "fill_ms": 1e3 * t_fill,
                  "update_ms": 1e3 * total,
                  "every_steps": every,
                  "amortized_ms_per_step": 1e3 * total / every,
                  "amortized_fraction_of_step": (1e3 * total / every) / ms_step,
                  "updated_hierarchy_ms_per_step": 1e3 * r_s / rsteps,
                  "updated_hierarchy_cell_stage_per_s": ncells * 3 * rsteps / r_s}
        log(f"[bench] layer update {1e3 * total:.2f} ms (criterion {1e3 * t_flag:.2f}, plan "
            f"{1e3 * t_plan:.2f}, fill {1e3 * t_fill:.2f}); {len(case.blocks)} -> {len(nblocks)} "
            f"blocks, {ncells} cells; every {every} steps: {1e3 * total / every:.3f} ms/step; "
            f"updated hierarchy {1e3 * r_s / rsteps:.3f} ms/step")
        nplan.close()
        return regrid
    regrid = None if args.no_regrid else optional("regrid", _regrid)

    # ------------------------------------------------------------ ensemble batching
    def _ensemble():
        ensemble = None
        from cases import ensemble_case
        ens = ensemble_case()
        ectx = janc.Context(janc.ONESTEP)
        eplan = ectx.plan(janc.domains_of(ens), ens.blocks, ens.pool_cells, janc.PLAN_DEFAULT)
        We = torch.tensor(ens.W, dtype=torch.float64, device=dev)
        Ue = torch.empty_like(We)
        Te = torch.empty(ens.pool_cells, dtype=torch.float64, device=dev)
        flops, ecells = 0.0, 0
        for b in ens.blocks:
            dom = ens.domains[int(b["domain"])]
            s0, n = int(b["offset"]), int(b["nx"]) * int(b["ny"])
            u, tt = ectx.init_state(janc.physics_of(dom), We[:, s0:s0 + n].contiguous())
            Ue[:, s0:s0 + n] = u
            Te[s0:s0 + n] = tt
            flops += n * stage_flops(1, 5, dom.ny > 1)
            ecells += n
        te = torch.zeros(len(ens.domains), dtype=torch.float64, device=dev)
        etm = janc.time_of(ens)
        ectx.step_blocks(eplan, etm, Ue, Te, 2, te)
        esteps = 20
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record()
        ectx.step_blocks(eplan, etm, Ue, Te, esteps, te)
        e1.record()
        torch.cuda.synchronize()
        e_s = e0.elapsed_time(e1) / 1e3
        est = float(np.mean([np.mean(ectx.profile_step(eplan, etm, Ue, Te, te)[0:3])
                             for _ in range(2)]))
        ectx.sync_status()
        tf = flops / (est * 1e-3) / 1e12
        gbs = ecells * stage_bytes(5) / (est * 1e-3) / 1e9
        ensemble = {"workload": f"{len(ens.domains)} one-step instances "
                                f"({sum(d.ny == 1 for d in ens.domains)} 1-D), {ecells} cells",
                    "ms_per_step": 1e3 * e_s / esteps, "steps": esteps,
                    "cell_stage_per_s": ecells * 3 * esteps / e_s,
                    "stage_kernel_ms": est, "fp64_tflops": tf,
                    "fp64_frac": tf / PEAK_FP64_VALU_TFLOPS,
                    "hbm_algorithmic_GBs": gbs, "hbm_frac": gbs / PEAK_HBM_GBS}
        log(f"[bench] ensemble {ensemble['workload']}: {ensemble['ms_per_step']:.3f} ms/step, "
            f"{ensemble['cell_stage_per_s']:.3e} cell-stage/s; stage kernel {est:.3f} ms = "
            f"{tf:.2f} TFLOP/s ({100 * tf / PEAK_FP64_VALU_TFLOPS:.1f} %), {gbs:.0f} GB/s algorithmic")
        eplan.close()
        ectx.close()
        return ensemble
    ensemble = None if args.no_ensemble else optional("ensemble", _ensemble)

    # ------------------------------------------------------------ adjoint / forward cost
    def _adjoint():
        adjoint = None
        from cases import adjoint_case
        a = adjoint_case()
        ac = a["case"]
        actx = janc.Context(janc.ONESTEP)
        aph = janc.physics_of(ac)
        ag = janc.grid_of(ac)
        atm = janc.make_time(0.0, ac.dt_fixed, 0.0)
        W0 = torch.tensor(ac.W, dtype=torch.float64, device=dev)

        def fwd():
            U0, T0 = actx.init_state(aph, W0)
            t0 = torch.zeros(1, dtype=torch.float64, device=dev)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            actx.step(ag, aph, atm, U0, T0, ac.nsteps, t0)
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / 1e3

        def adj():
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            out = actx.adjoint(ag, aph, atm, W0, ac.nsteps, a["ckpt_every"], a["probe_cell"],
                               a["probe_w"])
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / 1e3, out

        fwd()
        adj()                      # warm-up (workspace)
        tf = min(fwd() for _ in range(3))
        ta = min(adj()[0] for _ in range(3))
        actx.sync_status()
        adjoint = {"workload": f"one-step tube {ac.nx}x{ac.ny}, {ac.nsteps} steps, "
                               f"checkpoints every {a['ckpt_every']}",
                   "forward_s": tf, "adjoint_s": ta, "adjoint_over_forward": ta / tf}
        log(f"[bench] adjoint {ta * 1e3:.2f} ms vs forward {tf * 1e3:.2f} ms: "
            f"{ta / tf:.2f}x")
        actx.close()

        # the detailed model (9 species: NASA-7 Newton, point-implicit chemistry)
        from cases.amr import detailed_adjoint_case
        d = detailed_adjoint_case(nx=128, ny=64, nsteps=40)
        dc = d["case"]
        dctx = janc.Context(janc.DETAILED, dc.mech)
        dph, dg = janc.physics_of(dc), janc.grid_of(dc)
        dW0 = torch.tensor(dc.W, dtype=torch.float64, device=dev)
        # the fixed dt: the CFL step (at cfl_dt) of the initial state, from one GPU step
        U1, T1 = dctx.init_state(dph, dW0)
        dtl = torch.zeros(1, dtype=torch.float64, device=dev)
        dctx.step(dg, dph, janc.make_time(cfl=d["cfl_dt"]), U1, T1, 1,
                  torch.zeros(1, dtype=torch.float64, device=dev), dtl)
        dc.dt_fixed = float(dtl.item())
        del U1, T1
        dtm = janc.make_time(0.0, dc.dt_fixed, 0.0)
        dk = 10

        def dfwd():
            U0, T0 = dctx.init_state(dph, dW0)
            t0 = torch.zeros(1, dtype=torch.float64, device=dev)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            dctx.step(dg, dph, dtm, U0, T0, dc.nsteps, t0)
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / 1e3

        def dadj():
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            dctx.adjoint(dg, dph, dtm, dW0, dc.nsteps, dk, d["probe_cell"], d["probe_w"])
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / 1e3

        dfwd()
        dadj()
        tfd = min(dfwd() for _ in range(3))
        tad = min(dadj() for _ in range(3))
        # both runs with the generic chemistry kernels, for comparison
        dctx.chem_kernel = janc.CHEM_GENERIC
        dfwd()
        dadj()
        tfg = min(dfwd() for _ in range(3))
        tag = min(dadj() for _ in range(3))
        dctx.sync_status()
        dctx.close()
        adjoint["detailed"] = {"workload": f"9-species front {dc.nx}x{dc.ny}, {dc.nsteps} steps, "
                                           f"checkpoints every {dk}",
                               "forward_s": tfd, "adjoint_s": tad, "adjoint_over_forward": tad / tfd,
                               "generic_chemistry": {"forward_s": tfg, "adjoint_s": tag,
                                                     "adjoint_over_forward": tag / tfg}}
        log(f"[bench] detailed-model adjoint {tad * 1e3:.2f} ms vs forward {tfd * 1e3:.2f} ms: "
            f"{tad / tfd:.2f}x (generic chemistry kernels: {tag * 1e3:.2f} vs {tfg * 1e3:.2f} ms, "
            f"{tag / tfg:.2f}x)")
        return adjoint
    adjoint = None if args.no_adjoint else optional("adjoint", _adjoint)

    # ------------------------------------------------------------ uniform grid, paper's shape
    def _paper_shape():
        from cases.amr import detailed_front_case
        pc = detailed_front_case(nx=4000, ny=1000, mech=case.mech)
        pctx = janc.Context(janc.DETAILED, pc.mech)
        pph = janc.physics_of(pc)
        pg = janc.grid_of(pc)
        ptm = janc.time_of(pc)
        Wp = torch.tensor(pc.W, dtype=torch.float64, device=dev)
        Up, Tp = pctx.init_state(pph, Wp)
        del Wp
        tp = torch.zeros(1, dtype=torch.float64, device=dev)
        pctx.step(pg, pph, ptm, Up, Tp, 2, tp)
        psteps = 10
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record()
        pctx.step(pg, pph, ptm, Up, Tp, psteps, tp)
        e1.record()
        torch.cuda.synchronize()
        ps = e0.elapsed_time(e1) / 1e3
        pctx.sync_status()
        ncell = pc.nx * pc.ny
        res = {"workload": f"uniform {pc.nx}x{pc.ny}, synthetic 9 species / 19 reactions, "
                           f"CFL {pc.cfl}", "steps": psteps, "ms_per_step": 1e3 * ps / psteps,
               "steps_per_s": psteps / ps, "cell_stage_per_s": ncell * 3 * psteps / ps,
               "paper_context": "A100, H2-O2 9 species / 19 reactions, 4000x1000: 5.0 step/s"}
        log(f"[bench] uniform {pc.nx}x{pc.ny} 9-species: {res['ms_per_step']:.3f} ms/step, "
            f"{res['steps_per_s']:.1f} step/s, {res['cell_stage_per_s']:.3e} cell-stage/s")
        pctx.close()
        return res
    paper_shape = optional("paper_shape", _paper_shape) if args.paper_shape else None

    def _cpu():
        cpu = None
        log(f"[bench] CPU oracle baseline ({args.cpu_steps} step)")
        cpu = cpu_baseline(case, args.cpu_steps)
        log(f"[bench] oracle {cpu['value']:.4e} cell-stage/s on {cpu['cores']} threads")
        return cpu
    cpu = None if args.no_cpu_baseline else optional("cpu", _cpu)

    out = {
        "metric": METRIC,
        "value": value,
        "unit": "cell-stage/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {
            "workload": "amr-9sp-3lev-1024x512-637blk",
            "levels": 3, "blocks": int(len(case.blocks)), "cells": int(cells),
            "ring_cells": ring_cells, "ring_fraction": ring_cells / cells,
            "mechanism": "synthetic 9 species / 19 reactions (seed 13750)",
            "advance": "synchronous, CFL 0.5", "parallelism": "single GPU",
        },
        "roofline": {
            "bound": "alu",
            "kernel": "stage_kernel (fused RK stage)",
            "achieved": achieved_tf,
            "peak": PEAK_FP64_VALU_TFLOPS,
            "unit": "TFLOP/s",
            "frac": achieved_tf / PEAK_FP64_VALU_TFLOPS,
            "traffic": measured_traffic(*choice),
            "traffic_unit": "bytes per launch (FETCH_SIZE x 2.0 + WRITE_SIZE x 1.0, copy-calibrated)",
            "flops_per_cell_stage": stage_flops(2, nU, True),
            "solved_cells_per_launch": solved,
            "avg_launch_ms": stage_avg,
            "hbm_algorithmic_GBs": achieved_gbs,
            "hbm_frac": achieved_gbs / PEAK_HBM_GBS,
            # max(t_HBM, t_VALU) / t_measured at the peaks: the bound that binds
            "binding": "fp64-valu" if achieved_tf / PEAK_FP64_VALU_TFLOPS >=
                       achieved_gbs / PEAK_HBM_GBS else "hbm",
            "binding_frac": max(achieved_tf / PEAK_FP64_VALU_TFLOPS, achieved_gbs / PEAK_HBM_GBS),
        },
        "kernels_ms": {"stage": stage_avg, "chemistry": float(np.mean(chem_ms)),
                       "restriction": float(np.mean(restr_ms)), "ring": float(np.mean(ring_ms)),
                       "chemistry_generic": chem_generic_ms},
        "chem_kernel": chem_kernel,
        "autotune": autotune,
        "per_block": per_block,
        "crossover": crossover,
        "regrid": regrid,
        "ensemble": ensemble,
        "adjoint": adjoint,
        **({"paper_shape": paper_shape} if paper_shape is not None else {}),
        "cpu_baseline": cpu,
        "context": "paper (A100, real H2-O2 mechanism, 2.76 M cells incl. invalid blocks): "
                   "0.18 s/step synchronous AMR, about 4.6e7 cell-stage/s; not the same "
                   "workload, so vs_baseline is null",
    }
    print(json.dumps(out), flush=True)
    plan.close()
    ctx.close()


if __name__ == "__main__":
    main()
