#!/usr/bin/env python3
"""Benchmark: Gamma v = F solves per second at 1M cells, relres 1e-8, on one GPU.

One step is one pass of the whole hot path over the 1M-cell workload with all
inputs already resident in HBM: collide -> assemble_gamma -> build_tree ->
factor_tree -> pcg_solve (tree preconditioner, FP64, relres 1e-8).  The
workload: jittered FCC ball of 1,000,000 spheres (nearest-neighbour spacing
1.9, jitter N(0, 0.05^2)), radii U[0.95, 1.05], forces N(0, 1), seed 0.

Prints ONE JSON line.  Besides the headline value it carries:
  roofline      the CG's product Gamma p (the largest kernel; by default
                k_spmv_tile, from the cells' positions and radii): algorithmic bytes per launch / its average
                launch time, measured with HIP events attached to sampled
                launches on the library's stream inside the timed region;
  cpu_baseline  the FP64 CPU oracle timed on this host's cores on a bounded
                sample of the same workload (setup + a fixed number of CG
                iterations, extrapolated to the GPU's iteration count);
  extra         the other workloads, each bounded to seconds of GPU time:
                block-Jacobi PCG, the solve stopped on the Gauss-Radau
                bound of the energy error, the whole step recorded once and
                replayed as one hipGraph, the local-MST forest (Z-order clusters
                of 512 to 2048 cells) and the augmented tree with its nested
                flexible CG on the same 1M system; the 1k-cell solve's
                latency with and without hipGraph replay; FP32-inner refinement
                against plain FP64 at 4M cells; 256 independent spheroids in
                one batched pipeline with autotuned knobs; the learned warm
                start over 200 time steps of a 200k-cell spheroid; the
                paper's own geometries (Hertz cells, Section 5.1) at 5e4
                cells without a preconditioner, with block Jacobi and with
                the tree (residual rule 1e-8, and the error bound at 1e-5).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, published

# HBM bytes per launch of the product (4 waves per workgroup) on the 1M-cell
# workload, per form, from two rocprofv3 counter runs of `--kernel-only spmv`:
# FETCH_SIZE x 2.0 + WRITE_SIZE x 1.0, the factors that make a 512 MiB copy
# read and write 512 MiB (summary and commands under profiles/).  Must be
# re-measured, or set to None, whenever that kernel changes.
SPMV_TRAFFIC_1M = {0: None, 1: None, 2: 140.1e6}
TILE_MIN_CELLS = 8192   # beyond it the library's edge form is the product from the cells


def product_form(knob: int, n: int) -> int:
    """Form of spmv_bytes that the library runs: its knob spmv_form (0 blocks,
    1 contacts), the latter from the cells (2) beyond TILE_MIN_CELLS cells."""
    return 2 if knob == 1 and n > TILE_MIN_CELLS else knob


def spmv_bytes(n: int, nnzb: int, form: int = 1, val_bytes: int = 48) -> int:
    """Algorithmic bytes of one product y = Gamma x as the library forms it.
    Blocks (form 0): every block's 6 distinct entries (the blocks are
    symmetric, 48 B in FP64) and its column index once.  Edge form (form 1):
    every off-diagonal entry's v = sqrt(w) u (24 B) and column once, every
    diagonal block's 6 entries once.  Both: the row pointers once, x once, y
    once.  From the cells (form 2): every entry's 16-bit number, every cell's
    position and radius, x and y once."""
    if form == 0:
        return nnzb * (val_bytes + 4) + 4 * (n + 1) + 24 * n + 24 * n
    ne = nnzb - n
    if form == 2:
        return ne * 2 + n * (32 + 24 + 24)
    return ne * (24 + 4) + n * 48 + 4 * (n + 1) + 24 * n + 24 * n


def cpu_baseline(c, gpu_iters: int, sample_iters: int = 10):
    """Oracle on this host: full setup at the full size, then `sample_iters` CG
    iterations; the solve time is extrapolated to the GPU's iteration count."""
    from oracle import oracle as O
    t0 = time.perf_counter()
    g = O.collide(c["pos"], c["radius"])
    A = O.assemble(g)
    t = O.build_tree(g)
    f = O.tree_factor(g, t)
    t1 = time.perf_counter()
    O.pcg(A, c["force"], "tree", f, fixed_iters=sample_iters)
    t2 = time.perf_counter()
    per_iter = (t2 - t1) / sample_iters
    est = (t1 - t0) + per_iter * gpu_iters
    import platform
    model = platform.processor() or ""
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"value": 1.0 / est, "unit": "solves/s", "cores": 1, "kind": "oracle",
            "host_cores_visible": os.cpu_count(), "host_cpu": model,
            "sample": f"1M-cell workload: collide+assemble+Prim+root+TreeLDLT in full ({t1 - t0:.1f} s) "
                      f"plus {sample_iters} tree-PCG iterations ({t2 - t1:.1f} s), "
                      f"extrapolated to {gpu_iters} iterations; single-threaded C, -O2",
            "setup_s": t1 - t0, "per_iter_s": per_iter}


def _sync_time(fn):
    import torch
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r = fn()
    torch.cuda.synchronize()
    return time.perf_counter() - t0, r


def extra_jacobi(ctx, A, M, F):
    """Block-Jacobi PCG against tree-PCG on the same 1M system (solve only)."""
    import torch
    MJ = ctx.make_jacobi(A)
    tj, (_, ij) = _sync_time(lambda: ctx.pcg_solve(A, MJ, F, torch.zeros_like(F), rtol=1e-8))
    tt, (_, it) = _sync_time(lambda: ctx.pcg_solve(A, M, F, torch.zeros_like(F), rtol=1e-8))
    return {"jacobi_pcg": {"iters": ij["iters"], "solve_ms": 1e3 * tj},
            "tree_pcg": {"iters": it["iters"], "solve_ms": 1e3 * tt}}


def extra_errstop(ctx, A, M, F):
    """Tree-PCG on the same 1M system stopped on the Gauss-Radau bound of the
    relative energy error (node mu = 1, Section 4's lambda_min(P^-1 Gamma) >= 1)
    at 1e-5 (the paper's tolerance) and 1e-8, beside the residual rule at the
    same tolerances (solve only)."""
    import torch
    out = {}
    for tol in (1e-5, 1e-8):
        for stop in ("residual", "error"):
            ctx.pcg_solve(A, M, F, torch.zeros_like(F), rtol=tol, stop=stop)
            t, (_, info) = _sync_time(lambda: ctx.pcg_solve(A, M, F, torch.zeros_like(F), rtol=tol, stop=stop))
            r = {"iters": info["iters"], "solve_ms": 1e3 * t, "relres_true": info["relres_true"]}
            if stop == "error":
                r["err_bound"] = info["err_bound"]
            out[f"{stop}_{tol:.0e}"] = r
    return out


def extra_graph_step(P, ctx, pos, R, F, v_eager, reps=10):
    """The same 1M step (collide -> assemble -> tree -> factor -> tree-PCG)
    recorded once and replayed as one hipGraph (sgp_step_*): every kernel
    runs again on the GPU, the host's mid-step readbacks are replayed from
    the recording and checked on the device.  Not the headline (which
    launches every kernel eagerly); the replayed velocity is compared bit
    for bit with the eager step's."""
    import numpy as np
    import torch
    n = pos.shape[0]
    S = P.Step(ctx)
    v = torch.zeros_like(F)
    t_rec, infos = _sync_time(lambda: S.record_batched([0, n], pos, R, F, v))
    times = []
    for _ in range(reps):
        t, (code, rinfos) = _sync_time(lambda: S.replay())
        times.append(t)
    ms = 1e3 * float(np.median(times))
    nv, nb = S.size()
    out = {"workload": f"jittered FCC ball, {n} spheres, seed 0; whole step recorded once, replayed {reps} times",
           "replay_ms_per_step": ms, "replay_solves_per_s": 1e3 / ms, "record_ms": 1e3 * t_rec,
           "recorded_values": nv, "recorded_bytes": nb, "iters": rinfos[0]["iters"],
           "v_equal_eager": bool(torch.equal(v, v_eager)),
           "v_max_diff_rel": float((v - v_eager).abs().max() / v_eager.abs().max())}
    del S
    return out


def extra_forest(ctx, g, A, F, pos, R, sizes=(512, 1024, 2048)):
    """The local-MST forest (Section 6, Discussion) on the same 1M system:
    Z-order clusters of K cells, each with its own maximum spanning forest,
    every sweep one launch.  Setup (forest + factor) and solve ms,
    iterations."""
    import torch
    out = {}
    for K in sizes:
        t_setup, (T, M) = _sync_time(lambda: (lambda T: (T, ctx.factor_tree(g, T)))(ctx.build_forest(g, pos, R, K)))
        ctx.pcg_solve(A, M, F, torch.zeros_like(F), rtol=1e-8)
        ts, (_, info) = _sync_time(lambda: ctx.pcg_solve(A, M, F, torch.zeros_like(F), rtol=1e-8))
        nt, n_roots, depth = T.size()
        out[f"K{K}"] = {"iters": info["iters"], "solve_ms": 1e3 * ts, "setup_ms": 1e3 * t_setup,
                        "clusters": ctx.tree_clusters(T, g.size()[0])[1], "trees": n_roots, "max_depth": depth,
                        "elim_steps": M.steps(), "us_per_iter": 1e3 * 1e3 * ts / max(info["iters"], 1)}
    return out


def extra_augmented(ctx, g, T, A, F):
    """Vaidya's augmented tree (Section 3.1) on the same 1M system with the
    paper's nested solve: flexible CG around tree-PCG on P' to relative
    residual 0.1 (Sections 3 and 5); t = ceil(n^(1/4)) pieces, and 64."""
    import torch
    out = {}
    for parts in (0, 64):
        t_setup, M = _sync_time(lambda: ctx.factor_augmented(g, T, parts=parts, inner_rtol=0.1))
        npc, nad, _, _ = ctx.prec_augmented(M, g.size()[0])
        ts, (_, info) = _sync_time(lambda: ctx.pcg_solve(A, M, F, torch.zeros_like(F), rtol=1e-8))
        out[f"parts{parts if parts else 'auto'}"] = {
            "pieces": npc, "added": nad, "outer_iters": info["iters"], "inner_iters": info["inner_iters"],
            "solve_ms": 1e3 * ts, "setup_ms": 1e3 * t_setup, "relres_true": info["relres_true"]}
    return out


def extra_small(P, dev, reps=30):
    """1000-cell workload (seed 0): latency of one solve and of the whole
    pipeline; the one-workgroup PCG (knob small_solve, the default) against
    the launch-per-kernel path, eager and with hipGraph replay of the CG
    chunks."""
    import numpy as np
    from workloads import sphere_cluster
    c = sphere_cluster(1000, 0)
    pos, R, F = dev(c["pos"]), dev(c["radius"]), dev(c["force"])
    ctx = P.Context()
    out = {"workload": "jittered FCC ball, 1000 spheres, seed 0"}
    for name, small, graph, ce in (("one_workgroup", 1, 0, 2), ("launches_graph0_check8", 0, 0, 8),
                                   ("launches_graph1_check8", 0, 1, 8)):
        ctx.tune("small_solve", small)
        ctx.tune("graph", graph)
        ctx.tune("check_every", ce)
        ts, tp, iters = [], [], 0
        for r in range(reps + 2):
            t_all, (A, M, ts_) = _sync_time(lambda: _pipeline(ctx, pos, R, F))
            if r >= 2:
                tp.append(t_all)
                ts.append(ts_[0])
                iters = ts_[1]
        out[name] = {"solve_us": 1e6 * float(np.median(ts)), "pipeline_us": 1e6 * float(np.median(tp)),
                     "iters": iters}
    ctx.close()
    return out


def _pipeline(ctx, pos, R, F, schedule="contract"):
    import torch
    g = ctx.collide(pos, R)
    A = ctx.assemble_gamma(g)
    M = ctx.factor_tree(g, ctx.build_tree(g), schedule=schedule)
    ts, (_, info) = _sync_time(lambda: ctx.pcg_solve(A, M, F, torch.zeros_like(F), rtol=1e-8))
    return A, M, (ts, info["iters"])


def extra_mixed(P, dev, n=4_000_000):
    """4M cells (seed 0): FP32 product and sweeps inside FP64 refinement against
    plain FP64 tree-PCG on the same system; both solutions are compared with the
    GPU's own FP64 solve to relres 1e-13 (`err_vs_gpu_fp64_1e-13`).  Their
    errors against the FP64 oracle's solution are measured by the 4M parity
    test, which runs the oracle's 4M solve (minutes of CPU)."""
    import torch
    from workloads import sphere_cluster
    c = sphere_cluster(n, 0)
    pos, R, F = dev(c["pos"]), dev(c["radius"]), dev(c["force"])
    del c
    ctx = P.Context()
    g = ctx.collide(pos, R)
    A = ctx.assemble_gamma(g)
    M = ctx.factor_tree(g, ctx.build_tree(g))
    ref, _ = ctx.pcg_solve(A, M, F, rtol=1e-13, max_iter=20000)
    out = {"workload": f"jittered FCC ball, {n} spheres, seed 0; solve only, relres 1e-8"}
    for name, kw in (("f64", {}), ("f32ir", {"precision": "f32ir", "inner_rtol": 1e-4})):
        ctx.pcg_solve(A, M, F, rtol=1e-8, **kw)   # warm-up (FP32 copies built once)
        ts = []
        for _ in range(3):
            t, (v, info) = _sync_time(lambda: ctx.pcg_solve(A, M, F, rtol=1e-8, **kw))
            ts.append(t)
        err = float(torch.linalg.vector_norm(v - ref) / torch.linalg.vector_norm(ref))
        out[name] = {"solve_ms": 1e3 * min(ts), "iters": info["iters"], "outer": info["outer_iters"],
                     "relres_true": info["relres_true"], "err_vs_gpu_fp64_1e-13": err}
    out["wall_ratio_f32ir_vs_f64"] = out["f32ir"]["solve_ms"] / out["f64"]["solve_ms"]
    out["iter_ratio_f32ir_vs_f64"] = out["f32ir"]["iters"] / out["f64"]["iters"]
    ctx.close()
    return out


def extra_batched(P, dev, n_inst=256, steps=3, log=None):
    """256 spheroids, sizes log-uniform in [1e3, 2e5], seeds 1..256: one batched
    pipeline (collide -> assemble -> tree -> factor -> PCG over all instances at
    once), knobs chosen by the autotuner on this batch; eager steps, and the
    same step recorded once and replayed as one hipGraph (sgp_step_*)."""
    import numpy as np
    import torch
    from paper_2410_04512_amd import autotune
    from workloads import batched_instance
    parts = [batched_instance(k + 1) for k in range(n_inst)]
    sizes = np.array([p["pos"].shape[0] for p in parts])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pos = dev(np.concatenate([p["pos"] for p in parts]))
    R = dev(np.concatenate([p["radius"] for p in parts]))
    F = dev(np.concatenate([p["force"] for p in parts]))
    del parts
    ctx = P.Context()
    g = ctx.collide_batched(off, pos, R)
    A = ctx.assemble_gamma(g)
    T = ctx.build_tree(g)
    tuned = autotune.tune(ctx, g, T, A, F, offsets=off, log=log)
    sched = tuned["schedule"]
    del g, A, T, tuned["prec"]

    def step():
        g = ctx.collide_batched(off, pos, R)
        A = ctx.assemble_gamma(g)
        M = ctx.factor_tree(g, ctx.build_tree(g), schedule=sched)
        ts, (v, infos) = _sync_time(lambda: ctx.pcg_solve_batched(A, M, off, F, rtol=1e-8))
        return ts, infos

    step()
    times, solve_t = [], []
    for _ in range(steps):
        t, (ts, infos) = _sync_time(step)
        times.append(t)
        solve_t.append(ts)
    it = np.array([i["iters"] for i in infos])
    rel = np.array([i["relres_true"] for i in infos])
    st = np.array([i["status"] for i in infos])
    ms = 1e3 * float(np.median(times))
    # the same step recorded once and replayed as one hipGraph (the tuned
    # knobs stay set on ctx and are copied into the step)
    S = P.Step(ctx)
    vs = torch.zeros_like(F)
    t_rec, _ = _sync_time(lambda: S.record_batched(off, pos, R, F, vs, schedule=sched))
    rtimes = []
    for _ in range(steps):
        t, (code, rinfos) = _sync_time(lambda: S.replay())
        rtimes.append(t)
    replay_ms = 1e3 * float(np.median(rtimes))
    rvalues, rbytes = S.size()
    del S
    return {"workload": f"{n_inst} spheroids, sizes log-uniform [1e3, 2e5] (sum {int(off[-1])} cells), seeds 1..{n_inst}",
            "solves_per_s": n_inst / (ms * 1e-3), "ms_per_step": ms, "solve_ms": 1e3 * float(np.median(solve_t)),
            "iters_min": int(it.min()), "iters_mean": float(it.mean()), "iters_max": int(it.max()),
            "max_relres_true": float(rel.max()), "all_converged": bool((st == 0).all()),
            "graph_step": {"replay_ms_per_step": replay_ms, "replay_solves_per_s": n_inst / (replay_ms * 1e-3),
                           "record_ms": 1e3 * t_rec, "recorded_values": rvalues, "recorded_bytes": rbytes,
                           "iters_equal_eager": [i["iters"] for i in rinfos] == [i["iters"] for i in infos]},
            "tuned": {k: v for k, v in tuned.items() if k not in ("prec", "table", "defaults")},
            "tune_table_ms": {k: 1e3 * v for k, v in tuned["table"].items()}}


def extra_learned(P, dev, log=None):
    """200k-cell spheroid (seed 0), 200 overdamped steps (dt 0.01, repulsion
    5 w n plus N(0, 0.1^2) active force); the network trains on steps 1-100 and
    warm-starts steps 101-200; iterations and wall time to relres 1e-8 against
    the previous-step and the zero start."""
    import torch
    from paper_2410_04512_amd import warmstart as W
    from workloads import sphere_cluster, dynamics_noise
    c = sphere_cluster(200_000, 0)
    ctx = P.Context()
    pos, R = dev(c["pos"]), dev(c["radius"])
    res = W.run(ctx, pos, R, dynamics_noise, n_steps=200, n_train=100, epochs=30, lr=3e-3, log=log)
    s = W.summary(res)
    s["workload"] = "200k-cell spheroid, seed 0, 200 steps; train 1-100, test 101-200"
    del res
    ctx.close()
    torch.cuda.synchronize()
    return s


# the paper's iteration reductions against unpreconditioned CG (Section 5.2;
# single-threaded CPU, true error 1e-5, n ~ 5e4, the authors' Hertz cells)
PAPER_RATIOS = {"hex": {"tree": 4.9, "jacobi": 1.2}, "hex_ill": {"tree": 9.2, "jacobi": 1.2},
                "random": {"tree": 3.8}, "dumbbell": {"tree": 8.5}}


def extra_paper(P, dev, n=50_000, reps=3):
    """The paper's own geometries (Section 5.1) at n = 5e4, generated here:
    HCP with N(0, (0.3 r)^2) noise (g_med 3e4 and 3e3), a random spheroidal
    packing and a dumbbell (g_med 3e4); Hertz contact areas, g_par = 2e6,
    g_perp = 8e7; F = Gamma x_true with a known x_true.  For each: CG without
    a preconditioner, with block Jacobi and with the tree, to relres 1e-8;
    iterations, solve ms (best of `reps`), setup ms of the preconditioner,
    the true error, the iterations to the paper's own stopping rule (true
    error 1e-5, by bisection over fixed-iteration solves; the error of CG
    iterates shrinks monotonically in the energy norm, not strictly in the
    2-norm, so this is the first such iteration up to that caveat), and the
    iteration and wall-time ratios beside the paper's iteration ratios."""
    import torch
    from workloads import paper as W
    ctx = P.Context()
    ctx.set_contact_model("hertz")
    out = {"workload": f"paper geometries (Section 5.1), {n} cells each, seed 0; relres 1e-8, x0 = 0",
           "paper_iteration_ratio_vs_none": PAPER_RATIOS}
    for kind in ("hex", "hex_ill", "random", "dumbbell"):
        c = W.paper_cells(kind, n, 0)
        gp, gq, gm = c["g_par"], c["g_perp"], c["g_med"]
        pos, R, xt = dev(c["pos"]), dev(c["radius"]), dev(c["x_true"])
        g = ctx.collide(pos, R)
        A = ctx.assemble_gamma(g, gp, gq, gm)
        F = ctx.spmv(A, xt)
        t_tree, (T, M) = _sync_time(lambda: (lambda T: (T, ctx.factor_tree(g, T, gp, gq, gm)))(ctx.build_tree(g)))
        t_jac, J = _sync_time(lambda: ctx.make_jacobi(A))
        nt, n_roots, depth = T.size()
        res = {"contacts": g.size()[1], "trees": n_roots, "tree_depth": depth, "g_med": gm}
        nx = torch.linalg.vector_norm(xt)

        def true_err(k, MM):
            v, _ = ctx.pcg_solve(A, MM, F, fixed_iters=k)
            return float(torch.linalg.vector_norm(v - xt) / nx)

        for name, MM, setup in (("none", None, 0.0), ("jacobi", J, t_jac), ("tree", M, t_tree)):
            ctx.pcg_solve(A, MM, F)
            ts = []
            for _ in range(reps):
                t, (v, info) = _sync_time(lambda: ctx.pcg_solve(A, MM, F))
                ts.append(t)
            err = float(torch.linalg.vector_norm(v - xt) / nx)
            # the paper's stopping rule: the first iteration whose true error
            # is <= 1e-5, found by bisection over fixed-iteration solves
            lo, hi = 0, info["iters"]
            if err <= 1e-5:
                while hi - lo > 1:
                    mid = (lo + hi) // 2
                    if true_err(mid, MM) <= 1e-5:
                        hi = mid
                    else:
                        lo = mid
            res[name] = {"iters": info["iters"], "solve_ms": 1e3 * min(ts), "setup_ms": 1e3 * setup,
                         "true_err": err, "relres_true": info["relres_true"],
                         "iters_true_err_1e-5": hi if err <= 1e-5 else None}
        for name in ("jacobi", "tree"):
            res[f"iter_ratio_none_over_{name}"] = res["none"]["iters"] / res[name]["iters"]
            if res[name]["iters_true_err_1e-5"] and res["none"]["iters_true_err_1e-5"]:
                res[f"true_err_iter_ratio_none_over_{name}"] = (res["none"]["iters_true_err_1e-5"] /
                                                                res[name]["iters_true_err_1e-5"])
        res["iter_ratio_jacobi_over_tree"] = res["jacobi"]["iters"] / res["tree"]["iters"]
        res["wall_ratio_jacobi_over_tree"] = ((res["jacobi"]["solve_ms"] + res["jacobi"]["setup_ms"]) /
                                              (res["tree"]["solve_ms"] + res["tree"]["setup_ms"]))
        # CG stopped on the Gauss-Radau bound of the relative energy error at
        # the paper's tolerance 1e-5 (node mu = 1 with the tree, g_med without
        # a preconditioner), checked against the known solution
        xg = float(torch.dot(xt.reshape(-1), F.reshape(-1)))
        for name, MM in (("none", None), ("tree", M)):
            ctx.pcg_solve(A, MM, F, rtol=1e-5, stop="error")
            ts = []
            for _ in range(reps):
                t, (v, info) = _sync_time(lambda: ctx.pcg_solve(A, MM, F, rtol=1e-5, stop="error"))
                ts.append(t)
            e = v - xt
            eg = float(torch.dot(e.reshape(-1), ctx.spmv(A, e).reshape(-1)))
            res[f"error_rule_{name}"] = {"iters": info["iters"], "solve_ms": 1e3 * min(ts),
                                         "err_bound": info["err_bound"], "true_energy_err": (eg / xg) ** 0.5,
                                         "true_err": float(torch.linalg.vector_norm(e) / nx)}
        res["error_rule_iter_ratio_none_over_tree"] = (res["error_rule_none"]["iters"] /
                                                       res["error_rule_tree"]["iters"])
        out[kind] = res
    ctx.close()
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--n", type=int, default=1_000_000)
    ap.add_argument("--schedule", default="contract", choices=["contract", "level"])
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extra", action="store_true")
    ap.add_argument("--extras", default="jacobi,errstop,graph1M,forest,augmented,small,mixed,batched,learned,paper",
                    help="comma list of extra workloads to run after the headline")
    ap.add_argument("--spmv-form", type=int, choices=[0, 1], default=None,
                    help="product form: 0 stored 3x3 blocks, 1 contacts' (w, u) (the library default)")
    ap.add_argument("--kernel-only", choices=["spmv"], default=None,
                    help="build the system once, then run only the named kernel (for counter runs)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "the benchmark runs on one GPU only (a single solve is not sharded "
                                   "across GPUs); use --gpus 1"}))
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2410_04512_amd as P
    from workloads import sphere_cluster

    torch.cuda.set_device(0)
    c = sphere_cluster(args.n, 0)
    dev = lambda a: torch.as_tensor(a).to("cuda")  # noqa: E731
    pos, R, F = dev(c["pos"]), dev(c["radius"]), dev(c["force"])
    ctx = P.Context()
    if args.spmv_form is not None:
        ctx.tune("spmv_form", args.spmv_form)
    g, A, T, M = P.Graph(ctx), P.Bsr(ctx), P.Tree(ctx), P.Prec(ctx)
    v = torch.zeros_like(F)
    info = {}

    def step():
        nonlocal info
        ctx.collide(pos, R, 32, g)
        ctx.assemble_gamma(g, 1.0, 0.1, 1e-3, A)
        ctx.build_tree(g, T)
        ctx.factor_tree(g, T, 1.0, 0.1, 1e-3, args.schedule, M)
        _, info = ctx.pcg_solve(A, M, F, v, rtol=1e-8)

    if args.kernel_only == "spmv":
        # counter-run mode: a plain copy of known size (calibrates FETCH_SIZE /
        # WRITE_SIZE), then the block-CSR product alone, 20 times
        ctx.collide(pos, R, 32, g)
        ctx.assemble_gamma(g, 1.0, 0.1, 1e-3, A)
        n, _ = g.size()
        _, nnzb = A.size()
        src = torch.ones(64 * 1024 * 1024, dtype=torch.float64, device="cuda")   # 512 MiB
        dst = torch.empty_like(src)
        dst.copy_(src)
        x = torch.ones_like(F)
        y = torch.empty_like(F)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(20):
            ctx.spmv(A, x, y)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / 20
        print(json.dumps({"kernel": ("k_spmv_tile" if n > TILE_MIN_CELLS else "k_spmv_edge")
                          if ctx.tune_get("spmv_form") else "k_spmv_sym",
                          "copy_bytes": 2 * src.numel() * 8, "api_call_avg_ms": ms,
                          "bytes_per_launch": spmv_bytes(n, nnzb, product_form(ctx.tune_get("spmv_form"), n)),
                          "note": "api_call_avg_ms includes the two permutations of sgp_spmv; the kernel alone is in the trace"}), flush=True)
        ctx.close()
        return

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    ctx.kernel_timing(True)
    phase = {k: 0.0 for k in ("collide", "assemble", "build_tree", "factor", "solve")}
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
        for k, val in ctx.phase_times().items():
            phase[k] += val
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    spmv_ms, spmv_launches = ctx.kernel_stats()
    ctx.kernel_timing(False)
    elapsed = t1 - t0
    ms_per_step = 1e3 * elapsed / args.steps
    n, m = g.size()
    _, nnzb = A.size()
    nt, n_roots, max_depth = T.size()
    avg_spmv_ms = spmv_ms / max(spmv_launches, 1)
    form = product_form(ctx.tune_get("spmv_form"), n)
    bytes_spmv = spmv_bytes(n, nnzb, form)
    achieved = bytes_spmv / (avg_spmv_ms * 1e-3) / 1e9
    out = {
        "metric": "Gamma v=F solves/s @1M cells, relres 1e-8 (tree-PCG, FP64)",
        "value": args.steps / elapsed,
        "unit": "solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": f"jittered FCC ball, {n} spheres, seed 0; step = collide+assemble+tree+factor+tree-PCG",
                   "n_cells": n, "contacts": m, "nnzb": nnzb, "tree_depth": max_depth, "trees": n_roots,
                   "schedule": args.schedule, "elim_steps": M.steps(), "cg_iters": info.get("iters"),
                   "relres_true": info.get("relres_true")},
        "roofline": {"bound": "hbm",
                     "kernel": ("k_spmv_sym (block-CSR product, in CG)",
                                "k_spmv_edge (Gamma p from contacts, in CG)",
                                "k_spmv_tile (Gamma p from the cells, in CG)")[form],
                     "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS,
                     "traffic": SPMV_TRAFFIC_1M[form] if (args.n == 1_000_000 and ctx.tune_get("spmv_waves") == 4) else None,
                     "traffic_unit": "B/launch (counters)",
                     "bytes_per_launch": bytes_spmv, "avg_launch_ms": avg_spmv_ms,
                     "launches": spmv_launches,
                     "timed": "HIP start/stop events carried by the launch itself (hipExtLaunchKernel) of one "
                              "product in every 4 CG iterations (the third of a "
                              f"{ctx.tune_get('check_every')}-iteration chunk, or its last) in the timed region "
                              "(products after convergence excluded)"},
        "phase_ms": {k: v_ / args.steps for k, v_ in phase.items()},
    }
    if not args.no_extra:
        ex = {}
        wanted = [e for e in args.extras.split(",") if e]
        log = lambda m: print(m, file=sys.stderr, flush=True)  # noqa: E731
        for name in wanted:
            log(f"extra: {name}")
            t_x = time.perf_counter()
            if name == "jacobi":
                ex.update(extra_jacobi(ctx, A, M, F))
            elif name == "errstop":
                ex["error_rule_1M"] = extra_errstop(ctx, A, M, F)
            elif name == "graph1M":
                ex["graph_step_1M"] = extra_graph_step(P, ctx, pos, R, F, v)
            elif name == "forest":
                ex["forest_1M"] = extra_forest(ctx, g, A, F, pos, R)
            elif name == "augmented":
                ex["augmented_1M"] = extra_augmented(ctx, g, T, A, F)
            elif name == "small":
                ex["small_1k"] = extra_small(P, dev)
            elif name == "mixed":
                ex["mixed_4M"] = extra_mixed(P, dev)
            elif name == "batched":
                ex["batched_256"] = extra_batched(P, dev, log=log)
            elif name == "learned":
                ex["learned_200k"] = extra_learned(P, dev, log=log)
            elif name == "paper":
                ex["paper_5e4"] = extra_paper(P, dev)
            else:
                raise SystemExit(f"unknown extra '{name}'")
            log(f"extra: {name} done in {time.perf_counter() - t_x:.1f} s")
        out["extra"] = ex
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(c, int(info.get("iters") or 170))
    ctx.close()
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
