#!/usr/bin/env python3
"""Throughput of the PDHG iteration on one MI355X.

Workload: RGB transport at 256 x 256 x 3 colours x 32 time steps (Neumann x,
y, t; periodic colour), seeded smooth random densities (Gaussian-filtered
uniform noise, sigma 4 px, exponentiated, normalised).  A step is one full
iteration of Algorithm 1 (projection, prox, dual steps) in the library's
default projection mode (the carried potential: one transform solve).

Prints one JSON line: cell-iters/s (cells = X Y C P centred nodes), the
per-phase split measured with HIP events on the solver's stream in a
separate profiled run, the HBM roofline of the dominant kernel timed with HIP
events around its launches inside the timed region, and the FP64 CPU oracle
timed on a bounded sample of the same workload.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E
FP32_PEAK_TFLOPS = 157.3       # MI355X FP32 vector

# FP32 words per centred node and launch.
# METHOD_WORDS is the method's byte model (each element of the method's own
# arrays read or written once, the phases fused as far as the data
# dependences allow): a1+a2 (adjoint averages and divergence) 13, each
# transform pass 2, a4..a7 (update, prox, dual steps) 21; the iteration
# moves 44 words, 64 with a refinement solve (which adds a residual pass of
# 6 and a second solve of 10 and makes the update read one more word).
# KERNEL_WORDS adds what this implementation's kernels move on top, per
# projection mode (refine = 0 off, 1 refinement solve, 3 carried potential):
#   div     read x (4) + b_bar (4) (+ Phi 1), write a (4) + r (1)
#   update  read a (4) + phi (1, 2 when refined) + b (4) (+ Phi 1), write
#           x (4) + b (4) + b_bar (4) (+ Phi 1)
# Mode 3 runs the refinement solve too in the first carry_refine iterations
# after initialisation; the benchmark warms up past them, so the timed
# iterations are the steady ones.
METHOD_WORDS = {"div": 13, "xform_x": 2, "xform_y": 2, "tc": 2, "refine": 6, "update": 21}
METHOD_ITERATION_WORDS = 44
KERNEL_WORDS = {
    "div": {0: 13, 1: 13, 3: 14},
    "xform_x": 2, "xform_y": 2, "tc": 2,
    "refine": 6,
    "update": {0: 21, 1: 22, 3: 23},
}


def nt_store(N):
    """Whether the stencil kernels store the iteration's fields non-temporally:
    one problem's field of N values is 16 MB or more (the library's rule)."""
    return 4 * N >= 16 << 20


def kernel_name(phase, mode, C, X=0, xfold=False, xkind=0, fused=False, nt=False, dense=False):
    """Full name of the kernel a steady-state iteration launches for `phase`
    (row stencils and power-of-two transforms).  With xfold the divergence
    kernel also does the forward x transform (DCT-II, xkind 0, or Hartley, 2)
    of its rows of length X; with fused the Poisson solve is the three-pass
    one (x pass into a transposed scratch, the y and time pass, the inverse x
    pass with the colour transform), with dense that of the matrix products;
    nt: the stencil kernels' non-temporal variant (nt_store).  Rows of 128 or 256 nodes take the vector stencil
    kernels (one wavefront per row, X / 64 nodes per lane), the divergence
    without the folded x transform."""
    f = "true" if nt else "false"
    vec = X in (128, 256)
    if phase == "div":
        m = {0: 0, 1: 0, 3: 2}[mode]
        if vec and not xfold:
            return f"k_div_vec<{m}, {C}, {f}, {X // 64}>"
        return f"k_div_rows<{m}, {C}, {X if xfold else 0}, {xkind if xfold else 0}, {f}>"
    if phase == "update":
        nphi = {0: 1, 1: 2, 3: 3}[mode]
        if vec:
            return f"k_update_vec<{nphi}, {C}, {f}, {X // 64}>"
        return f"k_update_rows<0, {nphi}, {C}, {f}>"
    if phase == "refine":
        return f"k_div_vec<1, {C}, {f}, {X // 64}>" if vec and not xfold else f"k_div_rows<1, {C}>"
    if fused and dense:
        return {"xform_x": "k_dx", "tc": "k_dyt"}[phase]
    if fused:
        return {"xform_x": "k_xf_tr + k_xi_tr", "tc": "k_yt"}[phase]
    return {"xform_x": "k_rows_fft", "xform_y": "k_cols_fft", "tc": "k_tc_reg"}[phase]


def per_mode(table, name, mode):
    v = table[name]
    return v if not isinstance(v, dict) else v[mode]


# sources outside the solver's kernels: their changes leave the solver's
# counters valid
NOT_SOLVER_SOURCES = {"hue.hip"}


def kernel_sources_hash() -> str:
    """Hash of the solver's kernel sources (the counter summary records it)."""
    h = hashlib.sha256()
    for f in sorted(os.listdir(os.path.join(ROOT, "paper_1501_04840_amd", "csrc"))):
        if f in NOT_SOLVER_SOURCES:
            continue
        with open(os.path.join(ROOT, "paper_1501_04840_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(prefix: str, summary: str = "traffic.json", sources=None):
    """HBM bytes per launch (FETCH_SIZE + WRITE_SIZE, calibrated) of the
    kernels whose names start with `prefix`, from a committed counter
    summary, if it was taken on the current kernel sources."""
    path = os.path.join(ROOT, "profiles", summary)
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        t = json.load(fh)
    if t.get("sources") != (sources or kernel_sources_hash()):
        return None
    vals = [v["bytes_per_launch"] for k, v in t.get("kernels", {}).items()
            if k == prefix or k.startswith(prefix + "<")]
    return sum(vals) / len(vals) if vals else None


def host_cpu() -> str:
    """CPU model and the cores this process may run on (the oracle uses one)."""
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return f"{model}, {len(os.sched_getaffinity(0))} cores available"


def one_thread():
    """Context that holds NumPy/SciPy's thread pools to one thread, so that the
    oracle's timing uses exactly the one core it reports."""
    from threadpoolctl import threadpool_limits
    return threadpool_limits(limits=1)


def cpu_baseline(f0, f1, X, Y, C, P, iters):
    import numpy as np
    from oracle import grid as G, pdhg
    g = G.Grid(X, Y, C, P)
    a0, a1 = f0.astype(np.float64), f1.astype(np.float64)
    with one_thread():
        t0 = time.perf_counter()
        pdhg.solve(g, a0, a1, 10.0, 0.099, iters)
        dt = time.perf_counter() - t0
    return {
        "value": X * Y * C * P * iters / dt, "unit": "cell-iters/s", "cores": 1,
        "kind": "oracle", "host": host_cpu(),
        "sample": f"{iters} iterations of the {X}x{Y}x{C}x{P} workload, FP64 NumPy/SciPy oracle "
                  f"(single-threaded), {dt:.1f} s",
    }


def copy_ceiling(nbytes: int = 1 << 30, reps: int = 10) -> float:
    """Device-to-device copy rate (read + write bytes / s) of a 1 GiB buffer
    by torch's copy kernel (4-byte lanes), for context: kernels with 16-byte
    lanes and non-temporal stores move more on this GPU."""
    import torch
    src = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda:0").uniform_()
    dst = torch.empty_like(src)
    dst.copy_(src)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(reps):
        dst.copy_(src)
    b.record()
    b.synchronize()
    gbs = 2.0 * nbytes * reps / (a.elapsed_time(b) * 1e-3) / 1e9
    del src, dst
    return gbs


def hue_batch(args):
    """Batched 1D periodic hue transport: 1024 problems of uneven sizes solved
    to the certified tolerance as one batch (graph of shape groups), against
    the plain cold-started solver looped over a sample of the same problems."""
    import numpy as np
    import torch
    from paper_1501_04840_amd import otdyn
    from synth import inputs

    def say(msg):
        print(msg, file=sys.stderr, flush=True)

    os.environ.setdefault("OT_DYN_VERBOSE", "1")
    probs = inputs.cfg4_problems(args.hue_count)
    dims = [(n, 1, 1, T) for n, T, _, _ in probs]
    cells = sum(n * T for n, T, _, _ in probs)
    base = otdyn.ot_dyn_default_desc(1, 1, 1, 2)
    base.bc[0] = otdyn.OT_BC_PERIODIC
    base.tau, base.sigma = args.hue_tau, args.hue_sigma
    base.adapt = args.hue_adapt
    bt = otdyn.Batch(base, dims, "cuda:0")
    bt.set_boundary([p[2].reshape(1, 1, -1) for p in probs], [p[3].reshape(1, 1, -1) for p in probs])
    say(f"hue batch: {len(probs)} problems, {cells} cells; autotuning")
    t0 = time.perf_counter()
    bt.autotune(10)
    t_tune = time.perf_counter() - t0
    tuned = {}
    for i, (n, T, _, _) in enumerate(probs):
        if f"{n}x{T}" not in tuned:
            bx, dense = otdyn.ot_dyn_batch_tuning(bt.bt, i)
            tuned[f"{n}x{T}"] = {"row_bx": bx, "dense_xy": dense}
    say(f"hue batch: autotune {t_tune:.2f} s ({tuned}); solving")
    t0 = time.perf_counter()
    status, rep = bt.solve(args.hue_max_iters, chunk=args.hue_chunk)
    t_batch = time.perf_counter() - t0
    its = np.array([bt.problem(i).iterations for i in range(len(probs))])
    open_probs = []
    for i in range(len(probs)):
        r = bt.problem(i)
        if not r.converged:
            open_probs.append({"i": i, "n": probs[i][0], "T": probs[i][1],
                               "r_prim": r.r_prim, "r_dual": r.r_dual, "r_div": r.r_div})
    say(f"hue batch: {t_batch:.2f} s, {rep.converged} certified; looped sample next")
    bt.close()
    # plain solver, one problem at a time, on an evenly spaced sample
    idx = np.linspace(0, len(probs) - 1, args.hue_loop_sample).astype(int)
    t_loop, loop_conv = 0.0, 0
    for i in idx:
        n, T, h0, h1 = probs[i]
        d = otdyn.ot_dyn_default_desc(n, 1, 1, T)
        d.bc[0] = otdyn.OT_BC_PERIODIC
        d.tau, d.sigma = args.hue_tau, args.hue_sigma
        d.adapt = args.hue_adapt
        d.check_every = args.hue_chunk
        pr = otdyn.Problem(d, "cuda:0")
        pr.set_boundary(torch.from_numpy(h0.reshape(1, 1, n)), torch.from_numpy(h1.reshape(1, 1, n)))
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        pr.init()
        st, r = pr.solve(args.hue_max_iters)
        t_loop += time.perf_counter() - t1
        loop_conv += int(st == otdyn.OT_OK)
        say(f"looped problem {i} (n={n}, T={T}): {r.iterations} iterations, status {st}")
        pr.close()
    per_problem = t_loop / len(idx)
    cpu = None
    if not args.no_cpu:
        cpu = hue_cpu_baseline(probs, idx, args)
    out = {
        "metric": "time-to-tolerance of 1024 batched hue problems",
        "value": t_batch, "unit": "s", "higher_is_better": False,
        "n_gpus": 1, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"hue_batch_{len(probs)}", "bins": list(inputs.HUE_BINS),
                   "tau": args.hue_tau, "sigma": args.hue_sigma, "adapt": args.hue_adapt,
                   "steps": list(inputs.HUE_STEPS), "cells": cells,
                   "chunk": args.hue_chunk, "max_iters": args.hue_max_iters,
                   "certified": int(rep.converged), "iters_max": int(its.max()),
                   "iters_median": float(np.median(its)), "autotune_s": t_tune,
                   "tuning": tuned,
                   "cell_iters_per_s": float(cells * its.mean() / t_batch),
                   "uncertified": open_probs},
        "looped_plain_solver": {"sample": len(idx), "certified": loop_conv,
                                "s_per_problem": per_problem,
                                "extrapolated_s": per_problem * len(probs),
                                "batch_speedup": per_problem * len(probs) / t_batch},
    }
    if cpu:
        out["cpu_baseline"] = cpu
    return out


def hue_cpu_baseline(probs, idx, args, iters: int = 600):
    """The FP64 oracle on the looped sample of hue problems, a fixed number
    of iterations each (fixed step sizes, as in Algorithm 1)."""
    import numpy as np
    from oracle import grid as G, pdhg
    cells, dt = 0, 0.0
    for i in idx:
        n, T, h0, h1 = probs[i]
        g = G.Grid(n, 1, 1, T, (G.PERIODIC, G.NEUMANN, G.NEUMANN))
        with one_thread():
            t0 = time.perf_counter()
            pdhg.solve(g, h0.reshape(1, 1, -1).astype(np.float64),
                       h1.reshape(1, 1, -1).astype(np.float64), args.hue_tau, args.hue_sigma, iters)
            dt += time.perf_counter() - t0
        cells += n * T * iters
    return {"value": cells / dt, "unit": "cell-iters/s", "cores": 1, "kind": "oracle",
            "host": host_cpu(),
            "sample": f"{iters} iterations of each of {len(idx)} hue problems "
                      f"(the looped sample), FP64 NumPy/SciPy oracle (single-threaded), {dt:.1f} s"}


def warm_start(args):
    """Learned warm start on 64 x 64 x 3 x 16 problems: certified
    time-to-tolerance of held-out pairs from a cold start and from the
    committed trained network (coarse solve, network correction, fine
    solve; all of it inside the timed wall time)."""
    import torch
    from paper_1501_04840_amd import otnet
    from paper_1501_04840_amd import warmstart as W

    net = otnet.Net(W.net_desc(32), "cuda:0")
    net.set_params(torch.from_numpy(W.load_weights()))
    pairs = W.pairs_of(range(args.warm_count), held_out=True)
    res = W.evaluate(pairs, ("cold", "warm"), net, max_iters=args.warm_max_iters,
                     group=min(128, args.warm_count))
    net.close()
    summ = {m: {k: v for k, v in res[m].items() if k != "iterations"} for m in ("cold", "warm")}
    out = {
        "metric": "time-to-tolerance (r < 1e-6) of held-out 64x64x3x16 pairs, warm start vs cold",
        "value": res["warm"]["wall_s"], "unit": "s", "higher_is_better": False,
        "n_gpus": 1, "dtype": "f32 solver, bf16 network", "data": "synthetic",
        "config": {"workload": f"warm_64x64x3x16_{args.warm_count}", "pairs": args.warm_count,
                   "cold": summ["cold"], "warm": summ["warm"],
                   "prediction_rel_error": res.get("prediction_rel_error"),
                   "iterations_saved_mean": summ["cold"]["iterations_mean"] - summ["warm"]["iterations_mean"]},
        "vs_cold": res["cold"]["wall_s"] / res["warm"]["wall_s"],
    }
    print(json.dumps(out))


def hue_render(args):
    """Frames/s of the rendering stage of Sec. 5: an 8-bit RGB image whose hue
    histogram is specified to the densities of a transport path, all of its
    time levels per call (exact circular specification, saturation and value
    kept).  The source's hues, order and ranks are prepared once (timed
    apart); a call is one plan kernel (target counts and shift, a block per
    frame) and one pass over the pixels of every frame."""
    import numpy as np
    import torch
    from paper_1501_04840_amd import othue
    from oracle import hue as ref_hue
    from synth import inputs

    H, W = args.hue_image
    n = args.hue_bins
    F = args.hue_frames
    N = H * W
    img = inputs.hue_image(501, H, W, sigma=24.0)
    dens = np.stack([inputs.von_mises_hist(600 + i, n) for i in range(F)]).astype(np.float32)
    r = othue.HueRenderer(N, n)
    src = torch.from_numpy(img.reshape(-1).copy()).cuda()
    tg = torch.from_numpy(dens).cuda()
    out = torch.empty(F, N, 3, dtype=torch.uint8, device="cuda")
    r.set_source(src)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r.set_source(src)
    torch.cuda.synchronize()
    source_s = time.perf_counter() - t0
    for i in range(args.warmup):
        othue.ot_hue_render(r.h, tg, F, out)
    torch.cuda.synchronize()
    K = args.steps
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(K)]
    t0 = time.perf_counter()
    for k in range(K):
        othue.ot_hue_plan(r.h, tg, F)
        ev[k][0].record()
        othue.ot_hue_apply(r.h, out)
        ev[k][1].record()
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    apply_us = 1e3 * sum(a.elapsed_time(b) for a, b in ev) / K
    r.close()
    # read channels (2) + hue (4) + rank (4) once per four frames, write RGB (3)
    nbytes = N * (10.0 * ((F + 3) // 4) + 3.0 * F)
    from paper_1501_04840_amd import profile_traffic
    traffic = None
    if (H, W, n, F) == (2160, 3840, 360, 33):      # the counted workload
        traffic = measured_traffic("k_hue_render<true, 9, 4>", "traffic_hue.json",
                                   profile_traffic.hue_sources_hash())
    achieved = nbytes / (apply_us * 1e-6) / 1e9
    out_json = {
        "metric": f"frames/s, hue rendering {W}x{H}, {n} bins, {F} frames per call",
        "value": K * F / dt, "unit": "frames/s",
        "n_gpus": 1, "steps": K, "warmup": args.warmup, "ms_per_step": 1e3 * dt / K,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "u8 image, f32 hue", "data": "synthetic",
        "config": {"workload": f"hue_render_{W}x{H}_{n}", "pixels": N, "bins": n,
                   "frames_per_step": F, "targets": "von Mises mixtures",
                   "source_prep_s": source_s},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "limited_by": "vector instructions and LDS reads of the bin search",
                     "kernel": "k_hue_render", "algorithmic_bytes_per_launch": nbytes,
                     "avg_launch_us": apply_us, "launches": K},
    }
    if not args.no_cpu:
        sample = 8
        src_ref = ref_hue.Source(img, n)
        with one_thread():
            t0 = time.perf_counter()
            for i in range(sample):
                src_ref.render(dens[i % F])
            cpu_dt = time.perf_counter() - t0
        out_json["cpu_baseline"] = {"value": sample / cpu_dt, "unit": "frames/s", "cores": 1,
                                    "kind": "oracle", "host": host_cpu(),
                                    "sample": f"{sample} frames of the same {W}x{H} image "
                                              "(source preparation not timed)"}
    return out_json


def side_workloads(args) -> dict:
    """Short runs of the two other GPU workloads after the main line's timed
    region (default parameters otherwise): the 1024 batched hue problems to
    the certified tolerance (one looped problem for the looped rate) and 20
    calls of the 4K hue rendering.  Only their GPU figures, no CPU oracle."""
    import argparse as _ap
    hb = hue_batch(_ap.Namespace(**{**vars(args), "hue_loop_sample": 1, "no_cpu": True}))
    hr = hue_render(_ap.Namespace(**{**vars(args), "steps": 20, "warmup": 3, "no_cpu": True}))
    c = hb["config"]
    return {
        "hue_batch": {"metric": hb["metric"], "value": hb["value"], "unit": hb["unit"],
                      "certified": c["certified"], "count": args.hue_count,
                      "iters_median": c["iters_median"], "iters_max": c["iters_max"],
                      "cell_iters_per_s": c["cell_iters_per_s"], "autotune_s": c["autotune_s"],
                      "looped_s_per_problem": hb["looped_plain_solver"]["s_per_problem"],
                      "looped_sample": hb["looped_plain_solver"]["sample"]},
        "hue_render": {"metric": hr["metric"], "value": hr["value"], "unit": hr["unit"],
                       "ms_per_call": hr["ms_per_step"], "source_prep_s": hr["config"]["source_prep_s"],
                       "roofline": hr["roofline"]},
    }


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--workload", default="rgb", choices=["rgb", "hue_batch", "warm", "hue_render"])
    ap.add_argument("--warm-count", type=int, default=512)
    ap.add_argument("--warm-max-iters", type=int, default=30000)
    ap.add_argument("--hue-count", type=int, default=1024)
    ap.add_argument("--hue-max-iters", type=int, default=60000)
    ap.add_argument("--hue-chunk", type=int, default=200)
    ap.add_argument("--hue-loop-sample", type=int, default=8)
    ap.add_argument("--hue-tau", type=float, default=3.0)
    ap.add_argument("--hue-sigma", type=float, default=0.33)
    ap.add_argument("--hue-adapt", type=int, default=1, choices=[0, 1],
                    help="per-problem step balancing (both the batch and the looped solver)")
    ap.add_argument("--hue-image", type=int, nargs=2, default=[2160, 3840],
                    help="hue_render: image height and width")
    ap.add_argument("--hue-bins", type=int, default=360)
    ap.add_argument("--hue-frames", type=int, default=33,
                    help="hue_render: frames per call (time levels of a 32-step path)")
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=300)
    ap.add_argument("--warmup", type=int, default=64)
    ap.add_argument("--prox", default="newton", choices=["newton", "closed"],
                    help="root of the prox cubic: Newton steps or the closed form (Cardano)")
    ap.add_argument("--refine", type=int, default=None, choices=[0, 1, 3],
                    help="projection mode (default: the library default)")
    ap.add_argument("--size", type=int, nargs=4, default=[256, 256, 3, 32],
                    metavar=("X", "Y", "C", "P"))
    ap.add_argument("--cpu-iters", type=int, default=20)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-side", action="store_true",
                    help="rgb: skip the short hue batch and hue rendering runs after the timed region")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (got --gpus {args.gpus}); the solver has no "
              "multi-GPU path in this build", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_1501_04840_amd import otdyn
    from synth import inputs

    if not os.path.exists(otdyn.LIB_PATH):
        from paper_1501_04840_amd import build
        build.build()
    if args.workload == "hue_batch":
        print(json.dumps(hue_batch(args)))
        return
    if args.workload == "warm":
        warm_start(args)
        return
    if args.workload == "hue_render":
        print(json.dumps(hue_render(args)))
        return
    X, Y, C, P = args.size
    if (X, Y) == (256, 256):
        f0, f1 = inputs.cfg3_pair()
    else:
        f0, f1 = inputs.cfg3_pair(X, Y)
    N = X * Y * C * P
    d = otdyn.ot_dyn_default_desc(X, Y, C, P)
    if args.refine is not None:
        d.refine = args.refine
    d.prox = {"newton": 0, "closed": 1}[args.prox]
    mode = d.refine
    prob = otdyn.Problem(d, "cuda:0")
    prob.set_boundary(torch.from_numpy(f0), torch.from_numpy(f1))
    prob.init(otdyn.OT_INIT_COLD)
    # the carried-potential mode refines its first carry_refine iterations:
    # warm up past them so that the phase split and the timed region see the
    # steady-state launch sequence, whatever --warmup asks for
    warmup = max(args.warmup, d.carry_refine) if mode == otdyn.OT_REFINE_CARRY else args.warmup
    prob.step(warmup)
    torch.cuda.synchronize()

    # phase split: every phase bracketed by HIP events on the solver stream,
    # over a separate run of steps (events between all launches slow the
    # iteration down, so this run is not the timed one)
    n_split = min(args.steps, 100)
    otdyn.ot_dyn_profile(prob.plan, (1 << otdyn.OT_PHASE_COUNT) - 1)
    prob.step(n_split)
    phases = otdyn.ot_dyn_profile_read(prob.plan)
    split = {}
    iter_words = 0.0
    # one x pass per iteration: the forward one is folded into the divergence
    # kernel; no y pass: the three-pass solve (y and time in one pass)
    xfold = phases["xform_x"][1] == n_split
    fused = Y > 1 and phases["xform_y"][1] == 0
    # that of the register transforms takes power-of-two sides and times only
    pow2 = (32, 64, 128, 256)
    dense = not (X in pow2 and Y in pow2 and P in (8, 16, 32) and C in (1, 3))
    for name, (ms, n) in phases.items():
        if n == 0:
            continue
        kw = per_mode(KERNEL_WORDS, name, mode)
        mw = METHOD_WORDS[name]
        iter_words += kw * n / n_split
        split[name] = {"ms_per_iter": ms / n_split, "launches": n, "avg_launch_us": 1e3 * ms / n,
                       "kernel": kernel_name(name, mode, C, X, xfold, fused=fused, nt=nt_store(N),
                                             dense=dense),
                       "method_words_per_launch": mw, "kernel_words_per_launch": kw,
                       "algorithmic_GBs": mw * 4.0 * N * n / (ms * 1e-3) / 1e9,
                       "kernel_GBs": kw * 4.0 * N * n / (ms * 1e-3) / 1e9}
    assert "refine" not in split or mode != otdyn.OT_REFINE_CARRY, "timed past the refined start"
    dom = max(split, key=lambda k: split[k]["ms_per_iter"])

    # timed region: K steps with HIP events around the dominant kernel only
    otdyn.ot_dyn_profile(prob.plan, 1 << otdyn.PHASE_NAMES.index(dom))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    prob.step(args.steps)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    live = otdyn.ot_dyn_profile_read(prob.plan)[dom]
    otdyn.ot_dyn_profile(prob.plan, 0)
    _, rep = prob.residuals()
    prob.close()
    copy_gbs = copy_ceiling()

    K = args.steps
    per_launch_bytes = split[dom]["method_words_per_launch"] * 4.0 * N
    kernel_bytes = split[dom]["kernel_words_per_launch"] * 4.0 * N
    dom_us = 1e3 * live[0] / live[1]
    achieved = per_launch_bytes / (dom_us * 1e-6) / 1e9
    kname = split[dom]["kernel"]
    roof = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS, "traffic": measured_traffic(kname),
            "kernel": kname, "algorithmic_bytes_per_launch": per_launch_bytes,
            "method_words_per_node": split[dom]["method_words_per_launch"],
            "kernel_words_per_node": split[dom]["kernel_words_per_launch"],
            "kernel_bytes_per_launch": kernel_bytes,
            "kernel_GBs": kernel_bytes / (dom_us * 1e-6) / 1e9,
            "avg_launch_us": dom_us, "launches": live[1]}
    iter_bytes = iter_words * 4.0 * N
    method_iter_bytes = METHOD_ITERATION_WORDS * 4.0 * N
    out = {
        "metric": f"cell-iters/s at {X}x{Y}x{C}x{P}",
        "value": N * K / dt,
        "unit": "cell-iters/s",
        "n_gpus": 1, "steps": K, "warmup": warmup,
        "ms_per_step": 1e3 * dt / K,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {
            "workload": f"rgb_{X}x{Y}x{C}x{P}", "X": X, "Y": Y, "C": C, "P": P,
            "bc": "neumann x,y,t; periodic colour", "refine": mode, "prox": args.prox,
            "tau": d.tau, "sigma": d.sigma, "warmup_requested": args.warmup,
            "carry_refine": d.carry_refine,
            "iteration_GBs_method_44w": method_iter_bytes * K / dt / 1e9,
            "iteration_hbm_frac_method_44w": method_iter_bytes * K / dt / 1e9 / HBM_PEAK_GBS,
            "iteration_kernel_words": iter_words,
            "iteration_GBs_kernel": iter_bytes * K / dt / 1e9,
            "iteration_hbm_frac_kernel": iter_bytes * K / dt / 1e9 / HBM_PEAK_GBS,
            "phase_split_steps": n_split, "phases": split,
            "r_div": rep.r_div, "e_mass": rep.e_mass,
            "copy_GBs": copy_gbs,
        },
        "roofline": roof,
    }
    if not args.no_cpu:
        out["cpu_baseline"] = cpu_baseline(f0, f1, X, Y, C, P, args.cpu_iters)
    if not args.no_side:
        try:
            out["side_workloads"] = side_workloads(args)
        except Exception as e:          # the main line is printed whatever they do
            out["side_workloads"] = {"error": f"{type(e).__name__}: {e}"}
    print(json.dumps(out))


if __name__ == "__main__":
    main()
