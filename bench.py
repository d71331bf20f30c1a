#!/usr/bin/env python3
"""Benchmark: batched local-Hamiltonian application + sparse S/H on one MI355X.

A step is one pass of the whole hot path over every support function of the
workload: uncompress -> potential term (synthesis + magic filter up passes,
potential multiply, down passes) -> kinetic term -> compress, then the S and
H matrix values on their (resident) sparsity patterns.  Inputs are resident
in HBM before the timed region starts; patterns are built once at set-up and
timed separately (the localization regions do not change between steps).

    python bench.py [--steps K] [--warmup W] [--workload gpu16k|batch1k|sweep2k]
                    [--dtype f32|f64] [--no-cpu-baseline]

Prints one JSON line.  --gpus N with N > 1 exits: this build runs on one GPU.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0
FP32_PEAK_TFLOPS = 157.3
FP64_PEAK_TFLOPS = 78.6

WORKLOAD_TEXT = {
    "batch1k": "1,000 support functions, centres uniform in a 30 bohr cube, R ~ U(5,7) bohr, "
               "h = 0.45 bohr, fine radius 3.5 bohr, L' margin 8; one H apply + S + H per step",
    "gpu16k": "16,000 support functions, centres uniform in a 110 bohr cube, R ~ U(5,7) bohr, "
              "h = 0.45 bohr, fine radius 3.5 bohr, L' margin 8; one H apply + S + H per step",
    "sweep2k": "2,000 support functions, cubic boxes of edge E ~ U{16..48} coarse points, "
               "R = (E-1) h / 2, fine radius min(3.5, R) bohr, 0.012 centres per bohr^3, "
               "h = 0.45 bohr, L' margin 8; one H apply + S + H per step",
    "single": "one support function, 20^3 coarse box at h = 0.5 bohr, fine region the inner 10^3",
}


def log(*a):
    print(*a, file=sys.stderr, flush=True)


# ---------------------------------------------------------------------------
# algorithmic work per kernel kind (bytes moved at minimum, flops) per launch
# ---------------------------------------------------------------------------

def _count_up(N):
    """sum over output points of the number of coarse inputs a stride-2 up
    pass reads (per channel pair), for a line of N coarse points."""
    import numpy as np
    l = np.arange(2 * N + 29)
    lo = np.maximum(0, (l - 29) >> 1)
    hi = np.minimum(N - 1, l >> 1)
    return int(np.sum(np.maximum(0, hi - lo + 1)))


def _count_down(N, e):
    import numpy as np
    p = np.arange(N + 2 * e)
    two_i = 2 * (p - e)
    lo = np.maximum(0, two_i)
    hi = np.minimum(2 * N + 28, two_i + 30)
    return int(np.sum(np.maximum(0, hi - lo + 1)))


def work_model(locregs, sz):
    """{kernel kind: (bytes, flops)} of one launch over all functions (both
    terms on).  Bytes count each kernel's inputs and outputs once; flops
    count the multiply-adds of the filters as written (two per MAC)."""
    out = {}

    def add(k, b, f):
        ob, of = out.get(k, (0.0, 0.0))
        out[k] = (ob + b, of + f)
    for r in locregs:
        n0, n1, n2 = (int(v) for v in r["dims"])
        e = int(r["ext"])
        r0, r1, r2 = 2 * n0 + 29, 2 * n1 + 29, 2 * n2 + 29
        o0, o1, o2 = n0 + 2 * e, n1 + 2 * e, n2 + 2 * e
        nin = int(r["n_c"]) + 7 * int(r["n_f"])
        nout = int(r["on_c"]) + 7 * int(r["on_f"])
        c8 = 8 * n0 * n1 * n2
        g = r0 * r1 * r2
        g1, g2, q = 2 * n2 * r1 * r0, 2 * o2 * r1 * r0, 4 * o2 * r0 * o1
        kx, ky, kz = 8 * o0 * n1 * n2, 8 * n0 * o1 * n2, 8 * n0 * n1 * o2
        gx = 4 * n2 * n1 * r0
        # compressed phi -> two dense copies of the coarse box (x and y fastest)
        add("unpack", sz * (nin + 2 * c8), 0)
        # x up pass: 8 coarse components -> 4 channel pairs of x-fine rows
        add("up_x", sz * (c8 + gx), 2 * 2 * 4 * n1 * n2 * _count_up(n0))
        # y up pass: 4 channel pairs -> 2 (x, y)-fine planes per z
        add("up_y", sz * (gx + g1), 2 * 2 * 2 * r0 * n2 * _count_up(n1))
        # z up pass, V multiply, e_pot partials, z down pass
        add("pot_column", sz * (g1 + g + g2),
            2 * 2 * r0 * r1 * _count_up(n2) + 3 * g + 2 * 2 * r0 * r1 * _count_down(n2, e))
        # one axis of the kinetic term: 29 taps from each of two components
        for name, kout in (("kin_xcol", kx), ("kin_ycol", ky), ("kin_zcol", kz)):
            add(name, sz * (c8 + kout), 2 * 58 * kout)
        add("back_y", sz * (g2 + q), 2 * 2 * 2 * r0 * o2 * _count_down(n1, e))
        # x down pass + the three kinetic parts -> compressed output pattern
        add("back_x", sz * (q + kx + ky + kz + nout),
            2 * 2 * 4 * o1 * o2 * _count_down(n0, e) + 3 * 8 * o0 * o1 * o2)
        # the plane kernels: compressed phi -> (x, y)-fine planes; the z column
        # pass; the z kinetic part; x and y kinetic parts, y and x down passes
        # and the compression
        fx, fy = 2 * 2 * 4 * n1 * n2 * _count_up(n0), 2 * 2 * 2 * r0 * n2 * _count_up(n1)
        add("up_plane", sz * (nin + g1), fx + fy)
        add("col_tile", sz * (g1 + g + g2),
            2 * 2 * r0 * r1 * _count_up(n2) + 3 * g + 2 * 2 * r0 * r1 * _count_down(n2, e))
        add("kin_slab", sz * (nin + kz), 2 * 58 * kz)
        add("back_plane", sz * (nin + g2 + kz + nout),
            2 * 2 * 2 * r0 * o2 * _count_down(n1, e) + 2 * 2 * 4 * o1 * o2 * _count_down(n0, e)
            + 2 * 58 * (kx + ky) + 3 * 8 * o0 * o1 * o2)
    return out


def path_bytes(locregs, sz):
    """Algorithmic bytes of one step: compressed phi in, compressed H phi out,
    each function's potential block, and one read of phi (S) and phi + H phi (H)."""
    tot = 0
    for r in locregs:
        n = [int(v) for v in r["dims"]]
        nin = int(r["n_c"]) + 7 * int(r["n_f"])
        nout = int(r["on_c"]) + 7 * int(r["on_f"])
        g = (2 * n[0] + 29) * (2 * n[1] + 29) * (2 * n[2] + 29)
        tot += sz * (nin + nout + g) + sz * (nin + nin + nout)
    return tot


def source_hash():
    h = hashlib.sha256()
    for f in ("wvl_kernels.hip", "wvl_fused.hip", "wvl_planes.hip", "wvl_static.hip", "wvl_host.cpp",
              "wvl_internal.h", "wvl_filters.h"):
        with open(os.path.join(ROOT, "paper_1401_7441_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def load_traffic(kernel, workload, dtype):
    """HBM bytes per launch from committed rocprofv3 counter summaries, when
    they were taken on the current kernel sources."""
    path = os.path.join(ROOT, "profiles", "hbm_traffic.json")
    if not os.path.exists(path):
        return None
    try:
        with open(path) as f:
            tab = json.load(f)
        ent = tab.get(f"{workload}/{dtype}/{kernel}")
        if ent and ent.get("source_hash") == source_hash():
            return float(ent["bytes_per_launch"])
    except (OSError, ValueError, KeyError):
        return None
    return None


# ---------------------------------------------------------------------------
# workload set-up
# ---------------------------------------------------------------------------

def setup(workload, dtype_name):
    import numpy as np
    import torch

    import inputs
    import paper_1401_7441_amd as W

    t0 = time.perf_counter()
    g = inputs.geometry(workload)
    if workload == "single":
        raise SystemExit("the single-function workload is a parity case; use batch1k or gpu16k")
    lr, segs = W.build_locregs(g.h, g.grid_n, g.centers, g.radii, g.fine_radii, g.ext)
    t_lr = time.perf_counter() - t0
    dt = torch.float32 if dtype_name == "f32" else torch.float64
    coefs = []
    for k in range(len(lr)):
        r = lr[k]
        sc = segs[int(r["seg_c"]):int(r["seg_c"]) + int(r["nseg_c"])]
        sf = segs[int(r["seg_f"]):int(r["seg_f"]) + int(r["nseg_f"])]
        coefs.append(inputs.coefficients(g, k, _points(sc), _points(sf)))
    psi = torch.tensor(np.concatenate(coefs), dtype=dt, device="cuda")
    pot = inputs.potential(g, device="cuda").to(dt).contiguous()
    ctx = W.Context(g.h, g.grid_n)
    plan = W.Plan(ctx, lr, segs)
    hpsi = torch.zeros(plan.info["out_coefs"], dtype=dt, device="cuda")
    ek = torch.zeros(len(lr), dtype=torch.float64, device="cuda")
    ep = torch.zeros_like(ek)
    ws = plan.new_workspace(dt)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    nnz_s = W.sparse_pattern_nnz(plan, False)
    nnz_h = W.sparse_pattern_nnz(plan, True)
    t_pat = time.perf_counter() - t1
    s_out = (torch.empty(len(lr) + 1, dtype=torch.int64, device="cuda"),
             torch.empty(max(1, nnz_s), dtype=torch.int32, device="cuda"),
             torch.empty(max(1, nnz_s), dtype=torch.float64, device="cuda"))
    h_out = (torch.empty(len(lr) + 1, dtype=torch.int64, device="cuda"),
             torch.empty(max(1, nnz_h), dtype=torch.int32, device="cuda"),
             torch.empty(max(1, nnz_h), dtype=torch.float64, device="cuda"))
    return dict(g=g, lr=lr, segs=segs, psi=psi, pot=pot, ctx=ctx, plan=plan, hpsi=hpsi, ek=ek,
                ep=ep, ws=ws, s_out=s_out, h_out=h_out, nnz_s=nnz_s, nnz_h=nnz_h,
                t_locreg=t_lr, t_pattern=t_pat, dtype=dt)


def _points(seg):
    import numpy as np
    pts = [np.stack([np.arange(s["i1s"], s["i1e"] + 1),
                     np.full(s["i1e"] - s["i1s"] + 1, s["i2"]),
                     np.full(s["i1e"] - s["i1s"] + 1, s["i3"])], axis=1) for s in seg]
    return np.concatenate(pts) if pts else np.zeros((0, 3), np.int64)


def step(S):
    import paper_1401_7441_amd as W
    W.apply_local_ham(S["plan"], S["psi"], S["pot"], S["hpsi"], S["ek"], S["ep"], S["ws"])
    W.sparse_overlap(S["plan"], S["psi"], S["psi"], False, out=S["s_out"])
    W.sparse_overlap(S["plan"], S["psi"], S["hpsi"], True, out=S["h_out"])


def density_section(S, reps=3):
    """Fine-box values of every function (wvl_synthesize) and the density
    rho = sum_ab phi_a K^ab phi_b (wvl_density) with a smooth kernel
    K_ab = 0.5 exp(-|R_a - R_b|^2 / 18) on the overlap pattern."""
    import numpy as np
    import torch

    import paper_1401_7441_amd as W
    plan, psi, ctx = S["plan"], S["psi"], S["ctx"]
    g = S["g"]
    n = g.grid_n
    fine = torch.empty(plan.info["fine_box"], dtype=psi.dtype, device="cuda")
    work = None
    rho = torch.empty((2 * n[0] + 29) * (2 * n[1] + 29) * (2 * n[2] + 29), dtype=psi.dtype,
                      device="cuda")
    rowptr, col, _ = W.sparse_overlap(plan, psi, psi, False, values=False)
    rp = rowptr.cpu().numpy()
    row = np.repeat(np.arange(len(rp) - 1), np.diff(rp))
    c = np.asarray(g.centers, np.float64)
    d2 = np.sum((c[row] - c[col.cpu().numpy()]) ** 2, axis=1)
    kval = torch.tensor(0.5 * np.exp(-d2 / 18.0), dtype=torch.float64, device="cuda")
    W.synthesize(plan, psi, fine, S["ws"])
    W.density(plan, fine, rowptr, col, kval, rho, work)
    torch.cuda.synchronize()
    ctx.profile(True)
    ctx.profile_reset()
    t0 = time.perf_counter()
    for _ in range(reps):
        W.synthesize(plan, psi, fine, S["ws"])
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(reps):
        W.density(plan, fine, rowptr, col, kval, rho, work)
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    prof = ctx.profile_read()
    ctx.profile(False)
    sz = psi.element_size()
    nfine = plan.info["fine_box"]
    grid_pts = rho.numel()
    # pair work: every kernel entry over the common part of the two fine boxes
    lo = np.array([[int(v) for v in r["lo"]] for r in S["lr"]])
    dims = np.array([[int(v) for v in r["dims"]] for r in S["lr"]])
    a0, a1 = 2 * lo, 2 * lo + 2 * dims + 29
    cb = col.cpu().numpy()
    ov = np.prod(np.maximum(0, np.minimum(a1[row], a1[cb]) - np.maximum(a0[row], a0[cb])), axis=1)
    pair_pts = float(np.sum(ov))
    kern = {k: {"launches": v[0] // reps, "avg_ms": v[1] / v[0]} for k, v in prof.items() if v[0]}
    tile_ms = kern.get("dens_tile", {}).get("avg_ms")
    return {
        "synthesize_ms": (t1 - t0) * 1e3 / reps,
        "density_ms": (t2 - t1) * 1e3 / reps,
        "kernels": kern,
        "fine_box_points": nfine,
        "grid_points": grid_pts,
        "kernel_nnz": int(kval.numel()),
        "pair_box_points": pair_pts,
        # k_dens_tile: algorithmic bytes = the fine values read once and rho
        # written once; flops = a multiply-add per kernel entry and common
        # fine point (pair_box_points of them)
        "dens_tile_alg_gbps": ((nfine + grid_pts) * sz / (tile_ms * 1e-3) / 1e9)
        if tile_ms else None,
        "dens_tile_tflops": (2 * pair_pts / (tile_ms * 1e-3) / 1e12) if tile_ms else None,
        "note": "K on the overlap (S) pattern, smooth synthetic values; eager calls",
    }


def foe_section(S, npl=100, delta=1.0, reps=2):
    """Density kernel by the Fermi operator expansion on the step's S and H
    (overlap pattern, Gershgorin bounds, half the functions occupied)."""
    import torch

    import paper_1401_7441_amd as W
    plan, ctx = S["plan"], S["ctx"]
    psi, hpsi = S["psi"], S["hpsi"]
    _, _, sv = W.sparse_overlap(plan, psi, psi, False)
    _, _, hv = W.sparse_overlap(plan, psi, hpsi, True)
    nsf = plan.nsf
    W.foe(plan, sv, hv, npl, delta, 0.5 * nsf)
    torch.cuda.synchronize()
    ctx.profile(True)
    ctx.profile_reset()
    t0 = time.perf_counter()
    for _ in range(reps):
        _, mu, ebs = W.foe(plan, sv, hv, npl, delta, 0.5 * nsf)
    ms = (time.perf_counter() - t0) * 1e3 / reps
    prof = ctx.profile_read()
    ctx.profile(False)
    kern = {k: {"launches": v[0] // reps, "avg_ms": v[1] / v[0]} for k, v in prof.items() if v[0]}
    nnz = int(sv.numel())
    mm = kern.get("foe_mm", {})
    return {"ms": ms, "npl": npl, "delta": delta, "n_occ": 0.5 * nsf, "nnz": nnz, "mu": mu,
            "e_bs": ebs, "kernels": kern,
            # one truncated product reads the two operands and the third
            # term once and writes the result (plus the pattern): per entry
            # 4 doubles and 12 bytes of indices
            "foe_mm_alg_gbps": (nnz * 44 / (mm["avg_ms"] * 1e-3) / 1e9) if mm else None,
            "note": "S and H of the timed step; npl - 1 truncated products of the Chebyshev "
                    "recursion (every T^i kept, the traces and the kernel summed from them) "
                    "plus the transforms; the call synchronizes"}


# ---------------------------------------------------------------------------
# CPU baseline: the FP64 oracle on a bounded sample of the same workload
# ---------------------------------------------------------------------------

_ORACLE = {}


def _usable_cores():
    """Host cores this process may use: its CPU affinity, capped by
    OMP_NUM_THREADS when that is set (the share of the host given to a job)."""
    n = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    cap = os.environ.get("OMP_NUM_THREADS")
    if cap and cap.isdigit() and int(cap) > 0:
        n = min(n, int(cap))
    return max(1, n)


def _cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline_prepare(workload):
    """Oracle set-up for the CPU baseline, done before the GPU is touched so
    that the worker processes forked here hold no GPU state: the geometry,
    the oracle's sphere sets (fine-set union included) and the potential
    in FP64.  Returns the pool of workers (one per usable core)."""
    import multiprocessing as mp

    import inputs
    from oracle import locreg
    t0 = time.perf_counter()
    g = inputs.geometry(workload)
    _ORACLE["g"] = g
    _ORACLE["spheres"] = locreg.SphereSet(g.h, g.grid_n, g.centers, g.radii, g.fine_radii,
                                          g.ext)
    _ORACLE["pot"] = inputs.potential(g).numpy()
    cores = _usable_cores()
    pool = mp.get_context("fork").Pool(cores, initializer=_oracle_worker_init)
    log(f"cpu baseline: oracle set-up {time.perf_counter() - t0:.1f} s, {cores} workers")
    return pool, cores


def _oracle_worker_init():
    try:
        from threadpoolctl import threadpool_limits
        _ORACLE["limits"] = threadpool_limits(1)     # one core per worker
    except ImportError:
        pass


def _oracle_task(task):
    """One function: the oracle's FP64 local-H apply (timed), then its error
    against the GPU's output of the timed step.  Skipped (None) once the
    shared deadline has passed."""
    import numpy as np

    import inputs
    from oracle import hamiltonian, locreg
    k, deadline, got, ek, ep = task
    if time.time() > deadline:
        return None
    g = _ORACLE["g"]
    l = _ORACLE["spheres"].locreg(k)
    c = inputs.coefficients(g, k, locreg.points_from_segments(l.cseg),
                            locreg.points_from_segments(l.fseg))
    t = time.perf_counter()
    ref, rk, rp = hamiltonian.apply_local_ham(l, c, _ORACLE["pot"], g.h)
    dt = time.perf_counter() - t
    err = float(np.linalg.norm(got.astype(np.float64) - ref) / np.linalg.norm(ref))
    return k, dt, int(np.prod([2 * d + 29 for d in l.dims])), err, abs(ek - rk), abs(ep - rp)


def cpu_baseline_submit(pool, S, cores, deadline_s=20.0, per_core=48, seed=7441):
    """Starts the oracle on a seeded random sample of the workload's functions
    (at most per_core per worker; the GPU's outputs of the timed step, copied
    to the host here, go with each task); returns the pending result."""
    import numpy as np
    import torch
    nsf = len(S["lr"])
    order = [int(k) for k in np.random.default_rng(seed).permutation(nsf)[:per_core * cores]]
    ek = S["ek"].cpu().numpy()
    ep = S["ep"].cpu().numpy()
    spans = []
    for k in order:
        r = S["lr"][k]
        spans.append((int(r["ocoef_off"]), int(r["on_c"]) + 7 * int(r["on_f"])))
    flat = torch.cat([S["hpsi"][o:o + n] for o, n in spans]).cpu().numpy()
    ends = np.cumsum([n for _, n in spans])
    deadline = time.time() + deadline_s
    tasks = [(k, deadline, flat[e - n:e], float(ek[k]), float(ep[k]))
             for k, (_, n), e in zip(order, spans, ends)]
    return pool.imap_unordered(_oracle_task, tasks), deadline_s


def cpu_baseline_collect(pending, cores, workload, pool):
    results, deadline_s = pending
    done = [r for r in results if r is not None]
    pool.close()
    pool.join()
    if not done:
        return None, None
    t_apply = sum(r[1] for r in done)
    pts = sum(r[2] for r in done)
    rate = len(done) / (t_apply / cores)
    base = {"value": rate, "unit": "SF H-applies/s", "cores": cores, "kind": "oracle",
            "sample": f"{len(done)} of the workload's support functions in a seeded random "
                      f"order, local H apply only (no S/H), FP64 numpy oracle, one function "
                      f"per worker process at a time on {cores} cores for about "
                      f"{deadline_s:.0f} s; rate = functions / (summed apply time / cores)",
            "fine_grid_pts_per_s": pts / (t_apply / cores),
            "nproc": os.cpu_count(), "cpu_model": _cpu_model()}
    acc = {"n_sf": len(done), "workload": workload,
           "hpsi_rel_max": max(r[3] for r in done),
           "e_kin_abs_max_ha": max(r[4] for r in done),
           "e_pot_abs_max_ha": max(r[5] for r in done),
           "note": "GPU output of the timed step against the FP64 oracle on the sampled "
                   "functions (each normalized): H|phi> per-function relative 2-norm error, "
                   "energies absolute per function"}
    return base, acc


# ---------------------------------------------------------------------------

def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="gpu16k", choices=["batch1k", "gpu16k", "sweep2k"])
    ap.add_argument("--dtype", default="f32", choices=["f32", "f64"])
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-trace", action="store_true",
                    help="skip the traced eager pass (no per-kernel times, no roofline)")
    ap.add_argument("--eager", action="store_true",
                    help="time eager library calls instead of replays of the captured step")
    ap.add_argument("--no-autotune", action="store_true",
                    help="keep the plan's default schedule (one bin, largest row tiles)")
    ap.add_argument("--autotune-reps", type=int, default=2)
    ap.add_argument("--schedule", default=None, metavar="NBINS,KIN_MFMA",
                    help="set this schedule instead of autotuning (e.g. 8,1: eight bins, "
                         "kinetic z part on the matrix cores)")
    ap.add_argument("--no-serve", action="store_true",
                    help="skip the request-loop measurement (p50/p99 latency)")
    ap.add_argument("--serve-requests", type=int, default=200,
                    help="requests of the Poisson trace at 0.8 of the saturated rate")
    ap.add_argument("--serve-pool", type=int, default=32,
                    help="distinct systems the serving requests are drawn from")
    ap.add_argument("--serve-other", type=int, default=100,
                    help="requests at the other offered loads (0.5, 0.95)")
    ap.add_argument("--serve-saturated", type=int, default=100,
                    help="requests of the saturated run")
    ap.add_argument("--serve-baseline", type=int, default=4,
                    help="requests of the per-function FP64 baseline")
    ap.add_argument("--no-density", action="store_true",
                    help="skip the fine-grid values + density section")
    ap.add_argument("--no-foe", action="store_true",
                    help="skip the Fermi-operator-expansion section")
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="run one plain device copy of this size first (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}); the multi-GPU "
              "sharding of this path is a design in the notes, not part of this build",
              file=sys.stderr)
        sys.exit(2)
    pool = None
    if not args.no_cpu_baseline:
        # before the GPU is touched: the workers are forked here
        pool, cores = cpu_baseline_prepare(args.workload)
    import torch
    assert torch.cuda.is_available(), "bench.py needs a GPU"
    import paper_1401_7441_amd as W  # noqa: F401  (fails loudly without libwvl.so)

    if args.copy_calibration_mib:
        n = args.copy_calibration_mib * (1 << 20) // 4
        a = torch.ones(n, dtype=torch.float32, device="cuda")
        b = torch.empty_like(a)
        b.copy_(a)
        torch.cuda.synchronize()
        del a, b
    log(f"set-up: workload {args.workload}, {args.dtype}")
    S = setup(args.workload, args.dtype)
    nsf = len(S["lr"])
    log(f"set-up done: {nsf} functions, locregs {S['t_locreg']:.2f} s, patterns "
        f"{S['t_pattern'] * 1e3:.1f} ms (S nnz {S['nnz_s']}, H nnz {S['nnz_h']}), "
        f"workspace {S['ws'].numel() / 2**30:.2f} GiB")
    tune = None
    if args.schedule:
        nb, km = (int(v) for v in args.schedule.split(","))
        W.set_schedule(S["plan"], nb, km)
        tune = {"set": {"nbins": nb, "kin_mfma": km}}
        log(f"schedule set: {nb} bins, kin_mfma {km}")
    elif not args.no_autotune:
        t0 = time.perf_counter()
        best, tried = W.autotune(S["plan"], S["psi"], S["pot"], S["hpsi"], S["ws"],
                                 reps=args.autotune_reps)
        tune = {"best": best, "tried": tried, "seconds": time.perf_counter() - t0}
        log(f"autotune: {best} ({len(tried)} layouts, {tune['seconds']:.1f} s)")
    graph = None
    if not args.eager:
        graph = W.Graph(S["plan"], S["psi"], S["pot"], S["hpsi"], S["ek"], S["ep"],
                        workspace=S["ws"], s_val=S["s_out"][2], h_val=S["h_out"][2])
    run = graph.launch if graph is not None else (lambda: step(S))
    for _ in range(args.warmup):
        run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        run()
    torch.cuda.synchronize()
    dt_s = time.perf_counter() - t0
    # the oracle on a sample of the functions runs on the host cores while
    # the sections below use the GPU; the timed step's outputs go with it
    pending = cpu_baseline_submit(pool, S, cores) if pool is not None else None
    # per-kernel times: library events around every launch of K eager steps
    ctx = S["ctx"]
    prof = {}
    eager_ms = None
    conf_ms, cprof, precond_ms = None, {}, None
    if not args.no_trace:
        ctx.profile(True)
        ctx.profile_reset()
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        for _ in range(args.steps):
            step(S)
        torch.cuda.synchronize()
        eager_ms = (time.perf_counter() - t1) * 1e3 / args.steps
        prof = ctx.profile_read()
        # the same applies with a confining potential a |r - R|^4 on every function
        conf = torch.full((nsf,), 0.01, dtype=torch.float64, device="cuda")
        ctx.profile_reset()
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        for _ in range(args.steps):
            W.apply_local_ham(S["plan"], S["psi"], S["pot"], S["hpsi"], S["ek"], S["ep"],
                              S["ws"], conf=conf)
        torch.cuda.synchronize()
        conf_ms = (time.perf_counter() - t1) * 1e3 / args.steps
        cprof = ctx.profile_read()
        ctx.profile(False)
        # gradient preconditioning: 5 conjugate-gradient steps of
        # (T + C - eps) x = -g for every function
        eps = torch.full((nsf,), -0.5, dtype=torch.float64, device="cuda")
        gx = torch.empty_like(S["psi"])
        W.precondition(S["plan"], S["psi"], eps, 5, gx, conf=conf, workspace=S["ws"])
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        W.precondition(S["plan"], S["psi"], eps, 5, gx, conf=conf, workspace=S["ws"])
        torch.cuda.synchronize()
        precond_ms = (time.perf_counter() - t1) * 1e3
        del gx
    ms_step = dt_s * 1e3 / args.steps
    value = nsf * args.steps / dt_s
    sz = 4 if args.dtype == "f32" else 8
    fine_pts = sum(int((2 * r["dims"][0] + 29) * (2 * r["dims"][1] + 29) * (2 * r["dims"][2] + 29))
                   for r in S["lr"])
    model = work_model(S["lr"], sz)
    # S and H values: phi (and H phi) read once, one value per pair written
    info = S["plan"].info
    model["sparse_s"] = (sz * info["in_coefs"] + 8.0 * S["nnz_s"], 0.0)
    model["sparse_h"] = (sz * (info["in_coefs"] + info["out_coefs"]) + 8.0 * S["nnz_h"], 0.0)
    kernels = {}
    for k, (n, ms) in prof.items():
        if n:
            b, f = model.get(k, (0.0, 0.0))
            step_s = ms * 1e-3 / args.steps          # this kind's time per step
            kernels[k] = {"launches": n, "avg_ms": ms / n,
                          "ms_per_step": ms / args.steps,
                          "gbps": (b / step_s / 1e9) if b else None,
                          "tflops": (f / step_s / 1e12) if f else None}
    roofline = None
    if kernels:
        # dominant kernel: the largest share of a step.  A kind launches once
        # per chunk; the model's bytes and flops are per step, so per launch
        # they are divided by the launches per step.
        dom = max(kernels, key=lambda k: kernels[k]["ms_per_step"])
        b, f = model.get(dom, (0.0, 0.0))
        per_step = kernels[dom]["launches"] / args.steps
        b, f = b / per_step, f / per_step
        avg = kernels[dom]["avg_ms"] * 1e-3
        peak_f = FP32_PEAK_TFLOPS if args.dtype == "f32" else FP64_PEAK_TFLOPS
        ridge = peak_f * 1e12 / (HBM_PEAK_GBPS * 1e9)
        if f and f / max(b, 1.0) > ridge:
            ach = f / avg / 1e12
            roofline = {"kernel": dom, "bound": "alu", "achieved": ach, "peak": peak_f,
                        "unit": "TFLOP/s", "frac": ach / peak_f}
        else:
            ach = b / avg / 1e9
            roofline = {"kernel": dom, "bound": "hbm", "achieved": ach, "peak": HBM_PEAK_GBPS,
                        "unit": "GB/s", "frac": ach / HBM_PEAK_GBPS}
        roofline["algorithmic_bytes_per_launch"] = b
        roofline["flops_per_launch"] = f
        roofline["avg_launch_ms"] = kernels[dom]["avg_ms"]
        tr = load_traffic(dom, args.workload, args.dtype)   # measured on a one-chunk layout
        roofline["traffic"] = tr / per_step if tr is not None else None
    pb = path_bytes(S["lr"], sz)
    res = {
        "metric": "support-function H-applies/s (fine grid pts/s, % HBM peak); p50/p99 request "
                  "latency",
        "value": value,
        "unit": "SF H-applies/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": args.dtype,
        "data": "synthetic",
        "config": {"workload": f"{args.workload}: {WORKLOAD_TEXT[args.workload]}",
                   "nsf": nsf, "h_bohr": S["g"].h, "ext": int(S["g"].ext),
                   "grid": list(S["g"].grid_n), "conv_dtype": args.dtype,
                   "reduction_dtype": "f64", "s_nnz": S["nnz_s"], "h_nnz": S["nnz_h"]},
        "fine_grid_pts_per_s": fine_pts * args.steps / dt_s,
        "path_hbm": {"algorithmic_bytes_per_step": pb, "gbps": pb / (ms_step * 1e-3) / 1e9,
                     "frac": pb / (ms_step * 1e-3) / 1e9 / HBM_PEAK_GBPS},
        "roofline": roofline,
        "kernels": kernels,
        "kernel_timing": "HIP events the library records around each launch on its stream, "
                         "over a separate pass of the same number of eager steps",
        "confinement": None if conf_ms is None else {
            "apply_ms": conf_ms,
            "pot_column_ms": cprof["pot_column"][1] / max(1, args.steps),
            "pot_column_ms_without": prof["pot_column"][1] / max(1, args.steps),
            "prefactor": 0.01},
        "preconditioner": None if precond_ms is None else {
            "ms": precond_ms, "cg_steps": 5, "confinement": 0.01, "eps": -0.5,
            "note": "all functions, one apply (kinetic + confinement) per step"},
        "schedule": {"timed": "graph replay" if graph is not None else "eager calls",
                     "eager_ms_per_step": eager_ms,
                     "nbins": (tune["best"] if tune and "best" in tune else
                               tune["set"] if tune else {"nbins": 1})["nbins"],
                     "kin_mfma": (tune["best"] if tune and "best" in tune else
                                  tune["set"] if tune else {"kin_mfma": 0})["kin_mfma"],
                     "chunks": S["plan"].info["chunks"],
                     "autotune": tune},
        "setup": {"locregs_s": S["t_locreg"], "patterns_ms": S["t_pattern"] * 1e3},
        "source_hash": source_hash(),
    }
    if not args.no_density:
        log("density: fine-box values and rho on the fine grid")
        res["density"] = density_section(S)
        log(f"density: synthesize {res['density']['synthesize_ms']:.2f} ms, "
            f"density {res['density']['density_ms']:.2f} ms")
    if not args.no_foe:
        log("foe: density kernel by the Fermi operator expansion")
        res["foe"] = foe_section(S)
        log(f"foe: {res['foe']['ms']:.1f} ms")
    if pending is not None:
        res["cpu_baseline"], res["accuracy"] = cpu_baseline_collect(pending, cores,
                                                                    args.workload, pool)
        log(f"cpu baseline: {res['cpu_baseline']}")
        log(f"accuracy: {res['accuracy']}")
    if not args.no_serve:
        # free the batch before the serving run takes its HBM budget
        if graph is not None:
            graph.close()
        del graph, run
        S.clear()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        from paper_1401_7441_amd import serve
        res["serving"] = serve.benchmark(n_requests=args.serve_requests, dtype=args.dtype,
                                         pool_size=args.serve_pool, n_other=args.serve_other,
                                         n_saturated=args.serve_saturated,
                                         baseline_requests=args.serve_baseline,
                                         log=log)
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
