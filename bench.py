#!/usr/bin/env python3
"""Benchmark of the all-mode-averaging solve on one MI355X.

Workload (default): 32^3 x 64 lattice, U = exp(i 0.4 H) from seed 1,
kappa = 0.124, c_sw = 1.5; source positions x0 + g with g on the grid
{0,16,32,48} x {0,16}^3 (32 positions, block-checkerboard preserving);
12 point sources per position solved sloppily (FP16 link/clover storage,
FP32 SAP and Krylov vectors, relative residual 3e-3) and the 12 sources of
the first position solved exactly (FP64 outer, residual 1e-10), all with
SAP (n_cy = 5, n_mr = 4) and block-local deflation.

One step = the whole path on one gauge field: field preparation from links
already in HBM (site tables, storage copies, clover term and inverse),
deflation setup, all sloppy and exact solves.  The metric is seconds per
source position (step time / 32); lower is better.

Also reported: a roofline object for the kernel class that takes the most
time (HIP events on the launch stream, algorithmic work per launch from the
library's counters), the oracle's time on the host for a bounded sample
(scaled to the same work), and a per-phase breakdown.
"""

from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

import synth  # noqa: E402

F64, F32, F16, BF16 = 0, 1, 2, 3
PEAK_HBM_GBS = 8000.0
PEAK_FP32_TFLOPS = 157.3
# FP32 vector peak without packed-FP32 instructions (which this library is
# built without): 256 CUs x 64 lanes x 2 flop per FMA x 2.4 GHz
PEAK_FP32_UNPACKED_TFLOPS = 256 * 64 * 2 * 2.4e9 / 1e12
PEAK_FP64_TFLOPS = 78.6

WORKLOADS = {
    # the headline configuration
    "ama-32c64": dict(dims=(64, 32, 32, 32), eps=0.4, kappa=0.124, csw=1.5, seed=1,
                      grid=((0, 16, 32, 48), (0, 16), (0, 16), (0, 16))),
    # small configuration for quick checks
    "ama-16c32": dict(dims=(32, 16, 16, 16), eps=0.4, kappa=0.124, csw=1.5, seed=1,
                      grid=((0, 16), (0, 8), (0, 8), (0, 8))),
}


def positions(work, block):
    dims = work["dims"]
    x0 = synth.seeded_site(dims, work["seed"])
    t0, xx0, y0, z0 = (int(v) for v in synth.coords(dims, x0))
    # every shift is a whole number of blocks with an even number of block
    # steps for the 4^4, 8x4^3 and 8^4 blocks, so M_SAP is covariant under it
    out = []
    for gt in work["grid"][0]:
        for gx in work["grid"][1]:
            for gy in work["grid"][2]:
                for gz in work["grid"][3]:
                    out.append(((t0 + gt) % dims[0], (xx0 + gx) % dims[1], (y0 + gy) % dims[2], (z0 + gz) % dims[3]))
    return out


def sap_flops_per_site_sweep(block, nmr, first=False):
    hops = sum(2.0 * (b - 1) / b for b in block)
    h = 165.0 * hops
    pair = (0.0 if first else 3792.0) + 504 + (h + 72) + nmr * (2 * h + 1392) + (h + 576)
    return pair / 2


def cpu_baseline(work, block, prof, nsrc, ncy, nmr, threads):
    """Oracle on the host: M and M_SAP applications (one right-hand side,
    mean of two each) on the workload's lattice, scaled by the step's
    site-applications of the stencil and the Schwarz sweeps (deflation setup,
    little solves and vector algebra are not counted, so this is a lower
    bound of the oracle's time)."""
    import oracle
    dims = work["dims"]
    U = synth.gauge_field(dims, work["eps"], work["seed"])
    op = oracle.Operator(dims, U, work["kappa"], work["csw"], -1)
    _ = op.Ainv
    x = synth.gaussian_spinor(dims, 1, 1001)[0]
    reps = 2
    t = time.perf_counter()
    for _ in range(reps):
        op.M(x)
    tM = (time.perf_counter() - t) / reps
    t = time.perf_counter()
    for _ in range(reps):
        op.sap(x, block, ncy, nmr)
    tS = (time.perf_counter() - t) / reps
    V = synth.volume(dims)
    per_dirac_site = tM / V
    per_sap_site_sweep = tS / (V * ncy)
    est = prof["dirac"]["units"] * per_dirac_site + prof["sap"]["units"] * per_sap_site_sweep
    return {
        "value": est / nsrc,
        "unit": "s/source",
        "cores": threads,
        "kind": "oracle",
        "sample": (f"M ({tM:.2f} s) and M_SAP ({tS:.2f} s) applications, mean of {reps} each, 1 rhs, {dims} lattice, "
                   f"scaled by the step's {prof['dirac']['units']:.3g} stencil and {prof['sap']['units']:.3g} "
                   "Schwarz site-applications; deflation setup, little solves and vector algebra not counted"),
    }


def fp64_single_rhs(fld, d, pos, npos, setup_s, little_maxit, little_maxit_sloppy, log):
    """The comparator: the same deflated SAP-GCR solver with every step in
    FP64 (operator storage, Schwarz sweeps, Krylov vectors) and one
    right-hand side per solve, at the same final residuals.  Timed on a
    bounded sample (the 12 sloppy solves of one position, then its 12 exact
    solves) and scaled to the workload: (field and deflation setup +
    npos x sloppy set + one exact set) / npos."""
    import torch
    import paper_1605_00564_amd as dfl
    sap = dfl.SapParams(5, 4, F64)
    sloppy = dfl.GcrParams(nkv=8, nmx=24, res=3e-3, sap=sap, dfl=d, little_tol=1e-6, little_maxit=little_maxit_sloppy)
    exact = dfl.GcrParams(nkv=16, nmx=400, res=1e-10, sap=sap, dfl=d, little_tol=1e-10, little_maxit=little_maxit)
    V = fld.V
    xs = [torch.empty((12, V, 4, 3), dtype=torch.complex128, device="cuda")]
    xe = [torch.empty((12, V, 4, 3), dtype=torch.complex128, device="cuda")]
    # one untimed pass of each kind so that work buffers exist
    dfl.ama_solve(fld, pos[:1], [True], sloppy, exact, dtype=torch.complex128, batch=1, out_sloppy=xs, out_exact=xe)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    _, _, i_s, _ = dfl.ama_solve(fld, pos[:1], [False], sloppy, exact, dtype=torch.complex128, batch=1,
                                 out_sloppy=xs, out_exact=[])
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    _, _, _, i_e = dfl.ama_solve(fld, pos[:1], [True], sloppy, exact, dtype=torch.complex128, batch=1,
                                 out_sloppy=xs, out_exact=xe)
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    t_s = t1 - t0
    t_e = max((t2 - t1) - t_s, 0.0)
    est = (setup_s + npos * t_s + t_e) / npos
    log(f"[bench] fp64 single-rhs: 12 sloppy {t_s:.2f} s, 12 exact {t_e:.2f} s")
    return {"value": est, "unit": "s/source", "sloppy_set_s": t_s, "exact_set_s": t_e, "setup_s": setup_s,
            "sloppy_iters": [min(i.iters for i in i_s), max(i.iters for i in i_s)],
            "sloppy_max_rel_res": max(i.rel_res for i in i_s),
            "exact_iters": [min(i.iters for i in i_e), max(i.iters for i in i_e)],
            "exact_max_rel_res": max(i.rel_res for i in i_e),
            "sample": "12 sloppy and 12 exact single-rhs FP64 solves at one position, scaled to all positions"}


KERNEL_SOURCES = {
    "k_sap_sweep": ["paper_1605_00564_amd/csrc/sap.hip", "paper_1605_00564_amd/csrc/internal.h"],
    "k_dirac": ["paper_1605_00564_amd/csrc/dirac.hip", "paper_1605_00564_amd/csrc/internal.h"],
}


def measured_traffic(kernel, workload):
    """HBM bytes per launch of `kernel` on `workload` from the committed
    counter summary (FETCH_SIZE and WRITE_SIZE, each scaled by what the same
    counter reads for an elementwise kernel of known size), or None when there
    is no summary or the kernel's sources changed since it was taken."""
    import hashlib
    path = os.path.join(ROOT, "profiles", f"{kernel}_{workload}.txt")
    if kernel not in KERNEL_SOURCES or not os.path.exists(path):
        return None
    vals = {}
    for line in open(path):
        if not line.startswith((" ", "#")) and ":" in line:
            k, v = line.split(":", 1)
            vals[k.strip()] = v.split()[0] if v.split() else ""
    h = hashlib.sha256()
    for f in KERNEL_SOURCES[kernel]:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    if vals.get("sources_sha256") != h.hexdigest() or "traffic_bytes_per_launch" not in vals:
        return None
    return float(vals["traffic_bytes_per_launch"])


# stencil storage modes: (operator storage, spinor storage in and out)
STENCIL_MODES = {
    "f64": (F64, F64), "f32": (F32, F32),
    "f16": (F16, F32), "bf16": (BF16, F32),         # FP16 / BF16 links and clover, FP32 spinors
    "f16s": (F16, F16), "bf16s": (BF16, F16),       # the same with FP16 spinors (per-site scale)
}


def stencil_sweep(lattices, storages, nrhs_list, reps, log, cpu=True):
    """Dirac-operator GB/s and Gflop/s per storage mode and right-hand-side
    count, on the kernels of the internal layout that the solvers use (kernel
    time from HIP events; pack/unpack kernels excluded).  With
    cpu, the oracle's FP64 operator on the host is timed beside it (one
    application, one right-hand side, the same algorithmic bytes and flops)."""
    import torch
    import paper_1605_00564_amd as dfl
    rows = []
    for dims in lattices:
        U = synth.gauge_field(dims, 0.4, 1, progress=lambda f: log(f"[sweep] {dims}: gauge field {100 * f:.0f}%"))
        fld = dfl.Field(dims, (4, 4, 4, 4), 0.124, 1.5, torch.from_numpy(U).cuda())
        fld.tune(dfl.Field.TUNE_DIRAC_CANON, 2)
        V = synth.volume(dims)
        if cpu:
            import oracle
            log(f"[sweep] {dims}: oracle operator (clover term and its inverse) on the host")
            op = oracle.Operator(dims, U, 0.124, 1.5, -1)
            x = synth.gaussian_spinor(dims, 1, 1001)[0]
            op.M(x)
            t = time.perf_counter()
            op.M(x)
            dt = time.perf_counter() - t
            by = V * (4 * 144.0 + 576.0 + 2 * 192.0)
            row = {"lattice": "x".join(map(str, dims)), "storage": "f64", "nrhs": 1, "device": "oracle (host)",
                   "cores": int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1)), "ms": 1e3 * dt,
                   "GB/s": by / dt / 1e9, "Gflop/s": 1872.0 * V / dt / 1e9}
            rows.append(row)
            log(json.dumps(row))
            del op, x
        del U
        for mode in storages:
            st, sp = STENCIL_MODES[mode]
            dt = torch.complex128 if st == F64 else torch.complex64
            for n in nrhs_list:
                x = torch.randn((n, V, 4, 3), dtype=dt, device="cuda")
                y = torch.empty_like(x)
                for _ in range(2):
                    dfl.dirac_apply(fld, x, storage=st, out=y, spinor_in=sp, spinor_out=sp)
                torch.cuda.synchronize()
                dfl.prof_reset()
                dfl.prof_enable(True)
                for _ in range(reps):
                    dfl.dirac_apply(fld, x, storage=st, out=y, spinor_in=sp, spinor_out=sp)
                torch.cuda.synchronize()
                dfl.prof_enable(False)
                P = dfl.prof_get()["dirac"]
                ms = P["ms"] / reps
                row = {"lattice": "x".join(map(str, dims)), "storage": mode, "nrhs": n,
                       "ms": ms, "GB/s": P["bytes"] / (P["ms"] * 1e-3) / 1e9,
                       "Gflop/s": P["flops"] / (P["ms"] * 1e-3) / 1e9,
                       "frac_hbm": P["bytes"] / (P["ms"] * 1e-3) / 1e9 / PEAK_HBM_GBS}
                rows.append(row)
                log(json.dumps(row))
                del x, y
        fld.close()
    return rows


def run_exact16(args, log):
    """The 16^3 x 32 configuration: one point source (seeded site, spin-colour
    0) solved exactly (residual 1e-10; FP64 outer GCR, FP32 SAP on 4^4 blocks,
    deflation N_s = 12 on the same blocks), on the GPU and by the oracle on the
    host, each timed for its setup (field and deflation) and its solve; the
    two solutions are compared."""
    import torch
    import paper_1605_00564_amd as dfl
    import oracle
    dims, block, eps, kappa, csw = (32, 16, 16, 16), (4, 4, 4, 4), 0.4, 0.124, 1.5
    U = synth.gauge_field(dims, eps, 1)
    b = synth.point_source(dims, synth.seeded_site(dims, 1), 0)
    Ud, bd = torch.from_numpy(U).cuda(), torch.from_numpy(b[None]).cuda()
    sap = dfl.SapParams(5, 4, F32)
    rows = []
    for rep in range(args.warmup + args.steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        fld = dfl.Field(dims, block, kappa, csw, Ud)
        d = dfl.Deflation(fld, Ns=12, ninv=5, seed=7, sap=sap)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        p = dfl.GcrParams(nkv=16, nmx=300, res=1e-10, sap=sap, dfl=d, little_tol=1e-10, little_maxit=16)
        x, info = dfl.gcr_solve(fld, bd, p)
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        if rep >= args.warmup:
            rows.append((t1 - t0, t2 - t1, info[0]))
        xg = x.cpu().numpy()[0]
        d.close()
        fld.close()
    log(f"[exact16] GPU setup {rows[-1][0]:.3f} s, solve {rows[-1][1]:.3f} s, {rows[-1][2]}")
    result = {
        "metric": "exact deflated solve of one point source at 16^3x32 (residual 1e-10)",
        "value": float(np.mean([r[1] for r in rows])), "unit": "s/solve", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": 1000 * float(np.mean([r[0] + r[1] for r in rows])),
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "exact-16c32", "lattice": "32x16x16x16", "block": list(block), "Ns": 12,
                   "ninv": 5, "res": 1e-10, "sap": "FP32, ncy 5, nmr 4", "outer": "FP64"},
        "setup_s": float(np.mean([r[0] for r in rows])), "iters": rows[-1][2].iters,
        "rel_res": rows[-1][2].rel_res,
    }
    if not args.no_cpu_baseline:
        log("[exact16] oracle on the host")
        threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
        t0 = time.perf_counter()
        op = oracle.Operator(dims, U, kappa, csw, -1)
        ref = oracle.Deflation(op, block, Ns=12, ninv=5, seed=7)
        t1 = time.perf_counter()
        xo, io = oracle.solve(op, b, block=block, dfl=ref, res=1e-10)
        t2 = time.perf_counter()
        err = float(np.linalg.norm(xg - xo) / np.linalg.norm(xo))
        log(f"[exact16] oracle setup {t1 - t0:.2f} s, solve {t2 - t1:.2f} s; GPU vs oracle solution {err:.2e}")
        result["cpu_baseline"] = {"value": t2 - t1, "unit": "s/solve", "cores": threads, "kind": "oracle",
                                  "sample": "the same solve in full (one point source, deflated, to 1e-10); "
                                            f"its setup (clover, inverse, deflation subspace) took {t1 - t0:.2f} s",
                                  "setup_s": t1 - t0}
        result["gpu_vs_oracle_solution"] = err
    return result


# spin matrices in the library's chiral basis: gamma_0 couples the upper and
# lower spin pairs with -1; P+ = (1 + gamma_0)/2 projects the forward-moving
# nucleon (section 2.3)
GAMMA0 = np.array([[0, 0, -1, 0], [0, 0, 0, -1], [-1, 0, 0, 0], [0, -1, 0, 0]], dtype=np.complex128)
P_PLUS = 0.5 * (np.eye(4) + GAMMA0)
P_MINUS = 0.5 * (np.eye(4) - GAMMA0)


def _event_ms(fn, reps):
    """Average HIP-event time of fn() on torch's current stream (the library
    launches on it)."""
    import torch
    fn()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        fn()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / reps


def post_solve(fld, prop, t0, log, ape=(0.5, 20), gauss=(3.0, 30)):
    """Time the steps after the solve (section 2.3) on one exact point-source
    propagator prop [12, V, 4, 3] (complex128): APE smearing of the spatial
    links, Gaussian smearing of the 12 vectors, the nucleon two-point
    contraction, the forward (P+, t0 + T/4) and backward (P-, t0 - T/4)
    sequential sources of both flavours, the three-point contraction (with
    the sequential sources standing in for sequential propagators: the
    kernel's work does not depend on the values) and the AMA combination of
    32 approximate and 1 exact two-point function.  Smearing parameters are
    inputs (the paper takes them from earlier work).  Algorithmic bytes per
    launch: APE step 6 x 144 B per site (3 spatial FP64 links read and
    written); Gauss step 12 x 2 x 192 B + 3 x 144 B per site; two-point 2304
    B per site; sequential sources 2304 B per sink-timeslice site read and
    2304 B per site written; three-point 2 x 2304 B per site.  Each entry
    carries a roofline: HBM for the streaming kernels, FP64 ALU for the
    two-point contraction (28 800 flop per site)."""
    import torch
    import paper_1605_00564_amd as dfl
    V, T = fld.V, fld.dims[0]
    L3 = V // T
    out = {}

    def rec(name, ms, nbytes, flops=None, **extra):
        gbs = nbytes / (ms * 1e-3) / 1e9
        out[name] = {"ms": ms, "GB/s": gbs, "frac_hbm": gbs / PEAK_HBM_GBS, "bytes": nbytes, **extra}
        if flops is None:
            out[name]["roofline"] = {"bound": "hbm", "achieved": gbs, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                                     "frac": gbs / PEAK_HBM_GBS}
        else:
            tf = flops / (ms * 1e-3) / 1e12
            out[name]["roofline"] = {"bound": "alu", "achieved": tf, "peak": PEAK_FP64_TFLOPS, "unit": "TFLOP/s",
                                     "frac": tf / PEAK_FP64_TFLOPS, "flops": flops}
        log(f"[post] {name}: {ms:.3f} ms, {gbs:.0f} GB/s algorithmic")

    alpha, n_ape = ape
    ms = _event_ms(lambda: fld.ape_smear(alpha, n_ape), 2)
    rec("ape_smear", ms / n_ape, 6 * 144 * V, alpha=alpha, iterations=n_ape, per="iteration")
    kg, n_g = gauss
    sm = torch.empty_like(prop)
    ms = _event_ms(lambda: dfl.gauss_smear(fld, prop, kg, n_g, out=sm), 2)
    rec("gauss_smear", ms / n_g, (12 * 2 * 192 + 3 * 144) * V, kappa=kg, iterations=n_g, per="iteration, 12 vectors")
    ms = _event_ms(lambda: dfl.nucleon_2pt(fld, sm, t0), 5)
    # FP64 arithmetic, 3024 complex multiply-adds per site (through diquarks)
    rec("nucleon_2pt", ms, 2304 * V, flops=24192.0 * V)
    for flav in ("u", "d"):
        for tag, ts, P in (("forward", (t0 + T // 4) % T, P_PLUS), ("backward", (t0 - T // 4) % T, P_MINUS)):
            ms = _event_ms(lambda: dfl.nucleon_seq_sources(fld, sm, ts, P, flav), 5)
            rec(f"nucleon_seq_{flav}_{tag}", ms, 2304 * L3 + 2304 * V)
    seq = dfl.nucleon_seq_sources(fld, sm, (t0 + T // 4) % T, P_PLUS, "u")
    ms = _event_ms(lambda: dfl.nucleon_3pt(fld, seq, prop, t0, np.eye(4)), 5)
    rec("nucleon_3pt", ms, 2 * 2304 * V)
    g = torch.randn((32, T, 4, 4), dtype=torch.complex128, device="cuda")
    e = torch.randn((1, T, 4, 4), dtype=torch.complex128, device="cuda")
    ms = _event_ms(lambda: dfl.ama_combine(g, e, e), 5)
    rec("ama_combine", ms, (32 + 2) * T * 16 * 16)
    del seq, sm, g, e
    return out


def post_solve_oracle(work, log, ape=(0.5, 20), gauss=(3.0, 30)):
    """The oracle's versions of the steps after the solve (FP64 numpy) timed
    on the host on a bounded sample, an 8^4 lattice with the workload's
    field recipe, and scaled per site to the workload's lattice: two-point
    and three-point contractions and the APE and Gauss steps per site, the
    sequential sources per sink-timeslice site."""
    import oracle
    from oracle import nucleon as nuc, smear
    dims = (8, 8, 8, 8)
    Vs = synth.volume(dims)
    V = synth.volume(work["dims"])
    L3 = V // work["dims"][0]
    prop = synth.gaussian_spinor(dims, 12, 5)
    U = synth.gauge_field(dims, work["eps"], work["seed"])
    g, _ = oracle.gamma_matrices()
    Pp, _ = nuc.parity_projectors()
    out = {}

    def timed(fn):
        t = time.perf_counter()
        r = fn()
        return time.perf_counter() - t, r

    t, Us = timed(lambda: smear.ape_smear(dims, U, ape[0], 2))
    out["ape_smear"] = 1e3 * t / 2 / Vs * V
    t, _ = timed(lambda: smear.gauss_smear(dims, Us, prop, gauss[0], 2))
    out["gauss_smear"] = 1e3 * t / 2 / Vs * V
    t, _ = timed(lambda: nuc.nucleon_2pt(prop, dims, 0))
    out["nucleon_2pt"] = 1e3 * t / Vs * V
    t, seq = timed(lambda: nuc.nucleon_seq_sources(prop, dims, 2, Pp, "u"))
    out["nucleon_seq_u_forward"] = 1e3 * t / (Vs // dims[0]) * L3
    t, _ = timed(lambda: nuc.nucleon_3pt(seq, prop, dims, 0, g[3] @ g[4]))
    out["nucleon_3pt"] = 1e3 * t / Vs * V
    threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    log("[post] oracle, scaled to the workload: " + ", ".join(f"{k} {v:.0f} ms" for k, v in out.items()))
    return {"ms_scaled": out, "kind": "oracle", "cores": threads,
            "sample": "8^4 lattice (same field recipe), one call each (APE and Gauss: 2 steps), scaled per site "
                      "(sequential sources per sink-timeslice site) to the workload; per APE / Gauss step"}


def run_config3(args, log):
    """48^3 x 96, eps 0.4, kappa 0.1245, c_sw 1.5; 6^4 Schwarz and deflation
    blocks, N_s = 20; sloppy solves with BF16 link/clover storage, FP16 Schwarz
    vectors and FP32 arithmetic (3e-3), exact solves FP64 outer (1e-10).  One step: field
    preparation, deflation setup, the 12 point sources of one position
    (sloppy and exact), the 12 nucleon sequential sources (u line, P+, sink
    at t0 + 16) built on the device from the exact propagator, and their
    sloppy and exact solves.  value = step time / 2 source sets; the FP64
    residual of every solution is reported."""
    import torch
    import paper_1605_00564_amd as dfl
    dims, block = (96, 48, 48, 48), (6, 6, 6, 6)
    kappa, csw = 0.1245, 1.5
    t = time.perf_counter()
    U = synth.gauge_field(dims, 0.4, 1, progress=lambda f: log(f"[config3] gauge field {100 * f:.0f}%"))
    Ud = torch.from_numpy(U).cuda()
    del U
    log(f"[config3] gauge field generated in {time.perf_counter() - t:.1f} s")
    x0 = synth.seeded_site(dims, 1)
    pos = tuple(int(v) for v in synth.coords(dims, x0))
    t_sink = (pos[0] + 16) % dims[0]
    sap_s, sap_e = dfl.SapParams(5, 4, BF16, F16), dfl.SapParams(5, 4, F32)
    res = {}

    def step():
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        fld = dfl.Field(dims, block, kappa, csw, Ud)
        d = dfl.Deflation(fld, Ns=20, ninv=5, seed=7, sap=sap_s)
        sloppy = dfl.GcrParams(nkv=8, nmx=30, res=3e-3, sap=sap_s, dfl=d, little_tol=1e-6, little_maxit=4)
        exact = dfl.GcrParams(nkv=16, nmx=400, res=1e-10, sap=sap_e, dfl=d, little_tol=1e-10, little_maxit=16)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        xs, xe, i_ps, i_pe = dfl.ama_solve(fld, [dfl.point(pos)], [True], sloppy, exact, dtype=torch.complex128,
                                           sloppy_dtype=torch.complex64, batch=args.batch)
        # the solver's work buffers took what the batch could use; free them
        # before the next set's sources and outputs are allocated
        fld.trim()
        dfl.workspace_trim()
        eta = dfl.nucleon_seq_sources(fld, xe[0], t_sink, P_PLUS, "u")
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        ys, ye, i_qs, i_qe = dfl.ama_solve(fld, [dfl.vectors(eta)], [True], sloppy, exact, dtype=torch.complex128,
                                           sloppy_dtype=torch.complex64, batch=args.batch)
        torch.cuda.synchronize()
        t3 = time.perf_counter()
        res.update(point=(i_ps, i_pe), seq=(i_qs, i_qe), phases={"setup": t1 - t0, "point_set": t2 - t1,
                                                                  "sequential_set": t3 - t2, "total": t3 - t0})
        del xs, xe, ys, ye, eta
        d.close()
        fld.close()
        # every step starts from the same memory state
        torch.cuda.empty_cache()
        dfl.workspace_trim()
        return t3 - t0

    for w in range(args.warmup):
        log(f"[config3] warmup {w}: {step():.2f} s")
    tt = [step() for _ in range(args.steps)]
    for k, v in enumerate(tt):
        log(f"[config3] step {k}: {v:.2f} s")
    rr = lambda infos: [float(i.rel_res) for i in infos]
    i_ps, i_pe = res["point"]
    i_qs, i_qe = res["seq"]
    return {
        "metric": "AMA solve s/source-set at 48^3x96 (point + nucleon sequential sets, mixed precision)",
        "value": float(np.mean(tt)) / 2, "unit": "s/source", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": 1000 * float(np.mean(tt)), "higher_is_better": False,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "config3-48c96", "lattice": "96x48x48x48", "block": list(block), "Ns": 20,
                   "sloppy_storage": "bf16", "sloppy_res": 3e-3, "exact_res": 1e-10, "sets": 2,
                   "rhs_per_set": 12, "t_sink": "t0+16"},
        "phases_s": res["phases"],
        "iters": {"point_sloppy": sorted({i.iters for i in i_ps}), "point_exact": sorted({i.iters for i in i_pe}),
                  "seq_sloppy": sorted({i.iters for i in i_qs}), "seq_exact": sorted({i.iters for i in i_qe})},
        "fp64_rel_res": {"point_sloppy": rr(i_ps), "point_exact": rr(i_pe), "seq_sloppy": rr(i_qs),
                         "seq_exact": rr(i_qe)},
        "all_converged": all(i.status == 0 for i in i_ps + i_pe + i_qs + i_qe),
    }


# the uneven multi-field batch: (lattice T,X,Y,Z; gauge seed; sources)
MULTI_FIELDS = [((48, 24, 24, 24), 1, 8), ((64, 32, 32, 32), 2, 32), ((96, 48, 48, 48), 3, 64)]


def run_multi(args, log):
    """Three gauge fields with 8, 32 and 64 sources: half of them Z2 noise
    vectors built on the device, the other half point sources (whole
    positions of 12 spin-colours, so 1, 2 and 3 positions, two Schwarz
    blocks apart along t so that the set stays covariant); the first
    position of each field is also solved exactly (1e-10).  Per field the
    autotuner picks the Schwarz/deflation block shape, the right-hand sides
    per launch, the outer iteration count N_iter and the stencil variant
    (from the second field on it times only the two shapes the earlier
    fields ranked best per site).  Then one ama_solve_multi call solves every
    set of every field: sloppy solves at the tuned N_iter replayed from
    captured graphs, a solution still above 3e-3 solved again with the
    residual-stopping solver.  Timed: tuning (which builds the chosen
    handles) and the one library call; the host-side generation of the gauge
    fields is not timed."""
    import torch
    import paper_1605_00564_amd as dfl
    from paper_1605_00564_amd import tune
    prior = None
    fields, sets, rows = [], [], []
    t_tune = 0.0
    for dims, seed, nsrc in MULTI_FIELDS:
        t = time.perf_counter()
        U = synth.gauge_field(dims, 0.4, seed, progress=lambda f: log(f"[multi] {dims}: gauge field {100 * f:.0f}%"))
        Ud = torch.from_numpy(U).cuda()
        del U
        log(f"[multi] {dims}: gauge field generated in {time.perf_counter() - t:.1f} s")
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        # the smaller fields' tuning ranks the block shapes for the next one
        choice, fld, d = tune.tune_solver(dims, Ud, 0.124, 1.5, nsrc, fixed_iters=3, prior=prior, log=log)
        prior = (prior or []) + choice.table
        fld.trim()
        torch.cuda.synchronize()
        t_tune += time.perf_counter() - t0
        del Ud
        torch.cuda.empty_cache()
        sloppy = tune.sloppy_params(d, choice.fixed_iters)
        exact = dfl.GcrParams(nkv=16, nmx=400, res=1e-10, sap=dfl.SapParams(5, 4, F32), dfl=d, little_tol=1e-10,
                              little_maxit=16)
        # positions of one set differ by shifts that map the Schwarz block
        # checkerboard onto itself: two blocks along t per position
        npts = -(-(nsrc // 2) // 12)
        x0 = tuple(int(v) for v in synth.coords(dims, synth.seeded_site(dims, 1000 * seed)))
        pts = [((x0[0] + 2 * choice.block[0] * k) % dims[0],) + x0[1:] for k in range(npts)]
        srcs = [dfl.z2(seed=seed, index=0, nvec=nsrc // 2)] + [dfl.point(p) for p in pts]
        fields.append((fld, d))
        sets.append(dict(sources=srcs, exact_flags=[False, True] + [False] * (npts - 1), sloppy=sloppy, exact=exact,
                         batch=choice.batch))
        rows.append({"lattice": "x".join(map(str, dims)), "z2_vectors": nsrc // 2, "point_positions": npts,
                     "sloppy_rhs": nsrc // 2 + 12 * npts, "exact_rhs": 12, "block": list(choice.block),
                     "batch": choice.batch, "fixed_iters": choice.fixed_iters,
                     "stencil_variant": list(choice.stencil), "tune_s": time.perf_counter() - t0,
                     "tuning_table": choice.table})
        log(f"[multi] {dims}: tuned in {rows[-1]['tune_s']:.2f} s: block {choice.block}, batch {choice.batch}, "
            f"N_iter {choice.fixed_iters}")
    dfl.workspace_trim()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    out = dfl.ama_solve_multi([f for f, _ in fields], sets, dtype=torch.complex128, sloppy_dtype=torch.complex64)
    torch.cuda.synchronize()
    t_solve = time.perf_counter() - t1
    log(f"[multi] one ama_solve_multi call: {t_solve:.2f} s")
    for row, (xs, xe, i_s, i_e), st in zip(rows, out, sets):
        n_iter = row["fixed_iters"]
        row.update(sloppy_resolved=sum(1 for i in i_s if i.iters > n_iter),
                   sloppy_max_rel_res=max(i.rel_res for i in i_s), exact_max_rel_res=max(i.rel_res for i in i_e),
                   exact_iters=max(i.iters for i in i_e),
                   converged=all(i.status == 0 for i in i_s + i_e))
        log(f"[multi] {row['lattice']}: sloppy residual <= {row['sloppy_max_rel_res']:.2e} "
            f"({row['sloppy_resolved']} solved again), exact <= {row['exact_max_rel_res']:.2e}")
    del out
    for f, d in fields:
        d.close()
        f.close()
    total_rhs = sum(r["sloppy_rhs"] for r in rows)
    total_s = t_tune + t_solve
    return {
        "metric": f"uneven multi-field AMA batch (3 fields, {total_rhs} sloppy rhs): s/source incl. tuning",
        "value": total_s / total_rhs, "unit": "s/source", "n_gpus": 1, "steps": 1, "warmup": 0,
        "ms_per_step": 1000 * total_s, "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": "multi", "fields": [r["lattice"] for r in rows], "sources": [8, 32, 64],
                   "sloppy": "tuned fixed N_iter, graph replay, residual 3e-3", "exact_res": 1e-10,
                   "library_calls": 1},
        "tune_s": t_tune, "solve_s": t_solve, "fields": rows,
    }


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--stencil-sweep", action="store_true",
                    help="only measure the Dirac stencil over storage modes and rhs counts")
    ap.add_argument("--sweep-lattices", default="32x16x16x16,64x32x32x32", help="T x X x Y x Z, comma separated")
    ap.add_argument("--sweep-storage", default="f64,f32,f16,bf16,f16s,bf16s",
                    help="modes: " + ",".join(STENCIL_MODES))
    ap.add_argument("--sweep-nrhs", default="1,4,12,24")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run five 1 GiB device copies (reference for hardware byte counters)")
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="ama-32c64", choices=sorted(WORKLOADS) + ["multi", "exact-16c32", "config3-48c96"])
    ap.add_argument("--block", default="4,4,4,4")
    ap.add_argument("--ns", type=int, default=12)
    ap.add_argument("--ninv", type=int, default=5)
    ap.add_argument("--dfl-block", default="", help="deflation block t,x,y,z (default: the Schwarz block)")
    ap.add_argument("--nref", type=int, default=0,
                    help="rounds of inverse iteration with the deflated solver refining the subspace")
    ap.add_argument("--ref-res", type=float, default=1e-2, help="residual of the refinement solves")
    ap.add_argument("--no-deflation", action="store_true")
    ap.add_argument("--sweep-block-ns", default="",
                    help="one AMA step per block shape and N_s, e.g. '4,4,4,4:8,12,20;8,4,4,4:8,12,20'")
    ap.add_argument("--sloppy-storage", type=int, default=F16)
    ap.add_argument("--sloppy-vecs", type=int, default=None,
                    help="storage of the sloppy Schwarz sweeps' own vectors (2 = FP16, 1 = FP32; default FP16 "
                         "with FP16/BF16 link storage, else FP32)")
    ap.add_argument("--batch", type=int, default=24, help="right-hand sides per solver launch (0: from free memory)")
    ap.add_argument("--little-maxit", type=int, default=16,
                    help="little-solve iterations inside P_R for the exact solves")
    ap.add_argument("--little-maxit-sloppy", type=int, default=4,
                    help="little-solve iterations inside P_R for the sloppy solves")
    ap.add_argument("--chunk", type=int, default=4, help="source positions per ama_solve call")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-fp64", action="store_true", help="skip the FP64 single-rhs comparator")
    ap.add_argument("--sloppy-fixed-iters", type=int, default=0,
                    help="timed steps: sloppy solves at this fixed outer iteration count, replayed from captured "
                         "graphs (misses above 3e-3 solved again); 0 = stop on the residual")
    ap.add_argument("--no-graph-variant", action="store_true",
                    help="skip the extra step with graph-replayed fixed-iteration sloppy solves")
    ap.add_argument("--no-post", action="store_true", help="skip timing the steps after the solve")
    ap.add_argument("--json-only", action="store_true")
    args = ap.parse_args()

    if args.gpus != 1:
        print(f"bench.py runs on one GPU: the solve is measured on a single MI355X; --gpus {args.gpus} "
              "is not supported (multi-GPU sharding is a design note only).", file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_1605_00564_amd as dfl

    log = (lambda *a: None) if args.json_only else (lambda *a: print(*a, file=sys.stderr, flush=True))
    if args.copy_calibration:
        # a plain device copy of known size, to scale the HBM byte counters
        nbytes = 1 << 30
        a = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda").fill_(1.0)
        b = torch.empty_like(a)
        torch.mul(a, 1.0, out=b)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(5):
            torch.mul(a, 1.0, out=b)    # one elementwise kernel: reads a, writes b
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / 5
        print(json.dumps({"copy_calibration_bytes_each_way": nbytes, "copies": 5, "ms_per_copy": ms,
                          "GB/s": 2 * nbytes / (ms * 1e-3) / 1e9}), flush=True)
        return
    if args.workload == "multi":
        print(json.dumps(run_multi(args, log)), flush=True)
        return
    if args.workload == "exact-16c32":
        print(json.dumps(run_exact16(args, log)), flush=True)
        return
    if args.workload == "config3-48c96":
        print(json.dumps(run_config3(args, log)), flush=True)
        return
    if args.stencil_sweep:
        lats = [tuple(int(v) for v in s.split("x")) for s in args.sweep_lattices.split(",")]
        rows = stencil_sweep(lats, args.sweep_storage.split(","),
                             [int(v) for v in args.sweep_nrhs.split(",")], 10, log, cpu=not args.no_cpu_baseline)
        print(json.dumps({"stencil_sweep": rows}), flush=True)
        return
    work = WORKLOADS[args.workload]
    dims = work["dims"]
    block = tuple(int(b) for b in args.block.split(","))
    dblock = tuple(int(b) for b in args.dfl_block.split(",")) if args.dfl_block else None
    V = synth.volume(dims)
    pos = positions(work, block)
    npos = len(pos)
    exact_flags = [i == 0 for i in range(npos)]
    log(f"[bench] workload {args.workload} dims {dims} block {block} positions {npos}")

    t = time.perf_counter()
    U = synth.gauge_field(dims, work["eps"], work["seed"])
    Ud = torch.from_numpy(U).cuda()
    del U
    log(f"[bench] gauge field generated and uploaded in {time.perf_counter() - t:.1f} s")

    if args.sloppy_vecs is None:
        args.sloppy_vecs = F16 if args.sloppy_storage in (F16, BF16) else F32
    sap_sloppy = dfl.SapParams(5, 4, args.sloppy_storage, args.sloppy_vecs)
    sap_exact = dfl.SapParams(5, 4, F32)
    # sloppy solutions stored in FP32, exact ones in FP64
    xs = [torch.empty((12, V, 4, 3), dtype=torch.complex64, device="cuda") for _ in range(npos)]
    xe = [torch.empty((12, V, 4, 3), dtype=torch.complex128, device="cuda")]

    state = {}

    def step(block=block, ns=args.ns, pos=pos, fixed=args.sloppy_fixed_iters):
        ph = {}
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        fld = dfl.Field(dims, block, work["kappa"], work["csw"], Ud)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        d = None
        if not args.no_deflation:
            d = dfl.Deflation(fld, Ns=ns, ninv=args.ninv, seed=7, sap=sap_sloppy,
                              block=dblock, nref=args.nref, ref_res=args.ref_res)
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        # fixed > 0: truncated solves of `fixed` iterations from captured
        # graphs; a miss above 3e-3 is solved again on the residual
        sloppy = dfl.GcrParams(nkv=8, nmx=24, res=3e-3, sap=sap_sloppy, dfl=d, little_tol=1e-6,
                               little_maxit=args.little_maxit_sloppy, fixed_iters=fixed)
        exact = dfl.GcrParams(nkv=16, nmx=400, res=1e-10, sap=sap_exact, dfl=d, little_tol=1e-10,
                              little_maxit=args.little_maxit)
        infs, infe = [], []
        for c0 in range(0, npos, args.chunk):
            c1 = min(npos, c0 + args.chunk)
            ex = exact_flags[c0:c1]
            _, _, i_s, i_e = dfl.ama_solve(fld, pos[c0:c1], ex, sloppy, exact, dtype=torch.complex128,
                                           sloppy_dtype=torch.complex64, batch=args.batch,
                                           out_sloppy=xs[c0:c1], out_exact=xe if any(ex) else [])
            infs += i_s
            infe += i_e
            log(f"[bench]   positions {c0}..{c1 - 1} done at {time.perf_counter() - t2:.1f} s")
        torch.cuda.synchronize()
        t3 = time.perf_counter()
        ph.update(field=t1 - t0, deflation=t2 - t1, solves=t3 - t2, total=t3 - t0)
        state.update(infs=infs, infe=infe, fld=fld, dfl=d)
        return ph

    for w in range(args.warmup):
        ph = step()
        log(f"[bench] warmup {w}: {ph}")
        state.pop("dfl", None)
        state.pop("fld", None)

    if args.sweep_block_ns:
        # one AMA step per (block shape, N_s) on the same gauge field
        rows = []
        for bs in args.sweep_block_ns.split(";"):
            b_txt, ns_txt = bs.split(":")
            b = tuple(int(v) for v in b_txt.split(","))
            for ns in (int(v) for v in ns_txt.split(",")):
                ph = step(block=b, ns=ns, pos=positions(work, b))
                infs, infe = state.pop("infs"), state.pop("infe")
                state.pop("dfl", None)
                state.pop("fld", None)
                row = {"block": list(b), "Ns": ns, "s_per_source": ph["total"] / npos,
                       "setup_s": ph["field"] + ph["deflation"], "solves_s": ph["solves"],
                       "sloppy_iters": [min(i.iters for i in infs), max(i.iters for i in infs)],
                       "exact_iters": [min(i.iters for i in infe), max(i.iters for i in infe)],
                       "sloppy_max_rel_res": max(i.rel_res for i in infs),
                       "exact_max_rel_res": max(i.rel_res for i in infe)}
                rows.append(row)
                log("[sweep] " + json.dumps(row))
        print(json.dumps({"block_ns_sweep": rows, "workload": args.workload, "positions": npos}), flush=True)
        return

    dfl.prof_reset()
    dfl.prof_enable(True)
    torch.cuda.synchronize()
    phases = []
    t_start = time.perf_counter()
    for k in range(args.steps):
        phases.append(step())
        log(f"[bench] step {k}: {phases[-1]}")
        if k + 1 < args.steps:
            state.pop("dfl", None)
            state.pop("fld", None)
    torch.cuda.synchronize()
    t_total = time.perf_counter() - t_start
    dfl.prof_enable(False)
    prof = dfl.prof_get()
    ms_per_step = 1000.0 * t_total / args.steps
    s_per_source = t_total / args.steps / npos

    # dominant kernel class
    dom = max(prof, key=lambda c: prof[c]["ms"])
    P = prof[dom]
    avg_ms = P["ms"] / max(P["launches"], 1)
    if dom == "sap":
        per_launch = P["flops"] / max(P["launches"], 1)
        achieved = per_launch / (avg_ms * 1e-3) / 1e12
        # against the published FP32 vector peak (packed FP32); the ceiling
        # without packed instructions, which this build does not emit, is
        # reported beside it
        roof = {"bound": "alu", "achieved": achieved, "peak": PEAK_FP32_TFLOPS, "unit": "TFLOP/s",
                "frac": achieved / PEAK_FP32_TFLOPS, "traffic": None,
                "frac_of_unpacked_peak": achieved / PEAK_FP32_UNPACKED_TFLOPS}
    else:
        per_launch = P["bytes"] / max(P["launches"], 1)
        achieved = per_launch / (avg_ms * 1e-3) / 1e9
        roof = {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                "frac": achieved / PEAK_HBM_GBS, "traffic": None}
    roof["kernel"] = {"sap": "k_sap_sweep", "dirac": "k_dirac", "blas": "vector algebra"}.get(dom, dom)
    roof["traffic"] = measured_traffic(roof["kernel"], args.workload)
    roof["traffic_unit"] = "bytes per launch"
    roof["avg_launch_ms"] = avg_ms
    roof["launches"] = P["launches"]
    # stencil figures (the Dirac-operator half of the metric)
    Pd = prof["dirac"]
    stencil = None
    if Pd["launches"]:
        dms = Pd["ms"] / Pd["launches"]
        stencil = {"bound": "hbm", "achieved": Pd["bytes"] / Pd["launches"] / (dms * 1e-3) / 1e9,
                   "peak": PEAK_HBM_GBS, "unit": "GB/s", "gflops": Pd["flops"] / (Pd["ms"] * 1e-3) / 1e9,
                   "avg_launch_ms": dms, "launches": Pd["launches"]}
        stencil["frac"] = stencil["achieved"] / PEAK_HBM_GBS
        stencil["traffic"] = measured_traffic("k_dirac", args.workload)
        stencil["traffic_unit"] = "bytes per launch"

    infs, infe = state["infs"], state["infe"]
    result = {
        "metric": "AMA solve s/source at 32^3x64 (mixed precision); Dirac-op HBM GB/s vs peak",
        "value": s_per_source,
        "unit": "s/source",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": args.workload, "lattice": "x".join(str(d) for d in dims), "block": list(block),
                   "Ns": 0 if args.no_deflation else args.ns, "positions": npos,
                   "deflation_block": list(dblock or block), "nref": args.nref, "sloppy_rhs": 12 * npos,
                   "exact_rhs": 12, "sloppy_res": 3e-3, "exact_res": 1e-10,
                   "sloppy_storage": ["f64", "f32", "f16", "bf16"][args.sloppy_storage],
                   "sloppy_sap_vectors": ["f64", "f32", "f16", "bf16"][args.sloppy_vecs], "ncy": 5, "nmr": 4,
                   "little_maxit": {"sloppy": args.little_maxit_sloppy, "exact": args.little_maxit}},
        "roofline": roof,
        "stencil_roofline": stencil,
        "phases_s": {k: float(np.mean([p[k] for p in phases])) for k in phases[0]},
        "kernel_ms": {c: prof[c]["ms"] / args.steps for c in prof},
        "sloppy_iters": [int(min(i.iters for i in infs)), int(max(i.iters for i in infs))],
        "sloppy_max_rel_res": float(max(i.rel_res for i in infs)),
        "exact_iters": [int(min(i.iters for i in infe)), int(max(i.iters for i in infe))],
        "exact_max_rel_res": float(max(i.rel_res for i in infe)),
    }
    if not args.no_graph_variant and args.sloppy_fixed_iters == 0:
        # the same step with truncated sloppy solves replayed from captured
        # graphs (no host decision per iteration) at the iteration count the
        # residual-stopping solves needed
        n_it = result["sloppy_iters"][1]
        state.pop("dfl", None)
        state.pop("fld", None)
        log(f"[bench] graph-replay variant, sloppy N_iter = {n_it}")
        step(fixed=n_it)                       # warm-up: allocations at this setting
        state.pop("dfl", None)
        state.pop("fld", None)
        torch.cuda.synchronize()
        tg = time.perf_counter()
        phg = step(fixed=n_it)
        tg = time.perf_counter() - tg
        ig = state["infs"]
        result["graph_replay"] = {
            "s_per_source": tg / npos, "sloppy_fixed_iters": n_it, "phases_s": phg,
            "sloppy_solved_again": sum(1 for i in ig if i.iters > n_it),
            "sloppy_max_rel_res": float(max(i.rel_res for i in ig)),
            "exact_max_rel_res": float(max(i.rel_res for i in state["infe"])),
            "note": "one step (new handles, graphs captured on the first batch of each size within the step)"}
        log(f"[bench] graph replay: {tg / npos:.4f} s/source, residual <= {result['graph_replay']['sloppy_max_rel_res']:.2e}")
    if not args.no_post:
        log("[bench] steps after the solve")
        result["post_solve"] = post_solve(state["fld"], xe[0], pos[0][0], log)
        result["post_solve"]["workload"] = (f"{result['config']['lattice']}: the exact propagator of the first "
                                            "position; APE 0.5 x 20, Gauss kappa 3.0 x 30")
    if not args.no_fp64:
        log("[bench] FP64 single-rhs comparator")
        ph = result["phases_s"]
        f64 = fp64_single_rhs(state["fld"], state["dfl"], pos, npos, ph["field"] + ph["deflation"],
                              args.little_maxit, args.little_maxit_sloppy, log)
        f64["speedup_mixed"] = f64["value"] / s_per_source
        result["fp64_single_rhs"] = f64
    if not args.no_cpu_baseline:
        log("[bench] timing the oracle on the host")
        threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
        result["cpu_baseline"] = cpu_baseline(work, block, {c: prof[c] for c in prof}, npos * args.steps, 5, 4,
                                              threads)
        if "post_solve" in result:
            result["post_solve"]["oracle_cpu"] = post_solve_oracle(work, log)
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
