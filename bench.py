#!/usr/bin/env python3
"""Benchmark of the S-NFC thin-wire MoM hot path on one MI355X.

One step = the whole hot path over one batch of synthetic input:
neighbour search (chaff_build_cloud), impedance fill (chaff_fill_Z), the
preconditioner (chaff_nbhd_precond / chaff_cluster_precond as configured),
excitation + preconditioned Krylov solve with FP64 refinement (chaff_solve)
and monostatic RCS (chaff_rcs), with the inputs already resident in HBM.

    python bench.py [--steps K] [--warmup W] [--config c5] [--gpus 1]

Prints ONE JSON line.  `value` = solved (cloud, incidence) systems per
second over the K timed steps; a system counts as solved when its FP64 true
relative residual is <= tol (1e-6).  `roofline` is the dominant kernel of the
timed region: its algorithmic work (bytes or flops, computed by the library
from the exact sizes of each launch) over its HIP-event time measured on the
launch stream.  `cpu_baseline` is the FP64 oracle timed on a bounded sample
of the same workload on this host.
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

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, GB/s
FP32_PEAK_TFLOPS = 157.3       # MI355X FP32 vector (packed) peak, TFLOP/s
FP64_PEAK_TFLOPS = 78.6        # MI355X FP64 vector peak, TFLOP/s

# profile name -> (kernel symbol prefix in rocprofv3 output, source file), for complex64 COCG of many columns
# with 7 unknowns per wire, the workload that the counter records are of
KERNEL_SYMBOLS = {
    "spmm": ("chaff::kr7::k_cocg_mfma", "paper_2410_03060_amd/csrc/krylov_impl.hpp"),
    "k_cg_update": ("chaff::kr7::k_cg_update", "paper_2410_03060_amd/csrc/krylov_impl.hpp"),
    "k_cg_p": ("chaff::kr7::k_cg_p", "paper_2410_03060_amd/csrc/krylov_impl.hpp"),
    "fill_mutual": ("chaff::k_mutual", "paper_2410_03060_amd/csrc/fill.hip"),
    "fill_self": ("chaff::k_self", "paper_2410_03060_amd/csrc/fill.hip"),
    "rcs_mono": ("chaff::k_mono", "paper_2410_03060_amd/csrc/farfield.hip"),
    "cluster_build": ("chaff::k_cluster_build", "paper_2410_03060_amd/csrc/precond.hip"),
    "nbhd_apply": ("chaff::kr7::k_cocg_mfma", "paper_2410_03060_amd/csrc/krylov_impl.hpp"),
    "k_cg_rupd": ("chaff::kr7::k_cg_rupd", "paper_2410_03060_amd/csrc/krylov_impl.hpp"),
    "nbhd_build": ("chaff::k_nbhd_build", "paper_2410_03060_amd/csrc/precond.hip"),
}


def kernel_symbol(name, nb, c64, method, columns, cluster=False):
    """Symbol (prefix) of the kernel behind a profile name, for solves of `columns` right-hand sides with nb
    unknowns per wire: the product of a COCG step runs on the matrix cores (complex64, 7 unknowns), as a
    streaming row product (7 unknowns, up to 4 columns) or in the staged form."""
    space = f"chaff::kr{nb}::"
    if name in ("spmm", "spmm_narrow", "nbhd_apply", "nbhd_apply_narrow"):
        if method not in ("cocg", "cocg_rr"):
            return space + "k_spmm_"
        if nb == 7 and columns <= 4:
            return space + "k_cocg_stream"
        return space + ("k_cocg_mfma" if nb == 7 and c64 else "k_cocg_spmm")
    if name == "solve_small":
        return space + "small::k_solve_small"
    if name == "lone_solve":
        return space + ("k_lone_apply" if columns > 32 else "k_lone_solve")
    if cluster and name in ("k_cg_update", "k_cg_p"):   # the cluster path runs its own update and direction kernels
        return space + ("k_cg_update_cl" if name == "k_cg_update" else "k_cg_pdir_z")
    return KERNEL_SYMBOLS.get(name, (name,))[0].replace("chaff::kr7::", space)


TRAFFIC_FILE = os.path.join(ROOT, "profiles", "hbm_traffic.json")


def source_hash(rel: str):
    """First 16 hex digits of the source's SHA-256, or None if the file is gone."""
    import hashlib
    try:
        with open(os.path.join(ROOT, rel), "rb") as f:
            return hashlib.sha256(f.read()).hexdigest()[:16]
    except OSError:
        return None


def measured_traffic(config: str, kernel: str):
    """HBM bytes per launch from the committed FETCH_SIZE / WRITE_SIZE runs.

    Returns None unless the record matches this workload and the kernel's
    source file is unchanged since the counters were taken.
    """
    try:
        with open(TRAFFIC_FILE) as f:
            rec = json.load(f)
    except (OSError, ValueError):
        return None
    ent = rec.get(config, {}).get(kernel)
    if not ent or kernel not in KERNEL_SYMBOLS:
        return None
    if ent.get("source_sha256_16") != source_hash(KERNEL_SYMBOLS[kernel][1]):
        return None
    return ent["hbm_bytes_per_launch"]

MFMA_FILE = os.path.join(ROOT, "profiles", "mfma_counters.json")


def measured_mfma(config: str, kernel: str):
    """MFMA busy fraction and counted MFMA flop per launch from the committed counter run,
    or None unless the record matches this workload and the kernel source is unchanged."""
    try:
        with open(MFMA_FILE) as f:
            ent = json.load(f).get(config, {}).get(kernel)
    except (OSError, ValueError):
        return None
    if not ent or "source" not in ent or ent.get("source_sha256_16") != source_hash(ent["source"]):
        return None
    return ent


CONFIGS = {
    # prec: Krylov/fill precision; method: Krylov method per refinement cycle;
    # restart: GMRES cycle length or COCG step cap; inner_tol: reduction per cycle
    "c1": dict(prec="c128", method="gmres", restart=60, inner_tol=1e-4,
               desc="64 half-wave wires, 10-wavelength cube, d_c=2 lambda, 1 incidence, complex128"),
    "c2": dict(prec="c64", method="gmres", restart=30, inner_tol=1e-4,
               desc="2,000 wires, Gaussian sigma=15 lambda, d_c=1.5 lambda, 1 incidence, "
                    "complex64 + FP64 refinement"),
    "c3": dict(prec="c64", method="cocg", restart=2000, inner_tol=1e-5,
               desc="20,000-wire Gaussian cloud + 16 side clouds (500-5,000 wires), d_c=2 lambda, "
                    "360 azimuth incidences, one launch per stage for all 17 clouds"),
    "c4_eval": dict(prec="c64", method="cocg", restart=5000, inner_tol=1e-5, guess="bj", precond="nbhd", nbhd_size=4,
                    desc="100,000 wires, uniform sphere R=40 lambda, d_c=1.5 lambda, 8 incidences, "
                         "neighbourhood-inverse preconditioner (4 wires), initial guess M u; the learned "
                         "guess and the learned preconditioner are measured beside it"),
    "c5": dict(prec="c64", method="cocg", restart=5000, inner_tol=1e-5, guess="bj", precond="nbhd", nbhd_size=8,
               desc="1,000,000 wires (7M unknowns), uniform sphere R=50 lambda, d_c=1 lambda, "
                    "64 azimuth incidences, complex64 + FP64 refinement, neighbourhood-inverse "
                    "preconditioner (8 wires), initial guess M u; the learned guess and the learned "
                    "preconditioner are measured beside it"),
    "n2": dict(prec="c64", method="cocg", restart=2000, inner_tol=1e-5, guess="bj", precond="block",
               desc="the paper's 10^5-chaff case with its own discretisation: 19 unknowns per chaff "
                    "(1.9M unknowns), identical half-wave chaffs at 13 GHz, diameter 20 um, uniform "
                    "sphere at 119.37 chaffs/m^3 (radius 5.85 m), d_c=2 lambda, 64 azimuth incidences, "
                    "complex64 + FP64 refinement, block-diagonal preconditioner"),
}
GUESSES = {"zero": 0, "bj": 2, "mlp": 1}   # bj: x0 = P u with the solve's preconditioner P
PRECONDS = {"block": 0, "cluster": 1, "nbhd": 2, "nbhd_mlp": 2}   # nbhd_mlp: the learned neighbourhood inverse
NBHD_SIZE = 6   # wires per neighbourhood of the neighbourhood-inverse preconditioner (default)
# training recipe of the learned guess per evaluation workload: (generator, clouds, epochs)
MLP_TRAINING = {"c4_eval": ("c4_train_cloud", 200, 12), "c5": ("c5_train_cloud", 64, 12)}
# training recipe of the learned neighbourhood-inverse preconditioner: (generator, clouds, epochs)
NBHD_MLP_TRAINING = {"c4_eval": ("c4_train_cloud", 24, 6), "c5": ("c5_train_cloud", 16, 6)}
METHODS = {"gmres": 0, "cocg": 1, "cocg_rr": 2, "gcr": 3}


def make_workload(name):
    from paper_2410_03060_amd import workloads as W
    if name == "c1":
        return W.c1()
    if name == "c2":
        return W.c2()
    if name == "c3":
        return W.c3()
    if name == "c4_eval":
        return W.c4_eval()
    if name == "c5":
        return W.c5()
    if name == "n2":
        return W.n2()
    raise SystemExit(f"unknown config {name}")


def sub_sphere(cloud, n_keep):
    """The n_keep wires closest to the centroid of cloud 0 (same density)."""
    import numpy as np

    from paper_2410_03060_amd import workloads as W
    lo, hi = int(cloud.cloud_off[0]), int(cloud.cloud_off[1])
    c = cloud.center[lo:hi]
    d = np.linalg.norm(c - c.mean(axis=0), axis=1)
    idx = np.sort(np.argsort(d)[:n_keep]) + lo
    return W.single_cloud(cloud.center[idx], cloud.tangent[idx], cloud.length[idx], cloud.wavelength,
                          cloud.d_c, cloud.radius[idx], cloud.n_seg)


def cpu_baseline(wl, n_sample: int = 2000, r_sample: int = 8):
    """Oracle (FP64 CPU) on a bounded sample, scaled to the full workload.

    Sample: the n_sample wires of the first cloud nearest its centroid (same
    density) and the first r_sample incidences.  The oracle's setup (near
    set, Galerkin fill, SuperLU factorisation) and its per-incidence work
    (triangular solves + RCS) are timed separately and each is scaled by the
    wire ratio; the full workload then costs setup + R * per-incidence.
    """
    from oracle import mom, solve as osolve
    import scipy.sparse.linalg as spla
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] + [1])
    except Exception:
        threads = 1
    cloud = wl.cloud
    n_full = cloud.n
    R = wl.inc.k_hat.shape[0]
    n_s = int(min(cloud.cloud_off[1] - cloud.cloud_off[0], n_sample))
    sample = sub_sphere(cloud, n_s) if n_s < cloud.n else cloud
    r_s = min(R, r_sample)
    kh, eh = wl.inc.k_hat[:r_s], wl.inc.e_hat[:r_s]
    ph = {}
    t0 = time.perf_counter()
    pairs = mom.near_pairs(sample.center, sample.cloud_off, sample.d_c)
    ta = time.perf_counter()
    Zs, _ = mom.snfc_matrix(sample, n_seg=sample.n_seg, pairs=pairs)
    tb = time.perf_counter()
    lu = spla.splu(Zs.tocsc())
    t1 = time.perf_counter()
    u = mom.excitation(sample, kh, eh, sample.n_seg)
    tc = time.perf_counter()
    x = lu.solve(u)
    td = time.perf_counter()
    mom.monostatic_rcs(sample, x, kh, eh, sample.n_seg)
    t2 = time.perf_counter()
    ph = {"near_set": ta - t0, "fill": tb - ta, "factor": t1 - tb, "excitation": tc - t1, "solve": td - tc,
          "rcs": t2 - td}
    scale = n_full / sample.n
    t_full = (t1 - t0) * scale + (t2 - t1) / r_s * R * scale
    systems = cloud.n_clouds * R
    cpu_model = None
    try:
        with open("/proc/cpuinfo") as f:
            cpu_model = next((l.split(":", 1)[1].strip() for l in f if l.startswith("model name")), None)
    except OSError:
        pass
    try:
        affinity = len(os.sched_getaffinity(0))
    except (AttributeError, OSError):
        affinity = None
    return {"value": systems / t_full, "unit": "solved angles/s", "cores": int(threads), "kind": "oracle",
            "cpu_model": cpu_model, "cores_available": affinity,
            "sample_phase_seconds": {k: round(v, 4) for k, v in ph.items()},
            "sample": f"{sample.n} of {n_full} wires (first cloud, nearest its centroid) and {r_s} of {R} "
                      f"incidences: setup {t1 - t0:.2f} s + {r_s} incidences {t2 - t1:.2f} s, each scaled "
                      f"by the wire ratio {scale:.1f}; full workload estimated at {t_full:.1f} s"}


FLOPS_FILE = os.path.join(ROOT, "profiles", "valu_flops.json")


def executed_flop(config, kernel):
    """Executed FP32 flop per launch from the committed VALU counter record, if its source is unchanged."""
    try:
        with open(FLOPS_FILE) as f:
            ent = json.load(f).get(config, {}).get(kernel)
    except (OSError, ValueError):
        return None
    if not ent or ent.get("source_sha256_16") != source_hash(ent["source"]):
        return None
    return ent["executed_flop_per_launch"]


def fill_summary(prof, config=None):
    """Fill rate in the timed steps: algorithmic flop (24 per Green sample) over kernel time, and the
    executed FP32 flop counted by the VALU instruction counters (profiles/valu_flops.json) over the same time."""
    out = {}
    tot_w = tot_ms = 0.0
    for name in ("fill_mutual", "fill_self"):
        k = prof.get(name)
        if not k or k["total_ms"] <= 0:
            continue
        tf = k["flops"] / (k["total_ms"] * 1e-3) / 1e12
        ms = k["total_ms"] / k["launches"]
        out[name] = {"TFLOP/s": tf, "frac": tf / FP32_PEAK_TFLOPS, "ms_per_launch": ms}
        ex = executed_flop(config, name) if config else None
        if ex is not None:
            out[name]["executed_TFLOP/s"] = ex / (ms * 1e-3) / 1e12
            out[name]["executed_frac"] = out[name]["executed_TFLOP/s"] / FP32_PEAK_TFLOPS
        tot_w += k["flops"]
        tot_ms += k["total_ms"]
    if tot_ms > 0:
        tf = tot_w / (tot_ms * 1e-3) / 1e12
        out["combined"] = {"TFLOP/s": tf, "frac": tf / FP32_PEAK_TFLOPS, "GFLOP/s": tf * 1e3}
    return out


def roofline_of(k, matrix_cores: bool, fp64: bool = False):
    """Roofline of one kernel from its algorithmic bytes B and flops F per launch and its
    measured average launch time t: the bound is whichever of B / 8 TB/s and
    F / 157.3 TFLOP/s (fp64: 78.6) is longer; `achieved` is that resource's rate (B/t or F/t)
    and `frac` = achieved / peak (= bound time / t)."""
    sec = k["total_ms"] / 1e3 / k["launches"]
    b = k["bytes"] / k["launches"]
    f = k["flops"] / k["launches"]
    t_hbm = b / (HBM_PEAK_GBS * 1e9)
    peak = FP64_PEAK_TFLOPS if fp64 else FP32_PEAK_TFLOPS
    t_alu = f / (peak * 1e12)
    if t_alu > t_hbm:
        ach = f / sec / 1e12
        roof = {"bound": "mfma" if matrix_cores else "alu", "achieved": ach, "peak": peak,
                "unit": "TFLOP/s", "frac": ach / peak}
    else:
        ach = b / sec / 1e9
        roof = {"bound": "hbm", "achieved": ach, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": ach / HBM_PEAK_GBS}
    roof.update({"bytes_per_launch": b, "flops_per_launch": f,
                 "intensity_flop_per_byte": (f / b) if b > 0 else None,
                 "ridge_flop_per_byte": peak * 1e12 / (HBM_PEAK_GBS * 1e9),
                 "hbm_GB/s": b / sec / 1e9, "TFLOP/s": f / sec / 1e12})
    return roof


def train_guess(config, B):
    """Train the learned guess for this workload on clouds solved by the library (untimed)."""
    import numpy as np

    from paper_2410_03060_amd import learned, workloads as W
    gen, n_clouds, epochs = MLP_TRAINING[config]
    make = getattr(W, gen)
    samples = learned.solved_samples([make(j) for j in range(n_clouds)])
    print(f"[bench] mlp: {samples.feat.shape[0]} samples from {n_clouds} solved clouds in "
          f"{samples.solve_seconds:.1f} s", file=sys.stderr, flush=True)
    res = learned.train(samples, W.mlp_init(0), epochs=epochs, batch=4096, seed=0)
    err = learned.relative_target_error(res.theta, samples)
    print(f"[bench] mlp: {res.steps} Adam steps in {res.seconds:.1f} s, final epoch loss {res.losses[-1]:.4f}, "
          f"relative error of the predicted departure {err:.3f}", file=sys.stderr, flush=True)
    report = {"train_clouds": f"{gen}(0..{n_clouds - 1})", "samples": int(samples.feat.shape[0]),
              "data_seconds": samples.solve_seconds, "epochs": epochs, "batch": 4096, "adam_steps": res.steps,
              "train_seconds": res.seconds, "ms_per_adam_step": res.seconds / res.steps * 1e3,
              "epoch_losses": [round(x, 5) for x in res.losses], "train_relative_error": err,
              "excluded_from_timing": True}
    del samples
    return res.theta, report


def train_nbhd_mlp(config, size):
    """Train the learned neighbourhood-inverse preconditioner on raw rows computed by the library (untimed)."""
    from paper_2410_03060_amd import learned, workloads as W
    gen, n_clouds, epochs = NBHD_MLP_TRAINING[config]
    make = getattr(W, gen)
    samples = learned.nbhd_samples([make(j) for j in range(n_clouds)], size)
    print(f"[bench] nbhd mlp: {samples.feat.shape[0]} rows from {n_clouds} clouds in {samples.solve_seconds:.1f} s",
          file=sys.stderr, flush=True)
    res = learned.train(samples, W.mlp_init(0), epochs=epochs, batch=4096, seed=0)
    err = learned.relative_target_error(res.theta, samples)
    print(f"[bench] nbhd mlp: {res.steps} Adam steps in {res.seconds:.1f} s, final epoch loss {res.losses[-1]:.4f}, "
          f"relative error {err:.3f}", file=sys.stderr, flush=True)
    report = {"train_clouds": f"{gen}(0..{n_clouds - 1})", "rows": int(samples.feat.shape[0]),
              "data_seconds": samples.solve_seconds, "epochs": epochs, "batch": 4096, "adam_steps": res.steps,
              "train_seconds": res.seconds, "epoch_losses": [round(x, 5) for x in res.losses],
              "train_relative_error": err, "excluded_from_timing": True}
    del samples
    return res.theta, report


def spmm_sweep(B, geom, prec, sizes=(1, 4, 8, 16, 32, 64)):
    """Block-sparse product alone (chaff_spmm, autotuned per RHS count) on the
    workload's matrix: algorithmic bytes (Z once with its indices, X and Y
    once) over the best variant's time, against 8 TB/s; and flop rate."""
    cl = B.build_cloud(geom)
    Z, _ = B.fill_Z(cl, prec, with_pinv=False)
    zsz = 8 if prec == B.C64 else 16
    out = {}
    for s_ in sizes:
        best, ms = B.autotune(cl, Z, s_, prec)
        nb = cl.nb
        byt = (zsz * nb * nb + 4.0) * cl.nnzb + 4.0 * (cl.n + 1) + 2.0 * zsz * nb * cl.n * s_
        fl = 8.0 * nb * nb * cl.nnzb * s_
        row = [e for e in B.tune_report() if e["n"] == cl.n and e["nnzb"] == cl.nnzb and e["s"] == s_]
        t_bound = max(byt / (HBM_PEAK_GBS * 1e9), fl / (FP32_PEAK_TFLOPS * 1e12))
        out[f"s={s_}"] = {"variant": best, "ms": ms, "GB/s": byt / (ms * 1e-3) / 1e9,
                          "variant_ms": row[0]["ms"] if row else None,
                          "frac_hbm": byt / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                          "TFLOP/s": fl / (ms * 1e-3) / 1e12,
                          "frac_roofline": t_bound / (ms * 1e-3)}
        print(f"[bench] spmm s={s_}: variant {best} {ms:.3f} ms {out[f's={s_}']['GB/s']:.0f} GB/s",
              file=sys.stderr, flush=True)
    del Z, cl
    return out


def compare_guesses(step, kinds):
    """Iterations and wall time of one full step with each initial guess (untimed region)."""
    import torch
    out = {}
    for g in kinds:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        cl, X, info, sig, Z = step(g, bounded=True)
        torch.cuda.synchronize()
        out[g] = {"iterations": info["iterations"], "cycles": info["cycles"],
                  "max_rel_residual": info["max_rel_residual"], "step_seconds": time.perf_counter() - t0}
        del cl, X, sig, Z
        print(f"[bench] guess {g}: iterations {info['iterations']} step {out[g]['step_seconds']:.3f} s",
              file=sys.stderr, flush=True)
    return out


def compare_preconds(step, kinds, size, tol):
    """Iterations and wall time of one full step with each preconditioner (guess x0 = M u; untimed region)."""
    import torch
    out = {"neighbourhood_size": size}
    for kind in kinds:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        cl, X, info, sig, Z = step("bj", kind, bounded=True)
        torch.cuda.synchronize()
        out[kind] = {"iterations": info["iterations"], "cycles": info["cycles"],
                     "max_rel_residual": info["max_rel_residual"], "step_seconds": time.perf_counter() - t0,
                     "converged": bool(info["max_rel_residual"] <= tol)}
        del cl, X, sig, Z
        print(f"[bench] precond {kind}: iterations {info['iterations']} step {out[kind]['step_seconds']:.3f} s",
              file=sys.stderr, flush=True)
    return out


def fp64_comparator(B, geom, wl, kh, eh, tol, config, r_sample=4, X_ours=None, sig_ours=None):
    """The plain FP64 GPU solver: complex128 fill and COCG, zero initial guess,
    one incidence per solve.  Setup (neighbour search + fill) is timed once,
    r_sample incidences are solved one by one; the workload's cost is then
    setup + R x the mean per-incidence solve (+ RCS).  With the fast path's
    currents and sigma of the last timed step, the sampled incidences also give
    its accuracy against this FP64 solution (relative current error, sigma in dB)."""
    import torch
    R = kh.shape[0]
    r_s = min(R, r_sample)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    cl = B.build_cloud(geom)
    Z, P = B.fill_Z(cl, B.C128)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    o = B.solve_opts(tol=tol, inner_tol=1e-5, restart=5000, max_cycles=60, prec=B.C128, method=B.COCG)
    iters = []
    refs = []
    for r in range(r_s):
        X, info = B.solve(cl, Z, P, kh[r:r + 1], eh[r:r + 1], o)
        sg = B.rcs(cl, X, -kh[r:r + 1], eh[r:r + 1], monostatic=True)
        iters.append(info["iterations"])
        if X_ours is not None:
            refs.append((X, sg))
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    accuracy = None
    if X_ours is not None:
        cerr, dberr = [], []
        for r, (Xr, sg) in enumerate(refs):
            xr = Xr[:, 0]
            cerr.append(float(torch.linalg.vector_norm(X_ours[:, r] - xr) / torch.linalg.vector_norm(xr)))
            so = sig_ours[:, r].double().cpu()
            sr = sg[:, 0].double().cpu()
            live = sr > 0   # an empty cloud scatters nothing on either side
            dberr.append(float((10.0 * torch.log10(so[live] / sr[live])).abs().max()) if bool(live.any()) else 0.0)
        accuracy = {"incidences": r_s, "max_rel_current_error": max(cerr), "max_rcs_error_db": max(dberr),
                    "what": "fast path (last timed step) against this FP64 solver, per sampled incidence"}
    per = (t2 - t1) / r_s
    total = (t1 - t0) + R * per
    systems = wl.cloud.n_clouds * R
    del Z, P, cl
    print(f"[bench] FP64 comparator: setup {t1 - t0:.3f} s, {per:.3f} s per incidence, "
          f"iterations {iters}", file=sys.stderr, flush=True)
    return {"kind": "plain FP64 GPU solver: complex128 fill and COCG, zero initial guess, one incidence per solve",
            "value": systems / total, "unit": "solved angles/s", "setup_seconds": t1 - t0,
            "seconds_per_incidence": per, "incidences_sampled": r_s, "iterations": iters,
            "accuracy_of_value": accuracy, "speedup_of_value": None}


GOLDEN_DIR = os.path.join(ROOT, "tests", "golden")


def oracle_golden_check(config, X, sig):
    """The last timed step's currents and sigma against the oracle's FP64 solutions of the
    stored incidences (tests/golden/fullsize_<config>.npz, written from oracle/ alone):
    relative current error over the stored wires and sigma error in dB."""
    import numpy as np
    import torch
    path = os.path.join(GOLDEN_DIR, f"fullsize_{config}.npz")
    if not os.path.exists(path):
        return None
    g = np.load(path)
    gi = g["incidences"]
    nb = 7   # the stored solutions are of the 8-segment workloads
    rows = (nb * g["wires"][:, None] + np.arange(nb)[None, :]).reshape(-1)
    xs = X[:, torch.as_tensor(gi, device=X.device)][torch.as_tensor(rows, device=X.device)].cpu().numpy()
    cerr = np.linalg.norm(xs - g["currents"], axis=0) / np.linalg.norm(g["currents"], axis=0)
    db = np.abs(10 * np.log10(sig[0, torch.as_tensor(gi, device=sig.device)].double().cpu().numpy() / g["sigma"]))
    return {"incidences": gi.tolist(), "wires": int(g["wires"].size), "oracle_rel_residual": float(g["rel_res"].max()),
            "max_rel_current_error": float(cerr.max()), "max_rcs_error_db": float(db.max()),
            "what": "fast path (last timed step) against the FP64 oracle's GMRES solutions of these incidences"}


def main(argv=None) -> int:
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=2)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--config", default="c5", choices=sorted(CONFIGS))
    ap.add_argument("--tol", type=float, default=1e-6)
    ap.add_argument("--restart", type=int, default=None)
    ap.add_argument("--method", default=None, choices=sorted(METHODS))
    ap.add_argument("--inner-tol", type=float, default=None)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-autotune", action="store_true")
    ap.add_argument("--kernels", action="store_true", help="print the per-kernel table to stderr")
    ap.add_argument("--guess", default=None, choices=sorted(GUESSES),
                    help="initial guess: zero, bj (block-Jacobi) or mlp (learned; trained before timing)")
    ap.add_argument("--nbhd-size", type=int, default=None,
                    help="wires per neighbourhood of the neighbourhood-inverse preconditioner (1..8)")
    ap.add_argument("--precond", default=None, choices=sorted(PRECONDS),
                    help="preconditioner: block (inverse self blocks) or cluster (inverse diagonal "
                         "blocks of groups of 8 nearby wires)")
    ap.add_argument("--no-compare", action="store_true",
                    help="skip the untimed zero / block-Jacobi / learned guess comparison")
    ap.add_argument("--no-sweep", action="store_true", help="skip the product sweep over RHS counts")
    ap.add_argument("--no-comparator", action="store_true",
                    help="skip the plain FP64 one-RHS-at-a-time solver comparison")
    ap.add_argument("--no-profile", action="store_true",
                    help="time the steps without the per-launch HIP events (no roofline or kernel table); "
                         "for launch-bound workloads, where the events themselves cost a visible share")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run only a plain 1 GiB device-to-device copy (scale for HBM byte counters)")
    a = ap.parse_args(argv)
    if a.copy_calibration:
        import torch
        n = 1 << 30
        x = torch.ones(n // 4, dtype=torch.float32, device="cuda")
        y = torch.empty_like(x)
        for _ in range(4):
            y.copy_(x)
        torch.cuda.synchronize()
        print(json.dumps({"copy_calibration": {"bytes_read_per_launch": n, "bytes_written_per_launch": n,
                                               "launches": 4}}))
        return 0
    if a.gpus != 1:
        print(f"bench.py measures one GPU only (asked for --gpus {a.gpus}); the library has no multi-GPU "
              "path. Run with --gpus 1.", file=sys.stderr)
        return 2

    import numpy as np
    import torch

    from paper_2410_03060_amd import binding as B

    torch.cuda.set_device(0)
    cfg = CONFIGS[a.config]
    prec = B.C64 if cfg["prec"] == "c64" else B.C128
    restart = a.restart or cfg["restart"]
    wl = make_workload(a.config)
    geom = B.upload(wl.cloud)
    kh = torch.as_tensor(wl.inc.k_hat, device="cuda")
    eh = torch.as_tensor(wl.inc.e_hat, device="cuda")
    R = kh.shape[0]
    method = a.method or cfg["method"]
    opts = B.solve_opts(tol=a.tol, restart=restart, max_cycles=60, prec=prec, method=METHODS[method],
                        inner_tol=a.inner_tol or cfg["inner_tol"])
    torch.cuda.synchronize()

    guess = a.guess or cfg.get("guess", "zero")
    pc = a.precond or cfg.get("precond", "block")
    opts.precond = PRECONDS[pc]
    mlp_report = None
    theta = None
    compare = not a.no_compare and a.config in MLP_TRAINING
    if guess == "mlp" or compare:   # the learned guess is trained for the comparison too
        theta, mlp_report = train_guess(a.config, B)
    nbhd_mlp_report = None
    theta_nb = None

    nbhd_size = a.nbhd_size or cfg.get("nbhd_size", NBHD_SIZE)

    if pc == "nbhd_mlp" or (compare and a.config in NBHD_MLP_TRAINING):
        theta_nb, nbhd_mlp_report = train_nbhd_mlp(a.config, nbhd_size)

    def make_precond(cl, Z, P, kind=None):
        kind = kind or pc
        if kind == "cluster":
            return B.cluster_precond(cl, Z, prec)
        if kind == "nbhd":
            return B.nbhd_precond(cl, Z, nbhd_size, prec)
        if kind == "nbhd_mlp":
            return B.nbhd_mlp_precond(cl, theta_nb, P, nbhd_size, prec)
        return P

    def step(guess_kind=None, precond_kind=None, bounded=False):
        gk = guess_kind or guess
        kind = precond_kind or pc
        cl = B.build_cloud(geom)
        Z, P = B.fill_Z(cl, prec)
        M = make_precond(cl, Z, P, kind)
        x0 = B.mlp_guess(cl, P, theta, kh, eh, prec=prec) if gk == "mlp" else None
        opts.use_x0 = GUESSES[gk]
        opts.precond = PRECONDS[kind]
        if bounded:   # comparisons: at most 3 cycles of 1,500 steps, a non-converged solve is reported
            o = B.solve_opts(tol=opts.tol, inner_tol=opts.inner_tol, restart=min(opts.restart, 1500), max_cycles=3,
                             use_x0=opts.use_x0, prec=opts.prec, method=opts.method, precond=opts.precond)
            X, info = B.solve(cl, Z, M, kh, eh, o, x0=x0, raise_on_noconv=False)
        else:
            X, info = B.solve(cl, Z, M, kh, eh, opts, x0=x0)
        sig = B.rcs(cl, X, -kh, eh, monostatic=True)
        return cl, X, info, sig, Z

    print(f"[bench] config={a.config} N={wl.cloud.n} clouds={wl.cloud.n_clouds} R={R} warmup={a.warmup} "
          f"steps={a.steps}", file=sys.stderr, flush=True)
    tuning = None
    if not a.no_autotune:   # pick the product variant for this cloud and RHS count (outside the timed steps)
        cl0 = B.build_cloud(geom)
        Z0, _ = B.fill_Z(cl0, prec, with_pinv=False)
        best, best_ms = B.autotune(cl0, Z0, R, prec)
        tuning = {"best_variant": best, "best_ms": best_ms, "table": B.tune_report()}
        del Z0, cl0
        print(f"[bench] autotune: variant {best} ({best_ms:.3f} ms)", file=sys.stderr, flush=True)
    for w in range(a.warmup):
        _, _, info, _, _ = step()
        print(f"[bench] warmup {w}: cycles={info['cycles']} iters={info['iterations']} "
              f"res={info['max_rel_residual']:.2e} solve={info['seconds']:.3f}s", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    B.profile_enable(not a.no_profile)
    t0 = time.perf_counter()
    solved = 0
    infos = []
    for k in range(a.steps):
        cl, X, info, sig, _ = step()
        infos.append(info)
        solved += int((info["rel_res"] <= a.tol).sum())
    X_last, sig_last = X, sig
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    B.profile_enable(False)
    prof = B.profile_read()
    dt = t1 - t0
    free_b, total_b = torch.cuda.mem_get_info()
    memory = {"torch_peak_allocated_GB": torch.cuda.max_memory_allocated() / 1e9,
              "device_used_GB_after_steps": (total_b - free_b) / 1e9, "device_total_GB": total_b / 1e9}
    sig_np = sig.cpu().numpy()
    assert np.all(np.isfinite(sig_np))

    # dominant kernel of the timed region and its roofline
    roof, kernels = None, None
    if prof:
        ranked = sorted(prof.items(), key=lambda kv: -kv[1]["total_ms"])
        name, k = ranked[0]
        symbol = kernel_symbol(name, wl.cloud.n_seg - 1, prec == B.C64, method, R, pc == "cluster")
        # products on the FP32 matrix cores
        mfma = symbol.endswith("k_cocg_mfma") or (prec == B.C64 and symbol.endswith("k_cg_update_cl"))
        roof = roofline_of(k, mfma, prec == B.C128 or name in ("lone_solve", "rcs_bistatic", "rcs_mono"))
        roof["traffic"] = measured_traffic(a.config, name)
        mc = measured_mfma(a.config, name)
        if mc is not None:   # matrix-core counters of the same kernel (profiles/mfma_counters.json)
            roof["mfma_busy"] = mc["mfma_busy_fraction"]
            roof["mfma_flop_counted_per_launch"] = mc["mfma_flop"]
        roof.update({"kernel": name, "symbol": symbol, "launches": k["launches"],
                     "avg_ms": k["total_ms"] / k["launches"],
                     "timing": "HIP events recorded on the launch stream around every launch in the timed steps"})
        kernels = {}
        for n, v in ranked[:12]:
            row = {"ms_total": round(v["total_ms"], 3), "launches": v["launches"]}
            if v["total_ms"] > 0:
                if v["bytes"] > 0:
                    row["GB/s"] = round(v["bytes"] / (v["total_ms"] / 1e3) / 1e9, 2)
                if v["flops"] > 0:
                    row["TFLOP/s"] = round(v["flops"] / (v["total_ms"] / 1e3) / 1e12, 2)
            kernels[n] = row
        if a.kernels:
            for n, v in ranked:
                print(f"  {n:28s} {v['launches']:7d} {v['total_ms']:10.3f} ms", file=sys.stderr)

    out = {
        "metric": "solved angles/sec at <=0.1 dB RCS error; fill GFLOP/s and SpMM GB/s vs peak",
        "value": solved / dt,
        "unit": "solved angles/s",
        "n_gpus": 1,
        "steps": a.steps,
        "warmup": a.warmup,
        "ms_per_step": dt / a.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c64+f64" if prec == B.C64 else "c128",
        "data": "synthetic",
        "config": {"workload": a.config, "description": cfg["desc"], "wires": int(wl.cloud.n),
                   "clouds": int(wl.cloud.n_clouds), "rhs": int(R), "unknowns": int(wl.cloud.n * (wl.cloud.n_seg - 1)),
                   "unknowns_per_wire": int(wl.cloud.n_seg - 1),
                   "nnzb": int(cl.nnzb), "pairs": int(cl.n_pairs), "method": method, "restart": restart,
                   "tol": a.tol, "initial_guess": guess, "preconditioner": pc,
                   "neighbourhood_size": nbhd_size if pc in ("nbhd", "nbhd_mlp") else None},
        "solver": {"cycles": infos[-1]["cycles"], "iterations": infos[-1]["iterations"],
                   "max_rel_residual": infos[-1]["max_rel_residual"],
                   "systems_per_step": int(wl.cloud.n_clouds * R), "solved_total": solved},
        "roofline": roof,
        "autotune": tuning,
        "kernels": kernels,
        "fill": fill_summary(prof, a.config),
        "spmm_sweep": None,
        "memory": memory,
        "mlp": mlp_report,
        "nbhd_mlp": nbhd_mlp_report,
        "guess_comparison": None,
        "precond_comparison": None,
        "comparator": None,
        "cpu_baseline": None,
        "pcie_inclusive": None,
    }
    del X, sig, cl
    # PCIe-inclusive figure (untimed for `value`): the same step with the geometry
    # uploaded from host memory at its start and sigma copied back at its end
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    geom_h = B.upload(wl.cloud)
    cl_h = B.build_cloud(geom_h)
    Z_h, P_h = B.fill_Z(cl_h, prec)
    M_h = make_precond(cl_h, Z_h, P_h)
    x0_h = B.mlp_guess(cl_h, P_h, theta, kh, eh, prec=prec) if guess == "mlp" else None
    opts.use_x0 = GUESSES[guess]
    X_h, info_h = B.solve(cl_h, Z_h, M_h, kh, eh, opts, x0=x0_h)
    sig_h = B.rcs(cl_h, X_h, -kh, eh, monostatic=True).cpu()
    t_h = time.perf_counter() - t0
    out["pcie_inclusive"] = {"value": int((info_h["rel_res"] <= a.tol).sum()) / t_h, "ms_per_step": t_h * 1e3,
                             "what": "one step with the wire geometry uploaded from host memory and sigma "
                                     "copied to host memory inside the timed interval"}
    del geom_h, cl_h, Z_h, P_h, M_h, x0_h, X_h, sig_h
    if not a.no_sweep:
        out["spmm_sweep"] = spmm_sweep(B, geom, prec)
    if not a.no_compare and a.config in MLP_TRAINING:
        out["guess_comparison"] = compare_guesses(step, ["zero", "bj"] + (["mlp"] if theta is not None else []))
        kinds = ["block", "cluster", "nbhd"] + (["nbhd_mlp"] if theta_nb is not None else [])
        out["precond_comparison"] = compare_preconds(step, kinds, nbhd_size, a.tol)
    if not a.no_comparator:
        out["comparator"] = fp64_comparator(B, geom, wl, kh, eh, a.tol, a.config, X_ours=X_last, sig_ours=sig_last)
    if not a.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(wl)
    # accuracy gate of the metric (<= 0.1 dB RCS error, <= 1e-4 current error): every sampled
    # check against the oracle's solutions and against the FP64 GPU solver must pass, else value = 0
    checks = []
    gold = oracle_golden_check(a.config, X_last, sig_last)
    if gold is not None:
        checks.append(gold)
    if out["comparator"] and out["comparator"].get("accuracy_of_value"):
        checks.append(out["comparator"]["accuracy_of_value"])
    passed = all(c["max_rcs_error_db"] <= 0.1 and c["max_rel_current_error"] <= 1e-4 for c in checks)
    out["accuracy_gate"] = {"passed": passed, "checks": checks,
                            "rule": "value counts systems with FP64 residual <= tol; it is set to 0 unless every "
                                    "sampled incidence is within 0.1 dB and 1e-4 relative current error"}
    if not passed:
        out["value"] = 0.0
    if out["comparator"]:
        out["comparator"]["speedup_of_value"] = out["value"] / out["comparator"]["value"]
    print(json.dumps(out))
    return 0


if __name__ == "__main__":
    sys.exit(main())
