"""Benchmark: WENO5-Z RK3 nonhydrostatic step of a 256^3 free-convection LES
on one MI355X, through the C ABI.

Prints ONE JSON line with the whole-job throughput in cell-steps/s of the
FP32-mixed path (FP32 state and stencils, FP64 Poisson solve and projection),
the FP64 path beside it, the roofline figure of the dominant kernel (its
launches timed by HIP events on the model's stream inside the timed region),
per-kernel times from a second, untimed pass that records every launch, and
the CPU oracle timed on a bounded sample of the same workload.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--n 256] [--no-cpu]
"""
import argparse
import re
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, vendor figure
# FP32 vector peak without packed math: 256 CUs x 4 SIMDs x 16 lanes x 2 flops
# (FMA) x 2.4 GHz.  Packed FP32 instructions are disabled in this build.
FP32_VALU_PEAK_TFLOPS = 256 * 4 * 16 * 2 * 2.4e9 / 1e12
FP32_PUBLISHED_PEAK_TFLOPS = 157.3   # MI355X FP32 vector, vendor figure (packed math)

# Algorithmic floating-point operations of one cell-substage of the
# tendency + RK3 kernel (5 prognostic fields), counting + - * / each as one:
FLOPS_PER_CELL_STAGE = {
    "weno5z_flux": 15 * 79,        # 15 face fluxes: candidates 18, indicators 36,
                                   # tau 1, weights 15, normalisation 8, U*W 1
    "diffusive_flux": 15 * 3,
    "advecting_velocity": 9 * 5,   # fourth-order interpolation, momentum fluxes
    "flux_divergence": 15 * 3,
    "coriolis": 2 * 5,
    "buoyancy": 9,
    "rk3_combine": 5 * 4,
    "tracer_offset": 2 * 7,
}


def weno_flux_flops(r):
    """One WENO-Z face flux of order 2r - 1 (r = 4, 5) as the kernel forms it:
    2r - 2 deviations and 2r - 2 differences, r indicators of r - 1 squares
    ((r - 1)(r + 1) each), tau 2r, r candidates of r - 1 products 2(r - 1),
    weights 9 per candidate, normalisation 3, U * W 1."""
    return (4 * r - 4) + r * (r - 1) * (r + 1) + 2 * r + 2 * r * (r - 1) + 9 * r + 3 + 1


def flops_per_cell_stage(r):
    """FLOPS_PER_CELL_STAGE for stencil radius r (3: WENO5, 4: WENO7, 5: WENO9);
    the advecting velocity of order 2r - 2 costs 3r - 4."""
    if r == 3:
        return dict(FLOPS_PER_CELL_STAGE)
    out = dict(FLOPS_PER_CELL_STAGE)
    del out["weno5z_flux"]
    out[f"weno{2 * r - 1}z_flux"] = 15 * weno_flux_flops(r)
    out["advecting_velocity"] = 9 * (3 * r - 4)
    return out
COUNTERS = os.path.join(ROOT, "profiles", "tendency_rk3_fp32_256cubed_counters.json")
# the sources the WENO5 tendency kernel is compiled from
TENDENCY_SRC = [os.path.join(ROOT, "paper_2502_14148_amd", "csrc", f)
                for f in ("tendency.hip", "tendency_tile.h", "weno_dev.h", "weno_coeffs.h",
                          "oc_internal.h")]


def tendency_source_sha256():
    import hashlib
    h = hashlib.sha256()
    for f in TENDENCY_SRC:
        h.update(open(f, "rb").read())
    return h.hexdigest()


def measured_traffic():
    """HBM bytes per tendency launch from the committed rocprofv3 counter
    record, or None if the kernel sources changed since it was taken."""
    try:
        rec = json.load(open(COUNTERS))
        src = tendency_source_sha256()
    except (OSError, ValueError):
        return None
    return rec["traffic_bytes_per_launch"] if rec.get("source_sha256") == src else None


def record_counters(fetch_dir, write_dir):
    """Write the counter record (COUNTERS) from the two rocprofv3 counter
    runs of this script with `--steps 1 --warmup 0 --calibrate-copy`, one
    with `--pmc FETCH_SIZE` (output in fetch_dir), one with `--pmc
    WRITE_SIZE` (write_dir).  The calibration copy is the non-library kernel
    with the largest FETCH_SIZE (the fills before it fetch nothing); the
    scale factors map its counters onto the 1 GiB it reads and writes."""
    import csv
    import glob

    def rows(d, counter):
        f = glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True)
        if not f:
            raise SystemExit(f"no counter_collection.csv under {d}")
        out = []
        for r in csv.DictReader(open(f[0])):
            if r["Counter_Name"] == counter:
                name = r.get("Kernel_Name") or r.get("Kernel-Name")
                out.append((int(r["Dispatch_Id"]), name, float(r["Counter_Value"])))
        return sorted(out)

    fr, wr = rows(fetch_dir, "FETCH_SIZE"), rows(write_dir, "WRITE_SIZE")
    ours = lambda n: "oc::" in n
    copy_name = max((r for r in fr if not ours(r[1])), key=lambda r: r[2])[1]
    fetch_copy = max(r[2] for r in fr if r[1] == copy_name)
    write_copy = max(r[2] for r in wr if r[1] == copy_name)
    gib_kib = 1024.0 * 1024.0
    ff, wf = gib_kib / fetch_copy, gib_kib / write_copy
    # the FP32 WENO-Z kernel with two tracers, plain (no mask, no closure), any tile
    key = re.compile(r"tendency_zmarch<float, 1, 2, (\d+), (\d+), 3, false, false>")
    tf = [r[2] for r in fr if key.search(r[1])]
    tw = [r[2] for r in wr if key.search(r[1])]
    tile = next(key.search(r[1]).groups() for r in fr if key.search(r[1])) if tf else ("?", "?")
    if not tf or len(tf) != len(tw) or len(tf) % 3:
        raise SystemExit(f"expected whole RK3 steps of tendency launches, got {len(tf)}, {len(tw)}")
    per_sub = lambda v: [sum(v[s::3]) / len(v[s::3]) for s in range(3)]
    fk, wk = sum(tf) / len(tf), sum(tw) / len(tw)
    rec = {
        "kernel": f"tendency_zmarch<float, WENO-Z, 2 tracers, {tile[0]}x{tile[1]}, R = 3>",
        "workload": "256^3 free convection FP32",
        "source_sha256": tendency_source_sha256(),
        "sources": [os.path.relpath(f, ROOT) for f in TENDENCY_SRC],
        "fetch_kib_per_launch_raw": fk,
        "write_kib_per_launch_raw": wk,
        "fetch_kib_per_substage_raw": per_sub(tf),
        "write_kib_per_substage_raw": per_sub(tw),
        "fetch_factor": ff,
        "write_factor": wf,
        "calibration": (f"elementwise copy of 1 GiB whose source was written before another "
                        f"1 GiB (no last-level-cache hits): FETCH_SIZE {fetch_copy:.0f} KiB, "
                        f"WRITE_SIZE {write_copy:.0f} KiB"),
        "traffic_bytes_per_launch": (fk * ff + wk * wf) * 1024.0,
    }
    with open(COUNTERS, "w") as f:
        json.dump(rec, f, indent=1)
        f.write("\n")
    print(json.dumps(rec))


def algorithmic_tendency_bytes(ncells, nfields, esz, steps):
    """Bytes the fused tendency + RK3 kernel must move per RK3 step: every
    field read once and written once per substage, plus the G^{m-1} read
    (substages 2, 3) and the G^m write (substages 1, 2)."""
    per_cell = 0
    for st in range(3):
        per_cell += 2 * nfields * esz                    # read X^m, write X~
        per_cell += nfields * esz * ((st > 0) + (st < 2))  # G traffic
    return per_cell * ncells * steps


# Algorithmic HBM bytes per cell of each Poisson pass (FP32 velocities, FP64
# half spectrum of (nx/2 + 1) complex values per x line ~ 8 B per cell):
#   x forward: read u, v, w (12 B), write the half spectrum (8 B);
#   y forward / inverse, z solve: read and write the half spectrum (16 B);
#   x inverse (only where p is asked for, or in the immersed solve): read
#     the half spectrum (8 B), write p (8 B);
#   projection, which in a step is the x inverse fused with it: read the
#     half spectrum (8 B), read and write u, v, w (24 B).
POISSON_BYTES_PER_CELL = {"fft_x_fwd": 20, "fft_y_fwd": 16, "z_solve": 16, "fft_y_inv": 16,
                          "fft_x_inv": 16, "project": 32}


def poisson_hbm(prof, ncells, copy_gbs=None):
    out = {}
    for k, b in POISSON_BYTES_PER_CELL.items():
        ms, n = prof[k]
        if n:
            gbs = b * ncells / (ms / 1e3 / n) / 1e9
            out[k] = {"avg_launch_us": round(ms / n * 1e3, 1), "achieved_gbs": round(gbs, 1),
                      "frac": round(gbs / HBM_PEAK_GBS, 4), "bytes_per_cell": b}
            if copy_gbs:
                out[k]["frac_of_copy"] = round(gbs / copy_gbs, 4)
    return out


def copy_rate_gbs(mib=1024, reps=10):
    """Achieved HBM rate of a plain device copy (torch's elementwise kernel)
    of `mib` MiB, read + write bytes over time: the practical ceiling of a
    pass with equal reads and writes, reported beside the published peak."""
    import torch
    n = mib * 1024 * 1024 // 4
    src = torch.ones(n, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    for _ in range(3):
        dst.copy_(src)
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(reps):
        dst.copy_(src)
    e1.record()
    torch.cuda.synchronize()
    gbs = 2 * n * 4 * reps / (e0.elapsed_time(e1) / 1e3) / 1e9
    del src, dst
    torch.cuda.empty_cache()
    return gbs


def run_gpu(ph, s, precision, steps, warmup):
    """Time `steps` RK3 steps after `warmup` untimed ones.  Inside the timed
    region the model records HIP events around its tendency launches only
    (on the stream they run on), which give the tendency kernel's average
    launch; events around every launch would add about 5 % to the step.  A
    second, untimed pass of as many steps records every kernel class for the
    per-kernel breakdown.  Returns (ms of the timed region, its wall seconds,
    {class: (ms, launches)} with "tendency" from the timed region and the
    other classes from the second pass, diagnostics)."""
    import torch
    from paper_2502_14148_amd import oc
    m = oc.Model(ph, precision)
    m.set_states(s)
    dt = 1.0
    m.rk3_step(dt, warmup)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    m.profile(True, classes=("tendency",))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    e0.record(stream)
    m.rk3_step(dt, steps)
    e1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    m.profile(False)
    timed = m.profile_read()
    ms = e0.elapsed_time(e1)
    m.profile(True)
    m.rk3_step(dt, steps)
    m.profile(False)
    prof = m.profile_read()
    prof["tendency"] = timed["tendency"]
    diag = m.diagnostics()   # raises on non-finite state
    del m
    torch.cuda.empty_cache()
    return ms, wall, prof, diag


def hydro_tendency_bytes(ncells, esz):
    """Bytes the hydrostatic tendency + QAB2 kernel must move per launch:
    reads u, v, T, S, w, zeta, the two pressure gradients and G^{n-1} of
    u, v, T, S; writes the four predicted fields and G^n (12 + 8 fields)."""
    return 20 * esz * ncells


# Algorithmic flops per cell of the hydrostatic tendency + QAB2 kernel: ten
# WENO-Z reconstructions (the x and y faces of T and S, counted once per
# face; the z faces of u, v, T, S; the vorticity at the u and v points), and
# the rest of the cell's arithmetic: vertical fluxes and viscous fluxes 20,
# kinetic energy 8, each momentum point 35 (averages, Coriolis, gradients,
# vertical advection, viscosity, QAB2), each tracer 13 (area factors, flux
# divergence, QAB2).
HYDRO_FLOPS_PER_CELL = 10 * 79 + 20 + 8 + 2 * 35 + 2 * 13


def run_hydrostatic(steps, warmup, N=30):
    """The 1440 x 560 x 50 lat-lon sector in FP32: QAB2 baroclinic steps of
    600 s with N = 30 barotropic substeps per step (cosine-bell filter over
    M = 2N - 1 substeps)."""
    import torch
    from paper_2502_14148_amd import inputs, oc
    ph = inputs.sector_physics()
    print("# generating the 1440x560x50 sector state", file=sys.stderr, flush=True)
    s = inputs.hydrostatic_initial(ph, seed=0, flow=0.1)
    w = inputs.averaging_weights(N)
    m = oc.Model(ph, "fp32")
    m.set_states(s)
    for k in ("eta", "U", "V", "tau_x", "tau_y"):
        m.set_state(k, s[k])
    del s
    dt = 600.0
    m.hydrostatic_step(dt, N, w, warmup)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    # events around the tendency launches only in the timed region, every
    # class in a second pass (as in run_gpu)
    m.profile(True, classes=("hydro_tendency",))
    torch.cuda.synchronize()
    e0.record(stream)
    m.hydrostatic_step(dt, N, w, steps)
    e1.record(stream)
    torch.cuda.synchronize()
    m.profile(False)
    timed = m.profile_read()
    ms = e0.elapsed_time(e1)
    m.profile(True)
    m.hydrostatic_step(dt, N, w, steps)
    m.profile(False)
    prof = m.profile_read()
    prof["hydro_tendency"] = timed["hydro_tendency"]
    finite = bool(np.isfinite(m.get_state("eta")).all())
    del m
    torch.cuda.empty_cache()
    ncells = ph.nx * ph.ny * ph.nz
    t_tend, n_tend = prof["hydro_tendency"]
    t_launch = t_tend / 1e3 / max(n_tend, 1)
    gbs = hydro_tendency_bytes(ncells, 4) / t_launch / 1e9
    tfs = HYDRO_FLOPS_PER_CELL * ncells / t_launch / 1e12
    return {"value": ncells * steps / (ms / 1e3), "unit": "cell-steps/s", "steps": steps,
            "warmup": warmup, "ms_per_step": ms / steps, "dtype": "f32",
            "config": {"workload": "hydrostatic lat-lon sector 1440x560x50, 70S-70N, 3000 m, "
                                   "WENO vector-invariant momentum + WENO tracers, QAB2, "
                                   "split-explicit free surface (FP64)",
                       "dt_s": dt, "N": N, "M": len(w)},
            "kernels_ms_per_step": {k: v[0] / steps for k, v in prof.items() if v[1]},
            "tendency_alu": {"achieved": round(tfs, 2), "peak": FP32_VALU_PEAK_TFLOPS,
                             "unit": "TFLOP/s", "frac": round(tfs / FP32_VALU_PEAK_TFLOPS, 4),
                             "flops_per_cell": HYDRO_FLOPS_PER_CELL},
            "tendency_hbm": {"achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                             "frac": round(gbs / HBM_PEAK_GBS, 4),
                             "avg_launch_ms": t_launch * 1e3,
                             "algorithmic_bytes_per_launch": hydro_tendency_bytes(ncells, 4)},
            "finite": finite}


def run_ensemble(steps, warmup):
    """16 x 64^3 + 16 x 96^3 + 16 x 128^3 free-convection members (FP32),
    stepped together (autotuned fused launches, HIP graph replay) and, for
    comparison, one by one with oc_rk3_step."""
    import torch
    from paper_2502_14148_amd import inputs, oc
    members = inputs.ensemble_physics()
    print("# generating 48 ensemble members", file=sys.stderr, flush=True)
    ms = []
    for ph, seed in members:
        m = oc.Model(ph, "fp32")
        m.set_states(inputs.convection_initial(ph, seed=seed))
        ms.append(m)
    ncells = sum(ph.nx * ph.ny * ph.nz for ph, _ in members)
    dt = 1.0
    e = oc.Ensemble(ms, tune=True, graph=True)
    stream = torch.cuda.current_stream()
    e.step(dt, warmup)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    e.step(dt, steps)
    e1.record(stream)
    torch.cuda.synchronize()
    ms_ens = e0.elapsed_time(e1)
    for m in ms:
        m.rk3_step(dt, 1)
    torch.cuda.synchronize()
    e0.record(stream)
    for m in ms:
        m.rk3_step(dt, steps)
    e1.record(stream)
    torch.cuda.synchronize()
    ms_seq = e0.elapsed_time(e1)
    tn = e.tuning()
    del e, ms
    torch.cuda.empty_cache()
    return {"value": ncells * steps / (ms_ens / 1e3), "unit": "cell-steps/s", "steps": steps,
            "ms_per_step": ms_ens / steps, "dtype": "f32",
            "config": {"workload": "48 free-convection LES members: 16 x 64^3, 16 x 96^3, "
                                   "16 x 128^3, 512 x 512 x 256 m, surface flux U(0.5, 2)e-8",
                       "cells": ncells, "dt_s": dt},
            "one_by_one": {"value": ncells * steps / (ms_seq / 1e3), "ms_per_step": ms_seq / steps},
            "speedup_vs_one_by_one": ms_seq / ms_ens,
            "tuning": tn}


# Algorithmic HBM bytes per cell of the stretched-grid kernels (FP32 state):
#   z_solve (tridiagonal, FP64 half spectrum): read and write it, 16 B;
#   implicit_z: read and write the 5 fields once, 40 B per substage.
STRETCHED_BYTES_PER_CELL = {"z_solve": 16, "implicit_z": 40}


def run_stretched(steps, warmup, n):
    """The 256^3 free-convection step on a surface-refined grid (tanh faces,
    top cell 5.5x thinner than the bottom one) with vertically implicit
    diffusion: FFT-tridiagonal pressure solve and one implicit solve of every
    field per substage (FP32 state, FP64 Poisson)."""
    from paper_2502_14148_amd import inputs
    ph = inputs.stretched_convection_physics((n, n, n), (2.0 * n, 2.0 * n, 1.0 * n), sigma=1.5,
                                             implicit_z=True)
    print(f"# generating the stretched {n}^3 initial state", file=sys.stderr, flush=True)
    s = inputs.convection_initial(ph, seed=0)
    ms, _, prof, diag = run_gpu(ph, s, "fp32", steps, warmup)
    del s
    ncells = n ** 3
    kern = {}
    for k, b in STRETCHED_BYTES_PER_CELL.items():
        t, c = prof[k]
        if c:
            gbs = b * ncells / (t / 1e3 / c) / 1e9
            kern[k] = {"avg_launch_us": round(t / c * 1e3, 1), "achieved_gbs": round(gbs, 1),
                       "frac": round(gbs / HBM_PEAK_GBS, 4), "bytes_per_cell": b}
    zf = np.asarray(ph.z_faces)
    return {"value": ncells * steps / (ms / 1e3), "unit": "cell-steps/s", "steps": steps,
            "warmup": warmup, "ms_per_step": ms / steps, "dtype": "f32",
            "config": {"workload": f"free-convection LES {n}^3 on a surface-refined z grid "
                                   f"(tanh, sigma 1.5), implicit vertical diffusion, "
                                   f"FFT-tridiagonal pressure solve",
                       "dz_top_m": float(zf[-1] - zf[-2]), "dz_bottom_m": float(zf[1] - zf[0]),
                       "dt_s": 1.0},
            "kernels_ms_per_step": {k: v[0] / steps for k, v in prof.items() if v[1]},
            "hbm": kern, "final_max_w": diag["max_w"]}


# Algorithmic HBM bytes per cell of the LES kernels (FP32): the viscosity
# kernel reads u, v, w, T, S (20 B) and writes nu_e (+ AMD's two tracer
# diffusivities); the flux kernel reads u, v, w, T, S, nu_e (+ the
# diffusivities) and writes the five closure tendencies (20 B).
LES_BYTES_PER_CELL = {"smagorinsky": (20 + 4) + (24 + 20), "amd": (20 + 12) + (32 + 20)}


def run_les(steps, warmup, n):
    """The 256^3 free-convection step with an eddy-viscosity closure
    (Smagorinsky-Lilly, then AMD) beside the constant molecular nu, kappa."""
    from paper_2502_14148_amd import inputs
    out = {}
    for kind in ("smagorinsky", "amd"):
        ph = inputs.convection_physics((n, n, n), (2.0 * n, 2.0 * n, 1.0 * n))
        ph.les = kind
        print(f"# {kind} {n}^3 run", file=sys.stderr, flush=True)
        s = inputs.convection_initial(ph, seed=0)
        ms, _, prof, diag = run_gpu(ph, s, "fp32", steps, warmup)
        del s
        ncells = n ** 3
        t, c = prof["les"]
        gbs = LES_BYTES_PER_CELL[kind] * ncells / (t / 1e3 / c) / 1e9
        out[kind] = {"value": ncells * steps / (ms / 1e3), "unit": "cell-steps/s",
                     "ms_per_step": ms / steps,
                     "kernels_ms_per_step": {k: v[0] / steps for k, v in prof.items() if v[1]},
                     "les_hbm": {"avg_substage_us": round(t / c * 1e3, 1), "achieved_gbs": round(gbs, 1),
                                 "frac": round(gbs / HBM_PEAK_GBS, 4),
                                 "bytes_per_cell": LES_BYTES_PER_CELL[kind]},
                     "final_max_w": diag["max_w"]}
    out["config"] = {"workload": f"free-convection LES {n}^3 with Smagorinsky-Lilly (C_s 0.16, "
                                 f"C_b 1, Pr 1) or AMD (C 1/12) eddy viscosity, FP32", "dt_s": 1.0,
                     "steps": steps, "warmup": warmup, "dtype": "f32"}
    return out


def run_weno_high(steps, warmup, n):
    """The 256^3 free-convection step with WENO7-Z and WENO9-Z advection (the
    paper's choice for LES and its global-ocean runs): the same physics and
    initial state as the headline line; the tendency kernel's ALU roofline
    with the flops of the wider reconstructions."""
    from paper_2502_14148_amd import inputs
    ph = inputs.convection_physics((n, n, n), (2.0 * n, 2.0 * n, 1.0 * n))
    print(f"# generating the {n}^3 initial state (WENO7/9 runs)", file=sys.stderr, flush=True)
    s = inputs.convection_initial(ph, seed=0)
    ncells = n ** 3
    out = {}
    for scheme, r in (("weno7z", 4), ("weno9z", 5)):
        ph.advection = scheme
        print(f"# {scheme} {n}^3 run", file=sys.stderr, flush=True)
        ms, _, prof, diag = run_gpu(ph, s, "fp32", steps, warmup)
        t, c = prof["tendency"]
        t_launch = t / 1e3 / c
        flops = sum(flops_per_cell_stage(r).values()) * ncells
        tf = flops / t_launch / 1e12
        tbytes = algorithmic_tendency_bytes(ncells, 5, 4, steps) / c
        gbs = tbytes / t_launch / 1e9
        out[scheme] = {"value": ncells * steps / (ms / 1e3), "unit": "cell-steps/s",
                       "ms_per_step": ms / steps,
                       "kernels_ms_per_step": {k: v[0] / steps for k, v in prof.items() if v[1]},
                       "tendency_roofline": {
                           "bound": "alu", "achieved": round(tf, 2),
                           "peak": FP32_VALU_PEAK_TFLOPS, "unit": "TFLOP/s",
                           "frac": round(tf / FP32_VALU_PEAK_TFLOPS, 4),
                           "avg_launch_ms": t_launch * 1e3,
                           "algorithmic_flops_per_launch": flops,
                           "hbm": {"achieved": round(gbs, 1), "peak": HBM_PEAK_GBS,
                                   "unit": "GB/s", "frac": round(gbs / HBM_PEAK_GBS, 4)}},
                       "final_max_w": diag["max_w"]}
    out["config"] = {"workload": f"free-convection LES {n}^3 (as the headline line) with "
                                 f"WENO7-Z / WENO9-Z advection, FP32", "dt_s": 1.0,
                     "steps": steps, "warmup": warmup, "dtype": "f32"}
    return out


def run_immersed(steps, warmup, n):
    """The 256^3 free-convection step over a Gaussian seamount (grid-fitted
    immersed bottom, 40 % of the depth high): masked tendencies and the
    conjugate-gradient pressure solve preconditioned by the FFT/DCT solve."""
    from paper_2502_14148_amd import inputs, oc
    import torch
    ph = inputs.seamount_convection_physics((n, n, n), (2.0 * n, 2.0 * n, 1.0 * n), 0.4, 0.15)
    # FP32 state: a residual of 1e-10 leaves a divergence far below what the
    # FP32 velocities resolve (the parity tests solve to 1e-13)
    ph.cg_tol = 1e-10
    print(f"# generating the {n}^3 seamount initial state", file=sys.stderr, flush=True)
    s = inputs.convection_initial(ph, seed=0)
    m = oc.Model(ph, "fp32")
    m.set_states(s)
    del s
    m.rk3_step(1.0, warmup)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    # no events inside the timed region; every class in a second pass
    torch.cuda.synchronize()
    e0.record(stream)
    m.rk3_step(1.0, steps)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1)
    m.profile(True)
    m.rk3_step(1.0, steps)
    m.profile(False)
    prof = m.profile_read()
    it, res = m.pressure_stats()
    diag = m.diagnostics()
    del m
    torch.cuda.empty_cache()
    ncells = n ** 3
    solves = 3 * steps
    t_fft = sum(prof[k][0] for k in ("fft_x_fwd", "fft_y_fwd", "z_solve", "fft_y_inv", "fft_x_inv"))
    # box solves: the starting iterate, one per iteration, and the one for p
    n_fft = prof["fft_x_fwd"][1]
    iters_per_solve = n_fft / solves - 2
    cg_ms = prof["cg"][0]
    return {"value": ncells * steps / (ms / 1e3), "unit": "cell-steps/s", "steps": steps,
            "warmup": warmup, "ms_per_step": ms / steps, "dtype": "f32",
            "config": {"workload": f"free-convection LES {n}^3 over a Gaussian seamount "
                                   f"(grid-fitted bottom, 0.4 lz high, e-folding width 0.15 lx), "
                                   f"WENO5-Z, conjugate-gradient pressure solve preconditioned "
                                   f"by the FFT/DCT solve", "dt_s": 1.0,
                       "immersed_fraction": float(np.mean(ph.solid)), "cg_tol": ph.cg_tol},
            "kernels_ms_per_step": {k: v[0] / steps for k, v in prof.items() if v[1]},
            "cg": {"iterations_per_solve": iters_per_solve, "last_solve": {"iterations": it,
                                                                           "rel_residual": res},
                   "ms_per_solve": (cg_ms + t_fft) / solves},
            "final_max_w": diag["max_w"]}


MLP_FLOPS_PER_ROW = 2 * (500 * 256 + 256 * 256 + 256 * 4)   # forward, one cell
BF16_PEAK_TFLOPS = 2500.0      # MI355X dense BF16 MFMA


def run_closure_mlp(reps=20, batch=4096, cells=64 ** 3):
    """The closure network on the 64^3 coarse grid: inference over all
    262 144 cells (one substage's worth) and Adam training steps of 4096
    cells (forward + backward = 3 x the forward flops)."""
    import torch
    from paper_2502_14148_amd import oc
    rng = np.random.default_rng(0)
    x = torch.from_numpy(rng.standard_normal((cells, 500)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.standard_normal((cells, 4)).astype(np.float32)).cuda()
    net = oc.Mlp(cells)
    p = {}
    for k, shp in oc.MLP_SHAPES:
        p[k] = rng.standard_normal(shp) / np.sqrt(shp[1]) if k.startswith("W") else np.zeros(shp)
    net.set_params(p)
    stream = torch.cuda.current_stream()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    net.forward(x)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(reps):
        net.forward(x)
    e1.record(stream)
    torch.cuda.synchronize()
    t_inf = e0.elapsed_time(e1) / reps / 1e3
    nb = cells // batch
    net.train_step(x[:batch], t[:batch], 1e-4, want_loss=False)
    torch.cuda.synchronize()
    e0.record(stream)
    for b in range(nb):
        net.train_step(x[b * batch:(b + 1) * batch], t[b * batch:(b + 1) * batch], 1e-4,
                       want_loss=False)
    e1.record(stream)
    torch.cuda.synchronize()
    t_tr = e0.elapsed_time(e1) / nb / 1e3
    inf_tf = MLP_FLOPS_PER_ROW * cells / t_inf / 1e12
    tr_tf = 3 * MLP_FLOPS_PER_ROW * batch / t_tr / 1e12
    # the fused closure inside a 64^3 model step (gather + network + flux
    # divergence per substage), from the model's own event timing
    from paper_2502_14148_amd import inputs
    ph = inputs.convection_physics((64, 64, 64), (512.0, 512.0, 256.0))
    ph.closure = True
    m = oc.Model(ph, "fp32")
    m.set_states(inputs.convection_initial(ph, seed=0))
    stats = np.array([0, 0, 0, 0, 1e-3, 1e-3, 1e-3, 1e-6, 0, 0, 0, 0, 1e-6, 1e-6, 1e-6, 1e-9])
    m.set_closure(net, stats)
    m.rk3_step(1.0, 1)
    m.profile(True)
    m.rk3_step(1.0, 5)
    m.profile(False)
    cms, cn = m.profile_read()["closure"]
    t_fused = cms / 1e3 / max(cn, 1)
    fz_tf = MLP_FLOPS_PER_ROW * cells / t_fused / 1e12
    return {"inference": {"cells": cells, "ms": t_inf * 1e3, "tflops": round(inf_tf, 1),
                          "frac_bf16_peak": round(inf_tf / BF16_PEAK_TFLOPS, 4)},
            "train_step": {"batch": batch, "ms": t_tr * 1e3, "tflops": round(tr_tf, 1),
                           "frac_bf16_peak": round(tr_tf / BF16_PEAK_TFLOPS, 4)},
            "fused_in_model": {"cells": cells, "ms_per_substage": t_fused * 1e3,
                               "tflops": round(fz_tf, 1),
                               "frac_bf16_peak": round(fz_tf / BF16_PEAK_TFLOPS, 4),
                               "note": "gather + 3 layers + flux divergence, 64^3 model"},
            "flops_per_cell_forward": MLP_FLOPS_PER_ROW, "peak_tflops": BF16_PEAK_TFLOPS}


def _cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(n_sample):
    """The FP64 oracle (NumPy) on a bounded sample: one RK3 step of the same
    physics and horizontal grid on a slab of n_sample levels, once on one
    thread and once with the fields' tendencies on five threads (one per
    prognostic field: the most the oracle's structure uses)."""
    from paper_2502_14148_amd import inputs
    from oracle import timestep
    ph = inputs.convection_physics((256, 256, n_sample), (512.0, 512.0, float(n_sample)))
    s = inputs.convection_initial(ph, seed=0)
    st = timestep.make_state(s, ph)
    cells = ph.nx * ph.ny * ph.nz
    out = {}
    for workers in (1, 5):
        t0 = time.perf_counter()
        timestep.rk3_step(st, 1.0, ph, workers=workers)
        out[workers] = time.perf_counter() - t0
    host = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    sample = (f"1 RK3 step (FP64 NumPy oracle) of the free-convection physics on a "
              f"256x256x{n_sample} slab at 2 m x 2 m x 1 m spacing")
    return {"value": cells / out[5], "unit": "cell-steps/s", "cores": 5, "kind": "oracle",
            "sample": f"{sample}, tendencies of the 5 fields on 5 threads, {out[5]:.1f} s",
            "single_core": {"value": cells / out[1], "cores": 1, "seconds": out[1]},
            "host_cores": host, "cpu_model": _cpu_model()}


def main_leg(a):
    """The 256^3 nonhydrostatic step: the headline line of the benchmark."""
    from paper_2502_14148_amd import inputs
    n = a.n
    ph = inputs.convection_physics((n, n, n), (2.0 * n, 2.0 * n, 1.0 * n))
    print(f"# generating the {n}^3 initial state", file=sys.stderr, flush=True)
    s = inputs.convection_initial(ph, seed=0)
    ncells = n ** 3
    nf = 5

    print("# FP32-mixed run", file=sys.stderr, flush=True)
    ms32, wall32, prof32, diag32 = run_gpu(ph, s, "fp32", a.steps, a.warmup)
    res = {}
    if not a.no_fp64:
        print("# FP64 run", file=sys.stderr, flush=True)
        ms64, wall64, prof64, _ = run_gpu(ph, s, "fp64", a.steps, a.warmup)
        res = {"value": ncells * a.steps / (ms64 / 1e3), "ms_per_step": ms64 / a.steps,
               "kernels_ms_per_step": {k: v[0] / a.steps for k, v in prof64.items()}}

    value = ncells * a.steps / (ms32 / 1e3)
    t_tend_ms, n_tend = prof32["tendency"]
    t_launch = t_tend_ms / 1e3 / max(n_tend, 1)
    tbytes = algorithmic_tendency_bytes(ncells, nf, 4, a.steps) / max(n_tend, 1)
    flops = sum(FLOPS_PER_CELL_STAGE.values()) * ncells
    achieved_tf = flops / t_launch / 1e12
    achieved_gbs = tbytes / t_launch / 1e9
    # headline: the tendency kernel's algorithmic HBM bytes per launch over
    # its average launch time, against the HBM peak; the VALU figure beside it
    copy_gbs = copy_rate_gbs()
    roofline = {"bound": "hbm", "achieved": round(achieved_gbs, 1), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(achieved_gbs / HBM_PEAK_GBS, 4),
                "copy_kernel_gbs": round(copy_gbs, 1),
                "frac_of_copy": round(achieved_gbs / copy_gbs, 4),
                "traffic": measured_traffic(),
                "kernel": "tendency_rk3 (FP32, WENO5-Z, 256^3)",
                "avg_launch_ms": t_launch * 1e3,
                "algorithmic_bytes_per_launch": tbytes,
                "algorithmic_bytes_per_cell_step": algorithmic_tendency_bytes(1, nf, 4, 1),
                "valu": {"achieved": round(achieved_tf, 2), "unit": "TFLOP/s",
                         "algorithmic_flops_per_launch": flops,
                         "peak_published": FP32_PUBLISHED_PEAK_TFLOPS,
                         "frac_published": round(achieved_tf / FP32_PUBLISHED_PEAK_TFLOPS, 4),
                         "peak_non_packed": FP32_VALU_PEAK_TFLOPS,
                         "frac_non_packed": round(achieved_tf / FP32_VALU_PEAK_TFLOPS, 4)}}
    out = {
        "metric": "cell-steps/s (WENO5 RK3 step, 256^3) + tendency-kernel HBM GB/s vs peak",
        "value": value, "unit": "cell-steps/s", "n_gpus": 1, "steps": a.steps,
        "warmup": a.warmup, "ms_per_step": ms32 / a.steps, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"free-convection LES {n}^3, WENO5-Z RK3 with FFT/DCT pressure "
                               f"projection, FP32 state/stencils + FP64 Poisson",
                   "grid": [n, n, n], "extent_m": [2.0 * n, 2.0 * n, 1.0 * n], "dt_s": 1.0},
        "roofline": roofline,
        "kernels_ms_per_step": {k: v[0] / a.steps for k, v in prof32.items()},
        "poisson_hbm": poisson_hbm(prof32, ncells, copy_gbs),
        "fp64_path": res,
        "wall_s_timed": wall32,
        "final_max_w": diag32["max_w"],
    }
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--n", type=int, default=256)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-fp64", action="store_true")
    ap.add_argument("--cpu-levels", type=int, default=32)
    ap.add_argument("--no-hydrostatic", action="store_true")
    ap.add_argument("--no-ensemble", action="store_true")
    ap.add_argument("--no-closure", action="store_true")
    ap.add_argument("--no-stretched", action="store_true")
    ap.add_argument("--no-les", action="store_true")
    ap.add_argument("--no-weno-high", action="store_true")
    ap.add_argument("--no-immersed", action="store_true")
    ap.add_argument("--no-main", action="store_true",
                    help="skip the 256^3 step (profiling the other legs alone)")
    ap.add_argument("--ensemble-steps", type=int, default=200)
    ap.add_argument("--hydro-steps", type=int, default=20)
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="first run one plain 1 GiB device copy (counter calibration)")
    ap.add_argument("--record-counters", nargs=2, metavar=("FETCH_DIR", "WRITE_DIR"),
                    help="write the tendency kernel's counter record from two rocprofv3 "
                         "counter runs (no GPU work)")
    a = ap.parse_args()
    if a.record_counters:
        record_counters(*a.record_counters)
        return
    if a.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU only; --gpus must be 1"}))
        sys.exit(2)

    if a.calibrate_copy:
        # HBM counter calibration: an elementwise copy of 1 GiB whose source
        # was written before 1 GiB of other data, so that none of it is left
        # in the 256 MB last-level cache when the copy reads it
        import torch
        src = torch.ones(256 * 1024 * 1024, dtype=torch.float32, device="cuda")
        flush = torch.zeros_like(src)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        torch.mul(src, 1.0, out=dst)        # elementwise copy kernel
        torch.cuda.synchronize()
        del src, flush, dst

    if a.no_main:
        out = {"note": "the 256^3 nonhydrostatic leg was skipped (--no-main)"}
    else:
        out = main_leg(a)
    if not a.no_hydrostatic:
        print("# hydrostatic sector run", file=sys.stderr, flush=True)
        out["hydrostatic"] = run_hydrostatic(a.hydro_steps, 2)
    if not a.no_stretched:
        print("# stretched-grid run", file=sys.stderr, flush=True)
        out["stretched"] = run_stretched(a.steps, a.warmup, a.n)
    if not a.no_les:
        print("# LES closure runs", file=sys.stderr, flush=True)
        out["les"] = run_les(a.steps, a.warmup, a.n)
    if not a.no_weno_high:
        print("# WENO7/9 runs", file=sys.stderr, flush=True)
        out["weno_high"] = run_weno_high(a.steps, a.warmup, a.n)
    if not a.no_immersed:
        print("# immersed seamount run", file=sys.stderr, flush=True)
        out["immersed"] = run_immersed(a.steps, a.warmup, a.n)
    if not a.no_closure:
        print("# closure network", file=sys.stderr, flush=True)
        out["closure_mlp"] = run_closure_mlp()
    if not a.no_ensemble:
        print("# ensemble run", file=sys.stderr, flush=True)
        out["ensemble"] = run_ensemble(a.ensemble_steps, 2)
    if not a.no_cpu:
        print("# CPU oracle sample", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(a.cpu_levels)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
