#!/usr/bin/env python
"""Benchmark of the vectorial Richards-Wolf PSF engine on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W]

A step is one ``rwpsf_compute`` call of the Fourier (Cartesian) form on the
headline workload: 16 stacks, each 128 x 128 x 64 voxels at 20 nm from a
256 x 256 pupil, NA 1.4, 600 nm, circular polarisation, Gibson-Lanni (n_s 1.33,
emitter depth U[0, 5] um) and Noll 4..21 aberrations N(0, 0.05) waves; fields
(complex64) and intensity (float32) are both written.  Inputs are synthetic and
seeded (``workloads``), resident on the GPU before the timed region.

Prints one JSON line with the throughput (voxels/s), the roofline of the
dominant kernel (per-launch time from HIP events on the library's stream during
the timed steps), the CPU oracle timed on a bounded sample, and the other forms.
"""
from __future__ import annotations

import argparse
import glob
import json
import math
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP32_TFLOPS = 157.3   # MI355X dense FP32 matrix
PEAK_F16X3_TFLOPS = 2500.0 / 3   # dense F16 matrix over the three products of a split F32 operand pair
PEAK_HBM_GBS = 8000.0      # MI355X HBM3E
PEAK_BF16_TFLOPS = 2500.0  # MI355X dense BF16 matrix


def sources_digest() -> str:
    """SHA-256 over the library's kernel sources (csrc/*.hip, csrc/*.h, include/*.h)."""
    import hashlib
    root = os.path.dirname(os.path.abspath(__file__))
    files = sorted(glob.glob(os.path.join(root, "paper_2502_03170_amd", "csrc", "*.hip")) +
                   glob.glob(os.path.join(root, "paper_2502_03170_amd", "csrc", "*.h")) +
                   glob.glob(os.path.join(root, "include", "*.h")))
    h = hashlib.sha256()
    for f in files:
        h.update(os.path.basename(f).encode())
        h.update(open(f, "rb").read())
    return h.hexdigest()


def _summary_text(summary: str):
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "profiles", summary)
    try:
        with open(path) as f:
            return f.read()
    except OSError:
        return None


def summary_field(text: str, field: str, kernel: str, digest_now: str):
    """The number recorded as '<field> (<kernel>): <number>' in a profile summary that
    records the sources digest `digest_now`, else None."""
    digest = re.search(r"sources sha256: ([0-9a-f]{64})", text)
    if not digest or digest.group(1) != digest_now:
        return None
    m = re.search(re.escape(f"{field} ({kernel}):") + r" ([0-9]+(?:\.[0-9]*)?)", text)
    return float(m.group(1)) if m else None


def traffic_from_summary(text: str, kernel: str, digest_now: str):
    """HBM bytes per dispatch of `kernel` from a summary taken at `digest_now`, else None."""
    v = summary_field(text, "HBM bytes per dispatch", kernel, digest_now)
    return None if v is None else int(v)


def profiled_traffic(summary: str, kernel: str):
    """HBM bytes per dispatch of `kernel` from a committed rocprofv3 counter summary under
    profiles/ (FETCH_SIZE and WRITE_SIZE, scaled by a device copy of known size), or None
    when it is missing or was taken on other kernel sources."""
    text = _summary_text(summary)
    return None if text is None else traffic_from_summary(text, kernel, sources_digest())


def profiled_average(summary: str, kernel: str):
    """Average dispatch duration (us) of `kernel` in the committed rocprofv3 kernel trace of
    the same bench command, or None when missing or taken on other kernel sources."""
    text = _summary_text(summary)
    return None if text is None else summary_field(text, "trace average us", kernel, sources_digest())


def fourier_workload():
    import workloads as W
    w = W.fourier_plain()
    zp = np.linspace(-1000.0, 1000.0, 64)
    stacks = [dict(t_s=w["t_s"][b], z_offset=-w["t_s"][b], zernike=w["zernike"][b]) for b in range(16)]
    return w, zp, stacks


def bench_fourier(rw, torch, steps, warmup):
    w, zp, stacks = fourier_workload()
    o = w["optics"]
    n, nx, nz, B = 256, 128, 64, len(stacks)
    plan = rw.Plan(form=rw.FORM_FOURIER, na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], nx=nx,
                   ny=nx, dx=20.0, dy=20.0, z=zp, e_inc=w["e_inc"], gibson_lanni=w["gl"], n_pupil=n)
    E = torch.empty((B, nz, 3, nx, nx), dtype=torch.complex64, device="cuda")
    I = torch.empty((B, nz, nx, nx), dtype=torch.float32, device="cuda")
    for _ in range(warmup):
        plan.compute(stacks, E=E, I=I)
    torch.cuda.synchronize()
    plan.set_timing(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        plan.compute(stacks, E=E, I=I)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_step = (t1 - t0) * 1e3 / steps
    kt = {name: plan.timing(k) for name, k in (("pupil_build", rw.KERNEL_PUPIL_BUILD),
                                               ("gemm_pupil", rw.KERNEL_GEMM_PUPIL),
                                               ("gemm_image", rw.KERNEL_GEMM_IMAGE))}
    plan.set_timing(False)
    voxels = B * nz * nx * nx
    # algorithmic work of the mirror-folded separable transform, per component-plane:
    # two real GEMMs, [2n x n] x [n x ny] and [nx x n] x [n x 2ny] (half the flops of the
    # complex matrix DFT, 8 n ny (n + nx))
    f1 = 4.0 * n * n * nx            # T = Pf~ B1
    f2 = 4.0 * nx * n * nx           # E' = A2 T
    comp_planes = B * nz * 3
    g1_ms, g1_n = kt["gemm_pupil"]
    g2_ms, g2_n = kt["gemm_image"]
    per_launch_g1 = f1 * comp_planes * steps / g1_n      # launches are counted over all timed steps
    per_launch_g2 = f2 * comp_planes * steps / g2_n
    ach_g1 = per_launch_g1 / (g1_ms / g1_n * 1e-3) / 1e12
    ach_g2 = per_launch_g2 / (g2_ms / g2_n * 1e-3) / 1e12
    step_flops = (f1 + f2) * comp_planes
    plan.close()
    return dict(
        ms_per_step=ms_step, voxels=voxels, value=voxels / (ms_step * 1e-3),
        kernels={k: dict(total_ms=v[0], launches=v[1], avg_us=(v[0] / v[1] * 1e3 if v[1] else None))
                 for k, v in kt.items()},
        roofline=dict(kernel="gemm_pupil_kernel", bound="mfma", achieved=round(ach_g1, 3),
                      peak=PEAK_F16X3_TFLOPS, unit="TFLOP/s", frac=round(ach_g1 / PEAK_F16X3_TFLOPS, 4),
                      traffic=profiled_traffic("gemm_pupil_fourier_plain.txt", "gemm_pupil_kernel"),
                      flops_per_launch=per_launch_g1, avg_launch_us=g1_ms / g1_n * 1e3,
                      profiled_avg_us=profiled_average("gemm_pupil_fourier_plain.txt", "gemm_pupil_kernel")),
        image_gemm=dict(achieved_tflops=round(ach_g2, 3), frac=round(ach_g2 / PEAK_F16X3_TFLOPS, 4),
                        flops_per_launch=per_launch_g2, avg_launch_us=g2_ms / g2_n * 1e3),
        step_tflops=round(step_flops / (ms_step * 1e-3) / 1e12, 3),
        step_frac=round(step_flops / (ms_step * 1e-3) / 1e12 / PEAK_F16X3_TFLOPS, 4))


def bench_chirpz(rw, torch, steps, warmup):
    """The headline workload through the chirp-z (FFT) evaluation of the same sum, and the
    matrix DFT vs chirp-z crossover over pupil sizes (8 stacks, 128x128x64)."""
    w, zp, stacks = fourier_workload()
    o = w["optics"]

    def run(form, n, st, nsteps, timing=False):
        plan = rw.Plan(form=form, na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], nx=128, ny=128, dx=20.0,
                       dy=20.0, z=zp, e_inc=w["e_inc"], gibson_lanni=w["gl"], n_pupil=n)
        E = torch.empty((len(st), 64, 3, 128, 128), dtype=torch.complex64, device="cuda")
        I = torch.empty((len(st), 64, 128, 128), dtype=torch.float32, device="cuda")
        for _ in range(warmup):
            plan.compute(st, E=E, I=I)
        torch.cuda.synchronize()
        if timing:
            plan.set_timing(True)
        t0 = time.perf_counter()
        for _ in range(nsteps):
            plan.compute(st, E=E, I=I)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / nsteps
        kt = {k: plan.timing(v) for k, v in (("czt_rows", rw.KERNEL_CZT_ROWS), ("czt_cols", rw.KERNEL_CZT_COLS))}
        plan.close()
        return (ms, kt) if timing else ms

    ms, kt = run(rw.FORM_CHIRPZ, 256, stacks, steps, timing=True)
    voxels = len(stacks) * 64 * 128 * 128
    # algorithmic work: one forward and one inverse FFT of length L per transformed line,
    # 5 L log2 L flop each (split-radix-free count); the y pass transforms the N pupil rows,
    # the x pass the nx output columns, of every (stack, plane, component)
    L, n, nx = 512, 256, 128
    lines = len(stacks) * 64 * 3
    rows_flops = lines * n * 2 * 5.0 * L * math.log2(L)
    cols_flops = lines * nx * 2 * 5.0 * L * math.log2(L)
    r_ms, r_n = kt["czt_rows"]
    c_ms, c_n = kt["czt_cols"]
    per_launch = rows_flops * steps / r_n
    ach = per_launch / (r_ms / r_n * 1e-3) / 1e12
    ach_c = cols_flops * steps / c_n / (c_ms / c_n * 1e-3) / 1e12
    cross = {}
    for n in (128, 256, 512, 1024):
        cross[str(n)] = dict(matrix_dft_ms=run(rw.FORM_FOURIER, n, stacks[:8], 3),
                             chirpz_ms=run(rw.FORM_CHIRPZ, n, stacks[:8], 3))
    return dict(workload="chirp-z evaluation of the fourier_plain workload (same sum, FFT convolutions of "
                         "length 512 along y and x)", value=voxels / (ms * 1e-3), unit="voxels/s",
                ms_per_step=ms, crossover_8_stacks_128x128x64=cross,
                kernels={k: dict(total_ms=v[0], launches=v[1], avg_us=(v[0] / v[1] * 1e3 if v[1] else None))
                         for k, v in kt.items()},
                roofline=dict(kernel="czt_rows_kernel<512>", bound="alu", achieved=round(ach, 3),
                              peak=PEAK_FP32_TFLOPS, unit="TFLOP/s", frac=round(ach / PEAK_FP32_TFLOPS, 4),
                              traffic=profiled_traffic("czt_chirpz_fourier_plain.txt", "czt_rows_kernel"),
                              flops_per_launch=per_launch, avg_launch_us=r_ms / r_n * 1e3,
                              profiled_avg_us=profiled_average("czt_chirpz_fourier_plain.txt", "czt_rows_kernel")),
                cols_kernel=dict(kernel="czt_cols_kernel<512>", achieved_tflops=round(ach_c, 3),
                                 frac=round(ach_c / PEAK_FP32_TFLOPS, 4)))


def bench_speed_sweep(rw, torch, reps=10):
    """The speed benchmark of Sec. 5.2.1 on one GPU: one 201 x 201 image at focus, per
    propagator (scalar / vectorial x Cartesian / spherical) against the numerical pupil
    size (Cartesian: cells per axis; spherical: theta nodes), mean of `reps` calls after
    two warm-up calls, each call synchronised (pupil build and transform included).
    Optics: NA 1.4, 532 nm, n_i 1.518, circular polarisation, apodization."""
    sizes = (64, 128, 256, 512, 1024)
    props = (("cartesian_vectorial", rw.FORM_FOURIER, rw.MODEL_VECTORIAL),
             ("cartesian_scalar", rw.FORM_FOURIER, rw.MODEL_SCALAR),
             ("cartesian_chirpz_vectorial", rw.FORM_CHIRPZ, rw.MODEL_VECTORIAL),
             ("cartesian_chirpz_scalar", rw.FORM_CHIRPZ, rw.MODEL_SCALAR),
             ("spherical_vectorial", rw.FORM_BESSEL, rw.MODEL_VECTORIAL),
             ("spherical_scalar", rw.FORM_BESSEL, rw.MODEL_SCALAR))
    out = {}
    for name, form, model in props:
        row = {}
        for n in sizes:
            plan = rw.Plan(form=form, na=1.4, wavelength=532.0, n_i=1.518, nx=201, ny=201, dx=20.0, dy=20.0,
                           z=[0.0], n_pupil=n, n_theta=n, n_rho=256, model=model)
            nc = 1 if model == rw.MODEL_SCALAR else 3
            E = torch.empty((1, 1, nc, 201, 201), dtype=torch.complex64, device="cuda")
            I = torch.empty((1, 1, 201, 201), dtype=torch.float32, device="cuda")
            st = rw.Stacks([dict()])
            for _ in range(2):
                plan.compute(st, E=E, I=I)
            torch.cuda.synchronize()
            t = 0.0
            for _ in range(reps):
                t0 = time.perf_counter()
                plan.compute(st, E=E, I=I)
                torch.cuda.synchronize()
                t += time.perf_counter() - t0
            row[str(n)] = t * 1e3 / reps
            plan.close()
        out[name] = row
    return dict(workload="one 201x201 image at focus per call (Sec. 5.2.1 speed benchmark), ms per call vs "
                         "pupil size", ms_per_call=out)


def bench_bessel(rw, torch, steps, warmup, n_stacks=256):
    import workloads as W
    w = W.bessel_plain(n_stacks=n_stacks)
    o = w["optics"]
    plan = rw.Plan(form=rw.FORM_BESSEL, na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], nx=65,
                   ny=65, dx=20.0, dy=20.0, z=w["z"], e_inc=w["e_inc"], n_theta=200, n_rho=256)
    stacks = rw.Stacks([dict(z_offset=float(v)) for v in w["z_offsets"]])   # marshalled once
    nz = len(w["z"])
    E = torch.empty((n_stacks, nz, 3, 65, 65), dtype=torch.complex64, device="cuda")
    I = torch.empty((n_stacks, nz, 65, 65), dtype=torch.float32, device="cuda")
    one = [dict()]
    for _ in range(warmup):
        plan.compute(stacks, E=E, I=I)
        plan.compute(one, E=E[:1], I=I[:1])
    torch.cuda.synchronize()
    # single stack latency
    t0 = time.perf_counter()
    for _ in range(steps):
        plan.compute(one, E=E[:1], I=I[:1])
    torch.cuda.synchronize()
    single_ms = (time.perf_counter() - t0) * 1e3 / steps
    t0 = time.perf_counter()
    for _ in range(steps):
        plan.compute(stacks, E=E, I=I)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    plan.set_timing(True)          # per-launch events in a second pass
    for _ in range(steps):
        plan.compute(stacks, E=E, I=I)
    torch.cuda.synchronize()
    kt = {name: plan.timing(k) for name, k in (("phi", rw.KERNEL_BESSEL_PHI),
                                               ("contract", rw.KERNEL_BESSEL_CONTRACT),
                                               ("epilogue", rw.KERNEL_BESSEL_EPILOGUE))}
    plan.close()
    voxels = n_stacks * nz * 65 * 65
    e_ms, e_n = kt["epilogue"]
    bytes_per_launch = 28.0 * voxels * steps / e_n    # E (24 B) + I (4 B) per voxel written
    ach = bytes_per_launch / (e_ms / e_n * 1e-3) / 1e9
    return dict(workload="bessel_plain: NA 1.4, 532 nm, 65x65x33 at 20 nm, GL-200, 256 radial samples, "
                         f"{n_stacks} stacks per call (focal offsets U(+-100 nm))",
                value=voxels / (ms * 1e-3), unit="voxels/s", ms_per_call=ms,
                single_stack_ms=single_ms, single_stack_voxels_per_s=65 * 65 * nz / (single_ms * 1e-3),
                kernels={k: dict(total_ms=v[0], launches=v[1], avg_us=(v[0] / v[1] * 1e3 if v[1] else None))
                         for k, v in kt.items()},
                roofline=dict(kernel="bessel_epilogue_kernel", bound="hbm", achieved=round(ach, 1),
                              peak=PEAK_HBM_GBS, unit="GB/s", frac=round(ach / PEAK_HBM_GBS, 4),
                              traffic=profiled_traffic("bessel_bessel_plain.txt", "bessel_epilogue_kernel"),
                              bytes_per_launch=bytes_per_launch, avg_launch_us=e_ms / e_n * 1e3,
                              profiled_avg_us=profiled_average("bessel_bessel_plain.txt", "bessel_epilogue_kernel")))


def _cuda_time(torch, fn, reps):
    """Mean milliseconds of fn() over reps calls, HIP events on the current stream."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(reps):
        fn()
    b.record()
    b.synchronize()
    return a.elapsed_time(b) / reps


def bench_batched(rw, torch, steps, warmup):
    import workloads as W
    w = W.batched()
    o = w["optics"]
    em = rw.make_emitters(w["x0"], w["y0"], w["z_e"], w["S"], w["D"], w["zernike"])
    off = rw.batch_offsets(em)
    b = rw.Batch(na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], pixel=w["dx"], plane_pitch=w["dz"],
                 max_emitters=len(w["S"]), n_pupil=w["n_pupil"], e_inc=w["e_inc"])
    I = torch.zeros(off[-1], dtype=torch.float32, device="cuda")
    cfg, tune_ms = b.autotune(em, I)
    s = torch.cuda.Stream()
    b.set_graph(True)
    with torch.cuda.stream(s):
        for _ in range(max(1, warmup)):
            b.compute(em, I=I, stream=s.cuda_stream)
        ms = _cuda_time(torch, lambda: b.compute(em, I=I, stream=s.cuda_stream), max(3, steps // 4))
    b.set_graph(False)
    b.close()
    S = w["S"].astype(np.float64)
    D = w["D"].astype(np.float64)
    n = w["n_pupil"]
    flops = float(np.sum(D * 3 * 4.0 * S * n * (n + S)))     # folded: U = A2_S Pf~, E' = U B1_S per plane
    # executed work on the chosen row tiles (16- and 32-row crops run 32-row tiles, 48 and 64
    # run 64)
    SP = np.array([(cfg["tile_rows"][(int(s) - 1) // 16] + 31) // 32 * 32 for s in w["S"]], dtype=np.float64)
    flops_exec = float(np.sum(D * 3 * 4.0 * SP * n * (n + SP)))
    ach = flops / (ms * 1e-3) / 1e12
    return dict(workload="batched: 4096 emitters, crops U{24..64}, planes U{1..41}, 128x128 pupil, "
                         "Noll 4-21 N(0,0.04), sub-pixel x0/y0, intensity only, one persistent launch per "
                         "tile height (32 and 64 rows), replayed from a hipGraph, tile classes and residency "
                         "autotuned",
                value=off[-1] / (ms * 1e-3), unit="voxels/s", ms_per_launch=ms, voxels=off[-1],
                autotuned_config=dict(cfg, tuned_ms=tune_ms),
                roofline=dict(kernel="batch_planes_kernel (+ fold)", bound="mfma",
                              achieved=round(ach, 3), peak=PEAK_F16X3_TFLOPS, unit="TFLOP/s",
                              frac=round(ach / PEAK_F16X3_TFLOPS, 4),
                              traffic=profiled_traffic("batch_planes_batched.txt", "batched call"),
                              flops_per_launch=flops, avg_launch_us=ms * 1e3,
                              executed_over_algorithmic=round(flops_exec / flops, 4)))


def bench_adjoint(rw, torch, steps, warmup, n_stacks=64):
    import workloads as W
    w = W.adjoint(n_stacks=n_stacks)
    o = w["optics"]
    n, nx, nz = w["n_pupil"], w["nx"], len(w["z"])
    plan = rw.Plan(form=rw.FORM_FOURIER, na=o["na"], wavelength=o["wavelength"], n_i=o["n_i"], nx=nx, ny=nx,
                   dx=w["dx"], dy=w["dy"], z=w["z"], e_inc=w["e_inc"], n_pupil=n)
    rng = np.random.default_rng(404)
    w0 = torch.tensor(w["w0_eval"], dtype=torch.float32, device="cuda")
    st = rw.Stacks([dict(x0=rng.uniform(-50, 50), y0=rng.uniform(-50, 50), z_offset=rng.uniform(-200, 200),
                         zernike=w["c_eval"], phase_map=w0) for _ in range(n_stacks)])
    E = torch.empty((n_stacks, nz, 3, nx, nx), dtype=torch.complex64, device="cuda")
    I = torch.empty((n_stacks, nz, nx, nx), dtype=torch.float32, device="cuda")
    Y = torch.rand_like(I)
    dc = torch.empty(21, dtype=torch.float32, device="cuda")
    dw = torch.empty((n, n), dtype=torch.float32, device="cuda")

    def step():
        plan.compute(st, E=E, I=I)
        rw.adjoint(plan, st, E, (2.0 / I.numel()) * (I - Y), 21, dc, dw)

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    # the step time without per-launch events (each adds a timestamp packet to the stream);
    # the kernel breakdown from a second pass with them
    ms = _cuda_time(torch, step, max(3, steps // 4))
    plan.set_timing(True)
    _cuda_time(torch, step, max(3, steps // 4))
    kt = {k: plan.timing(v) for k, v in (("gemm_pupil", rw.KERNEL_GEMM_PUPIL), ("gemm_image", rw.KERNEL_GEMM_IMAGE),
                                          ("adj_scale", rw.KERNEL_ADJ_H), ("adj", rw.KERNEL_ADJ_G),
                                          ("adj_reduce", rw.KERNEL_ADJ_REDUCE))}
    plan.close()
    comp = n_stacks * nz * 3
    fwd = comp * 4.0 * (n * n * nx + nx * n * nx)     # folded real GEMMs
    adj = comp * 4.0 * (nx * nx * n + n * nx * n)     # folded real GEMMs of the adjoint
    ach = (fwd + adj) / (ms * 1e-3) / 1e12
    vox = n_stacks * nz * nx * nx
    return dict(workload=f"adjoint: {n_stacks} stacks of {nx}x{nx}x{nz} at 100 nm, 256x256 pupil, shared Noll "
                         "1-21 + free 256x256 phase map; step = forward (fields) + adjoint (dL/dc, dL/dW0)",
                value=vox / (ms * 1e-3), unit="voxels/s (forward+adjoint)", ms_per_step=ms,
                gradient_steps_per_s=1e3 / ms,
                kernels={k: dict(total_ms=v[0], launches=v[1], avg_us=(v[0] / v[1] * 1e3 if v[1] else None))
                         for k, v in kt.items()},
                roofline=dict(kernel="whole step", bound="mfma", achieved=round(ach, 3), peak=PEAK_F16X3_TFLOPS,
                              unit="TFLOP/s", frac=round(ach / PEAK_F16X3_TFLOPS, 4),
                              traffic=profiled_traffic("adjoint_adjoint.txt", "adjoint step"),
                              avg_launch_us=ms * 1e3,
                              profiled_avg_us=profiled_average("adjoint_adjoint.txt", "adjoint step"),
                              flops_per_step=fwd + adj))


def bench_adjoint_bessel(rw, torch, steps, warmup, n_stacks=64):
    """Gradient step of the Bessel form at the Bessel workload's grid (65x65x33 at 20 nm,
    200 Gauss-Legendre nodes split at the critical angle, 256 radial samples) with the
    Gibson-Lanni layer: forward (fields) + adjoint (dL/dc for Noll 1, 4, 11, 22, dL/dt_s,
    dL/dz_offset per stack) for an MSE loss."""
    import workloads as W
    w = W.bessel_plain()
    z = np.asarray(w["z"])
    plan = rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=65, ny=65, dx=20.0, dy=20.0,
                   z=z, e_inc=w["e_inc"], gibson_lanni=dict(W.GIBSON_LANNI), n_theta=200, n_rho=256)
    rng = np.random.default_rng(405)
    coeffs = np.zeros(22)
    coeffs[3], coeffs[10], coeffs[21] = 0.04, -0.03, 0.02
    st = []
    for _ in range(n_stacks):
        ts = rng.uniform(0.0, 5000.0)
        st.append(dict(t_s=ts, z_offset=-ts, x0=rng.uniform(-10, 10), y0=rng.uniform(-10, 10), zernike=coeffs))
    st = rw.Stacks(st)
    nz = z.size
    E = torch.empty((n_stacks, nz, 3, 65, 65), dtype=torch.complex64, device="cuda")
    I = torch.empty((n_stacks, nz, 65, 65), dtype=torch.float32, device="cuda")
    Y = torch.rand_like(I)
    dc = torch.empty(4, dtype=torch.float32, device="cuda")
    dts = torch.empty(n_stacks, dtype=torch.float32, device="cuda")
    dz = torch.empty(n_stacks, dtype=torch.float32, device="cuda")

    def step():
        plan.compute(st, E=E, I=I)
        rw.adjoint_bessel(plan, st, E, (2.0 / I.numel()) * (I - Y), dc, dts, dz)

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    ms = _cuda_time(torch, step, max(3, steps // 4))
    plan.set_timing(True)
    _cuda_time(torch, step, max(3, steps // 4))
    kt = {k: plan.timing(v) for k, v in (("bessel_phi", rw.KERNEL_BESSEL_PHI),
                                          ("bessel_contract", rw.KERNEL_BESSEL_CONTRACT),
                                          ("bessel_epilogue", rw.KERNEL_BESSEL_EPILOGUE),
                                          ("adjb_radial", rw.KERNEL_ADJB_RADIAL),
                                          ("adjb_contract", rw.KERNEL_ADJB_CONTRACT),
                                          ("adjb_reduce", rw.KERNEL_ADJB_REDUCE))}
    plan.close()
    vox = n_stacks * nz * 65 * 65
    nsteps = max(3, steps // 4)         # the timed repetitions
    r_ms, r_n = kt["adjb_radial"]
    # algorithmic bytes of the transposed interpolation: E (24 B) and dL/dI (4 B) read per voxel
    bytes_per_launch = 28.0 * vox * nsteps / r_n if r_n else None
    ach = bytes_per_launch / (r_ms / r_n * 1e-3) / 1e9 if r_n else None
    return dict(workload=f"Bessel adjoint: {n_stacks} stacks of 65x65x{nz} at 20 nm, Gibson-Lanni depths "
                         "U[0, 5] um, m = 0 Zernike; step = forward (fields) + adjoint (dL/dc, dL/dt_s, dL/dz)",
                value=vox / (ms * 1e-3), unit="voxels/s (forward+adjoint)", ms_per_step=ms,
                gradient_steps_per_s=1e3 / ms,
                kernels={k: dict(total_ms=v[0], launches=v[1], avg_us=(v[0] / v[1] * 1e3 if v[1] else None))
                         for k, v in kt.items()},
                roofline=dict(kernel="adjb_radial_kernel", bound="hbm", achieved=ach and round(ach, 1),
                              peak=PEAK_HBM_GBS, unit="GB/s", frac=ach and round(ach / PEAK_HBM_GBS, 4),
                              traffic=profiled_traffic("adjb_bessel_adjoint.txt", "adjb_radial_kernel"),
                              bytes_per_launch=bytes_per_launch, avg_launch_us=r_n and r_ms / r_n * 1e3,
                              note="bound in practice by its LDS atomics and the pixels' arithmetic, not by HBM"))


def surrogate_flops_per_crop() -> float:
    """Algorithmic flops of one surrogate crop: the dense layers (22->1024->1024->1024, the
    basis branch 1024->256->4096) and the three transposed convolutions (each output takes
    Ci x 4 taps: 16x16x16 outputs x 64, 8x32x32 x 64, 64x64 x 32)."""
    dense = 22 * 1024 + 1024 * 1024 * 2 + 1024 * 256 + 256 * 4096
    conv = 16 * 16 * 16 * 64 + 8 * 32 * 32 * 64 + 64 * 64 * 32
    return 2.0 * (dense + conv)


def bench_surrogate(rw, torch, train_seconds, bar=0.1):
    """Train the surrogate for about `train_seconds` on 200000 engine crops, fit its
    error-gated fallback at the stated bar (p95 rel-L2 of the crops the network serves)
    on 8192 calibration crops, judge it on 2048 held-out crops, and time inference and
    gated serving against the plain path on 65536 inputs."""
    from paper_2502_03170_amd import surrogate_train as ST
    eng = ST.CropEngine(max_emitters=4096)
    train = ST.make_dataset(eng, 200_000, seed=505)
    calib = ST.make_dataset(eng, 8192, seed=507)
    test = ST.make_dataset(eng, 2048, seed=506)
    basis = ST.crop_basis(train, 4096)
    sg = rw.Surrogate(max_batch=65536)
    sg.set_state(ST.init_params(0, basis=basis))
    # time a short run (after a few untimed steps that absorb first-call costs) to size
    # the schedule to the budget, then one cosine schedule from fresh parameters
    ST.train(sg, train, steps=20, batch=ST.BATCH, lr=1e-5, seed=0, log_every=20)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ST.train(sg, train, steps=30, batch=ST.BATCH, lr=1e-5, seed=0, log_every=30)
    torch.cuda.synchronize()
    per_step = (time.perf_counter() - t0) / 30
    steps = max(100, int(train_seconds / per_step))
    sg.set_state(ST.init_params(0, basis=basis))
    t0 = time.perf_counter()
    ST.train(sg, train, steps=steps, batch=ST.BATCH, lr=ST.LR, lr_end=1e-5, seed=1, log_every=max(1, steps // 4))
    torch.cuda.synchronize()
    train_s = time.perf_counter() - t0
    print(f"# surrogate: {steps} training steps in {train_s:.0f} s", file=sys.stderr, flush=True)
    acc = {name: ST.audit(sg, eng, test, precision=p) for name, p in (("bf16x3", rw.SG_BF16X3), ("bf16", rw.SG_BF16))}
    gate = ST.fit_gate(sg, calib, bar)
    judged = ST.judge(sg, eng, test, gate)
    B = 65536
    serve = ST.make_dataset(eng, B, seed=508)
    coef, z = serve["coef"], serve["z"]
    out = torch.empty((B, 64, 64), dtype=torch.float32, device="cuda")
    res = {}
    flops = surrogate_flops_per_crop() * B
    for name, p in (("bf16x3", rw.SG_BF16X3), ("bf16", rw.SG_BF16)):
        sg.forward(coef, z, out=out, precision=p)
        ms = _cuda_time(torch, lambda: sg.forward(coef, z, out=out, precision=p), 5)
        res[name] = dict(ms_per_batch=ms, crops_per_s=B / (ms * 1e-3), px_per_s=B * 4096 / (ms * 1e-3),
                         tflops=flops / (ms * 1e-3) / 1e12)

    def wall(fn, reps=3):
        fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / reps * 1e3

    plain_ms = wall(lambda: eng.crops(coef, z))
    gated_ms = wall(lambda: ST.predict(sg, eng, coef, z, gate))
    _, fb = ST.predict(sg, eng, coef, z, gate)
    fallback_serve = float(fb.float().mean().item())
    # context: the plain path on a 32 x 32 pupil (its aliasing period, 6.9 um, still exceeds
    # the 6.4 um crop) against the 128 x 128 reference crops
    coarse = ST.CropEngine(max_emitters=4096, n_pupil=32)
    cc = coarse.crops(test["coef"], test["z"]) * (coarse.norm / eng.norm)
    ec = ST.rel_l2_per_crop(cc, test["target"]).cpu().numpy()
    coarse_ms = wall(lambda: coarse.crops(coef, z))
    sg.close()
    ach = res["bf16x3"]["tflops"]
    return dict(workload="surrogate: (Noll 1-21, z) -> 64x64 crop, 3.44M parameters (3 dense layers of 1024, a "
                         "256-crop basis branch and a transposed-convolution branch), trained on 200000 engine crops "
                         "(Noll 4-21 N(0,0.05), z U(+-1 um), 128x128 pupil, 100 nm pixels) for "
                         f"{steps} Adam steps of {ST.BATCH} ({train_s:.0f} s); inference batch 65536",
                value=res["bf16x3"]["px_per_s"], unit="px/s (inference, bf16x3: FP32-level products)",
                inference=res,
                roofline=dict(kernel="whole inference (dense GEMMs + fused decoder)", bound="mfma",
                              achieved=round(ach, 2), peak=PEAK_BF16_TFLOPS, unit="TFLOP/s",
                              frac=round(ach / PEAK_BF16_TFLOPS, 4),
                              traffic=profiled_traffic("sg_inference_surrogate.txt", "surrogate inference"),
                              flops_per_batch=flops, avg_launch_us=res["bf16x3"]["ms_per_batch"] * 1e3,
                              profiled_avg_us=profiled_average("sg_inference_surrogate.txt", "surrogate inference"),
                              note="bf16x3 executes three BF16 products per algorithmic one"),
                accuracy_network_vs_plain=acc,
                gate=dict(bar=f"p95 rel-L2 <= {bar} over the crops the network serves", bar_value=bar,
                          calibration_crops=8192, accepted_on_calibration=gate["accepted_calibration"],
                          error_model_corr=gate["fit_corr"]),
                judged_held_out=judged,
                serving_65536=dict(plain_ms=plain_ms, gated_ms=gated_ms, fallback_fraction=fallback_serve,
                                   gain_vs_plain=plain_ms / gated_ms,
                                   plain_crops_per_s=B / (plain_ms * 1e-3), gated_crops_per_s=B / (gated_ms * 1e-3)),
                plain_pupil_32=dict(median_rel_l2=float(np.median(ec)), p95_rel_l2=float(np.percentile(ec, 95)),
                                    ms_per_65536=coarse_ms, crops_per_s=B / (coarse_ms * 1e-3)),
                train_ms_per_step=train_s * 1e3 / steps, train_steps=steps, train_batch=ST.BATCH)


def cpu_model() -> str | None:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def _oracle_separable_rate(seconds: float, threads: int | None):
    """Voxels/s of the separable FP64 oracle (pupil build included) over the headline
    workload's stacks in order, with BLAS limited to `threads` (None: as configured)."""
    from contextlib import nullcontext

    from oracle import fourier as OF
    from tests.helpers import oracle_optics
    try:
        from threadpoolctl import threadpool_limits
        ctx = threadpool_limits(threads) if threads else nullcontext()
    except ImportError:
        ctx = nullcontext()
    w, _, _ = fourier_workload()
    opt = oracle_optics(w)
    g = OF.pupil_geometry(256, opt)
    planes = 0
    with ctx:
        t0 = time.perf_counter()
        b = 0
        while time.perf_counter() - t0 < seconds:
            s = b % 16
            P = OF.base_pupil(g, opt, OF.pupil_phase(g, opt, zernike=w["zernike"][s], t_s=w["t_s"][s]))
            for z in w["z"][s]:
                OF.field_separable(P, g, opt, 128, 128, 20.0, 20.0, [z])
                planes += 1
                if time.perf_counter() - t0 > seconds:
                    break
            b += 1
        dt = time.perf_counter() - t0
    return planes * 128 * 128 / dt, planes, dt


def _oracle_direct_rate(seconds: float):
    """Voxels/s of the brute-force double sum over the pupil (one complex exponential of
    the whole phase per cell and voxel) on seeded voxels of the first headline stack."""
    from oracle import fourier as OF
    from oracle import optics as O
    from tests.helpers import oracle_optics
    w, _, _ = fourier_workload()
    opt = oracle_optics(w)
    g = OF.pupil_geometry(256, opt)
    P = OF.base_pupil(g, opt, OF.pupil_phase(g, opt, zernike=w["zernike"][0], t_s=w["t_s"][0]))
    t0 = time.perf_counter()
    rng = np.random.default_rng(2024)
    xs, ys = O.output_axis(128, 20.0), O.output_axis(128, 20.0)
    n = 0
    try:
        from threadpoolctl import threadpool_limits
        ctx = threadpool_limits(1)
    except ImportError:
        from contextlib import nullcontext
        ctx = nullcontext()
    with ctx:
        while time.perf_counter() - t0 < seconds:
            pts = np.stack([xs[rng.integers(0, 128, 64)], ys[rng.integers(0, 128, 64)],
                            w["z"][0][rng.integers(0, 64, 64)]], axis=1)
            OF.field_direct(P, g, opt, pts)
            n += 64
    dt = time.perf_counter() - t0
    return n / dt, n, dt


def cpu_baseline(seconds: float):
    """The FP64 oracle on the host cores: the separable evaluation (whole planes, pupil
    build included) with every core BLAS uses and with one thread, and the brute-force
    double sum on seeded voxels; `seconds` is split 2 : 1 : 1 between the three."""
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        threads = 1
    affinity = len(os.sched_getaffinity(0))
    v_all, planes_all, dt_all = _oracle_separable_rate(seconds * 0.5, None)
    v_one, planes_one, dt_one = _oracle_separable_rate(seconds * 0.25, 1)
    v_dir, n_dir, dt_dir = _oracle_direct_rate(seconds * 0.25)
    return dict(value=v_all, unit="voxels/s", cores=threads, kind="oracle",
                sample=f"separable FP64 oracle (pupil build included) over the headline workload's stacks in "
                       f"order: {planes_all} planes of 128x128 (3 field components) in {dt_all:.1f} s with "
                       f"{threads} BLAS threads; the same with 1 thread: {planes_one} planes in {dt_one:.1f} s; "
                       f"brute-force double sum over the 51,468-cell disk: {n_dir} seeded voxels of stack 0 in "
                       f"{dt_dir:.1f} s (1 thread)",
                cpu_model=cpu_model(), affinity_cores=affinity, blas_threads=threads,
                single_thread=dict(value=v_one, unit="voxels/s", planes=planes_one, seconds=dt_one),
                direct_double_sum=dict(value=v_dir, unit="voxels/s", voxels=n_dir, seconds=dt_dir,
                                       threads=1))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--cpu-seconds", type=float, default=24.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--forms", default="chirpz,sweep,bessel,batched,adjoint,adjoint_bessel,surrogate",
                    help="comma list of extra forms, or 'none'")
    ap.add_argument("--train-seconds", type=float, default=150.0)
    ap.add_argument("--copy-reference", action="store_true",
                    help="also run a 256 MiB device-to-device copy (calibrates rocprofv3 byte counters)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: the library has no multi-GPU path; run with --gpus 1",
              file=sys.stderr)
        sys.exit(2)
    import torch
    import paper_2502_03170_amd as rw
    rw.load()
    if not torch.cuda.is_available():
        print("no GPU visible", file=sys.stderr)
        sys.exit(1)
    torch.cuda.synchronize()
    if args.copy_reference:
        src = torch.ones(64 << 20, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    res = bench_fourier(rw, torch, args.steps, args.warmup)
    print(f"# fourier: {res['ms_per_step']:.3f} ms/step, {res['value']:.3e} voxels/s", file=sys.stderr,
          flush=True)
    forms = {}
    if "chirpz" in args.forms.split(","):
        forms["chirpz"] = bench_chirpz(rw, torch, args.steps, args.warmup)
        print(f"# chirpz: {forms['chirpz']['ms_per_step']:.3f} ms/step", file=sys.stderr, flush=True)
    if "sweep" in args.forms.split(","):
        forms["speed_sweep"] = bench_speed_sweep(rw, torch)
        print(f"# speed sweep: {forms['speed_sweep']['ms_per_call']}", file=sys.stderr, flush=True)
    if "bessel" in args.forms.split(","):
        forms["bessel"] = bench_bessel(rw, torch, args.steps, args.warmup)
        print(f"# bessel: {forms['bessel']['value']:.3e} voxels/s", file=sys.stderr, flush=True)
    if "batched" in args.forms.split(","):
        forms["batched"] = bench_batched(rw, torch, args.steps, args.warmup)
        print(f"# batched: {forms['batched']['value']:.3e} voxels/s", file=sys.stderr, flush=True)
    if "adjoint" in args.forms.split(","):
        forms["adjoint"] = bench_adjoint(rw, torch, args.steps, args.warmup)
        print(f"# adjoint: {forms['adjoint']['ms_per_step']:.2f} ms/step", file=sys.stderr, flush=True)
    if "adjoint_bessel" in args.forms.split(","):
        forms["adjoint_bessel"] = bench_adjoint_bessel(rw, torch, args.steps, args.warmup)
        print(f"# adjoint_bessel: {forms['adjoint_bessel']['ms_per_step']:.2f} ms/step", file=sys.stderr,
              flush=True)
    if "surrogate" in args.forms.split(","):
        forms["surrogate"] = bench_surrogate(rw, torch, args.train_seconds)
        print(f"# surrogate: {forms['surrogate']['serving_65536']}", file=sys.stderr, flush=True)
    cpu = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(args.cpu_seconds)
    out = {
        "metric": "PSF voxels/sec (vectorial FP32) plain vs batched/surrogate at rel-L2 \u22641e-5",
        "value": res["value"], "unit": "voxels/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": res["ms_per_step"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "fourier_plain: NA 1.4, 600 nm, n_i 1.518, 256x256 pupil, Gibson-Lanni "
                               "(n_s 1.33, t_s U[0,5] um) + Noll 4-21 N(0,0.05) waves, 128x128x64 at "
                               "20 nm, fields + intensity, 16 stacks per call",
                   "stacks_per_step": 16, "voxels_per_step": res["voxels"], "form": "fourier"},
        "roofline": res["roofline"],
        "cpu_baseline": cpu,
        "kernels": res["kernels"],
        "image_gemm": res["image_gemm"],
        "step_tflops": res["step_tflops"], "step_frac": res["step_frac"],
        "forms": forms,
    }
    print(json.dumps(out))


if __name__ == "__main__":
    main()
