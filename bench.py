"""Benchmark of the Pinv-Recon hot path on one MI355X.

Default workload (the shape the R-build bar is stated at): 128x128 image
(N=16384), 8 coils, variable-density spiral of 2N = 32768 samples per coil
(M=262144), 1000 dynamic frames, shift 1e-3 * mean diag(E^H E).

One step = build R with the FP32 path from the encoding alone (Gram through the
point-spread function in FP64, FP64 blocked Cholesky with L^-1, W = L^-1 E^H
and R = L^-H W on FP32 MFMA), then reconstruct all frames (image = R data)
with the refinement steps needed for 1e-5 relative error against the plain
FP64 GPU path.  Inputs are resident in HBM before the timed region; every step
builds a fresh, uncached plan.

value = executed complex-equivalent TFLOP/s of the whole step: the work the
kernels run (PSF Gram 8K(2nx-1)(2ny-1) + coil products 8CN^2, Cholesky with
L^-1 8N^3/3, W 4MN^2, R 4MN^2, apply 8NMF, refinement 8MNF + 16N^2F per step)
divided by the step time.  The standard count of a normal-equation build
(12MN^2 + 4N^3/3: a Gram over all M rows) is reported beside it, labelled as
an effective rate, since the PSF Gram does not run those flops.

The JSON line also carries the build's stage times and executed rate, apply
frames/s (plain and refined), the FP32 plan with R formed in FP64 (no
refinement needed), the BF16-split and factor-only plans, the plain FP64 GPU
comparator, few-frame applies against HBM bandwidth, the 64x64 / 8-coil
workload's figures, a roofline entry for the dominant kernel and the CPU
oracle baseline.
"""
from __future__ import annotations

import argparse
import json
import os
import platform
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

METRIC = "R-build TFLOP/s + apply frames/s vs plain FP64 GPU at stated error; p50/p99"
PEAK_FP64_MFMA = 78.6
PEAK_BF16_MFMA = 2500.0  # TFLOP/s, MI355X dense BF16 matrix (no sparsity)
PEAK_F16_MFMA = 2500.0   # TFLOP/s, MI355X dense FP16 matrix (no sparsity)
# FP32 products on f16 pieces: executed f16 flops per complex-equivalent flop (16 or 12
# real products of pieces per complex product against the 4 counted)
F16_TRMM, F16_APPLY = 4.0, 3.0
PEAK_HBM = 8.0e12        # B/s
ROW_APPLY_MAX_F = 2      # FP32 and BF16X3 plans stream R row by row (VALU) for at most this many frames,
STREAM_MAX_F = 32        # and into the matrix cores up to this many


def log(*a):
    print(*a, file=sys.stderr, flush=True)


# ----------------------------------------------------------------------------
# work counts (complex-equivalent: 8 real flops per complex multiply-add)
# ----------------------------------------------------------------------------

def gram_flops_executed(enc, form: str) -> float:
    N, K, C, S = enc.N, enc.K, enc.C, enc.S
    if form == "psf":
        return 8.0 * K * (2 * enc.nx - 1) * (2 * enc.ny - 1) * S * S + 8.0 * C * N * N
    if form == "shared":
        return 4.0 * K * N * N + 8.0 * C * N * N / 2
    return 4.0 * enc.M * N * N


def build_flops_executed(enc, form: str = "psf") -> dict:
    N, M = enc.N, enc.M
    if M < N:
        # right pseudoinverse: the M x M Gram E E^H over the N unknowns (lower
        # triangle), its factor and inverse, Z = L'^-1 E and R^H = L'^-H Z
        return {"gram": 4.0 * N * M * M, "chol_inv": 8.0 * M ** 3 / 3.0,
                "trmm_w": 4.0 * N * M * M, "trmm_r": 4.0 * N * M * M}
    return {"gram": gram_flops_executed(enc, form), "chol_inv": 8.0 * N ** 3 / 3.0,
            "trmm_w": 4.0 * M * N * N, "trmm_r": 4.0 * M * N * N}


def bf16x3_mfma(ex: dict, stage_ms: dict, apply_ms_=None, F=0, enc=None) -> dict:
    """BF16 MFMA rates of a BF16X3 plan's products: each complex multiply-add
    runs 3 split products x 4 real products (24 bf16 flops, 3x the 8 counted
    complex-equivalent), against the dense BF16 peak."""
    out = {}
    for k in ("trmm_w", "trmm_r"):
        t = stage_ms[k] * 1e-3
        out[k] = {"bf16_tflops": 3.0 * ex[k] / t / 1e12, "frac_bf16_peak": 3.0 * ex[k] / t / 1e12 / PEAK_BF16_MFMA}
    if apply_ms_:
        fl = 3.0 * 8.0 * F * enc.M * enc.N
        out["apply"] = {"bf16_tflops": fl / (apply_ms_ * 1e-3) / 1e12,
                        "frac_bf16_peak": fl / (apply_ms_ * 1e-3) / 1e12 / PEAK_BF16_MFMA}
    out["peak"] = PEAK_BF16_MFMA
    return out


def build_flops_standard(enc) -> float:
    N, M = enc.N, enc.M
    return 12.0 * M * N * N + 4.0 * N ** 3 / 3.0


def refine_flops(enc, F: int, steps: int) -> float:
    if steps <= 0:
        return 0.0
    N, M = enc.N, enc.M
    adjoint = 8.0 * M * N * F
    if enc.b0_hz is None:   # E^H d by gridding: 529 cells by real weights, two transforms
        rows, img = F * enc.C * enc.S, enc.nx * enc.ny
        adjoint = min(adjoint, rows * (4.0 * 529 * enc.K + 8.0 * img * (4 * enc.nx + 2 * enc.ny)))
    return adjoint + steps * 16.0 * N * N * F


# ----------------------------------------------------------------------------
# CPU oracle baseline
# ----------------------------------------------------------------------------

def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or "unknown"


def cpu_baseline(enc, rows: int = 4096) -> dict:
    """The oracle's Gram (explicit FP64 E, E_b^H E_b with a library matmul) over
    the first `rows` rows of the workload's encoding: one row block of the sum
    over all M rows it forms for a full build, about 10-20 s on the host."""
    import oracle
    from threadpoolctl import threadpool_info
    sub = type(enc)(enc.nx, enc.ny, enc.k[:rows], t=None if enc.t is None else enc.t[:rows],
                    coil=None if enc.coil is None else enc.coil[:1], b0_hz=enc.b0_hz,
                    species_hz=enc.species_hz)
    t0 = time.perf_counter()
    oracle.gram(sub)
    dt = time.perf_counter() - t0
    flops = 4.0 * rows * enc.N * enc.N
    blas = [p.get("num_threads", 0) for p in threadpool_info() if p.get("user_api") == "blas"]
    threads = max(blas) if blas else 1
    full_s = dt * (4.0 * enc.M * enc.N ** 2) / flops
    return {"value": flops / dt / 1e12, "unit": "TFLOP/s", "cores": threads, "kind": "oracle",
            "sample": f"oracle Gram over the first {rows} of M={enc.M} rows (N={enc.N}, E formed "
                      f"explicitly in FP64, one coil): {flops:.3g} complex-equivalent flops in "
                      f"{dt:.2f} s; the full Gram alone would take about {full_s:.0f} s",
            "cpu_model": cpu_model(), "affinity_cores": len(os.sched_getaffinity(0)),
            "blas_threads": threads}


# ----------------------------------------------------------------------------
# HBM traffic of the dominant kernels from the counter record
# ----------------------------------------------------------------------------

DEVICE_SOURCES = ("pinv_device.h", "pinv_internal.h", "pinv_trmm.hip", "pinv_apply.hip",
                  "pinv_split.hip", "pinv_half.hip")


def kernel_source_hash() -> str:
    """Hash of the device sources the counted kernels come from; counter
    readings are valid only for this hash."""
    import hashlib
    h = hashlib.sha256()
    for f in DEVICE_SOURCES:
        with open(os.path.join(ROOT, "paper_2410_06129_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(kernel: str, workload: str):
    """HBM bytes per launch of `kernel` from profiles/pmc_traffic.json (FETCH_SIZE
    and WRITE_SIZE counter runs, scaled by a plain copy of known size), or None
    if no reading exists for the current sources and this workload."""
    path = os.path.join(ROOT, "profiles", "pmc_traffic.json")
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        rec = json.load(fh)
    if (rec.get("source_hash") != kernel_source_hash() or rec.get("workload") != workload
            or kernel not in rec.get("kernels", {})):
        return None
    k = rec["kernels"][kernel]
    return {"bytes_per_launch": k["fetch_bytes"] + k["write_bytes"], "fetch_bytes": k["fetch_bytes"],
            "write_bytes": k["write_bytes"], "algorithmic_bytes": k.get("algorithmic_bytes"),
            "source": "profiles/pmc_traffic.json"}


# the FP32 plan's kernels (f16 pieces) and the BF16X3 plan's split
# kernels, by their template signature
PMC_KERNELS = {"trmm_w": "k_trmm_wh(",
               "trmm_r": "k_trmm_rh(",
               "apply": "k_apply_half<pinv::HalfCfg<128, 128,",
               "trmm_w_bf16x3": "k_trmm_w_sp(",
               "trmm_r_bf16x3": "k_trmm_r_sp(",
               "apply_bf16x3": "k_apply<pinv::TileCfgB3<128, 64, 2, 2, 1>, false>",
               # few-frame applies, one launch each in the counter run (FP32 3M
               # plan: rows at 1 frame, streamed at 16 and 32; BF16X3: 16)
               "apply_rows_f1": "k_apply_rows<float, 1, 1, 2>",
               "apply_stream_f16": "k_apply_stream<1, 2, 2, 1>",
               "apply_stream_f32": "k_apply_stream<2, 2, 2, 1>",
               "apply_stream_bf16x3_f16": "k_apply_stream<1, 2, 2, 2>"}
FEW_FRAMES = {"apply_rows_f1": 1, "apply_stream_f16": 16, "apply_stream_f32": 32,
              "apply_stream_bf16x3_f16": 16}


def algorithmic_bytes(N: int, M: int, F: int) -> dict:
    """Compulsory HBM bytes per launch (8 bytes per complex value, complex64 or
    split-packed): L^-1 lower triangle read and W written once; L^-1 (or L^-H)
    and W read and R written once; for the apply D, R and X once."""
    tri = 8.0 * N * N / 2
    out = {"trmm_w": tri + 8.0 * N * M, "trmm_r": tri + 16.0 * N * M,
           "apply": 8.0 * F * M + 8.0 * N * M + 8.0 * F * N}
    for k in ("trmm_w", "trmm_r", "apply"):
        out[k + "_bf16x3"] = out[k]
    for k, f in FEW_FRAMES.items():
        out[k] = 8.0 * f * M + 8.0 * N * M + 8.0 * f * N
    return out


def pmc_mfma_summary(d) -> dict:
    """Per-kernel MFMA counters of one rocprofv3 --pmc run of `bench.py
    --pmc-run`: busy = SQ_VALU_MFMA_BUSY_CYCLES / (GRBM_GUI_ACTIVE / 8 XCDs x
    1024 SIMDs), executed matrix flops = SQ_INSTS_VALU_MFMA_MOPS_* x 512, LDS
    bank-conflict cycles per CU over the kernel's cycles."""
    import sqlite3
    import glob
    from collections import defaultdict
    db = sorted(glob.glob(os.path.join(d, "**", "*results.db"), recursive=True))[0]
    con = sqlite3.connect(db)
    rows = con.execute("select kernel_name, counter_name, value, dispatch_id from counters_collection").fetchall()
    con.close()
    agg = defaultdict(lambda: defaultdict(float))
    disp = defaultdict(set)
    names = dict(PMC_KERNELS, gram_psf="k_psf(", chol_trailing="k_chol_trailing", chol_panel="k_chol_panel",
                 gen_e_bf16x3="k_gen_e_sp<", gram_shared="k_gram_shared<", gram_full="k_gram<",
                 chol_diag="k_chol_diag", gen_e_half="k_gen_e_h<", apply_pack="k_pack_half<", adjoint_fp64="k_grid_spread<", resid="k_resid", tri_frames="k_tri_frames",
                 trmm_w_fp64_formed="k_trmm_w<pinv::TileCfg<double",
                 trmm_r_fp64_formed="k_trmm_r<pinv::TileCfg<double, 64, 64, 8, false, 2>, float>",
                 apply_seg="k_apply<pinv::TileCfg<float, 128, 64, 8, false, 2>, true>")
    for k, c, v, did in rows:
        for key, pat in names.items():
            if pat in k:
                agg[key][c] += v
                disp[key].add(did)
    out = {"source_hash": kernel_source_hash(), "kernels": {}}
    for key, a in agg.items():
        g = a.get("GRBM_GUI_ACTIVE", 0.0) / 8
        if g <= 0:
            continue
        mops = {t: a.get("SQ_INSTS_VALU_MFMA_MOPS_" + t, 0.0) * 512 for t in ("F32", "F64", "BF16", "F16")}
        out["kernels"][key] = {"dispatches": len(disp[key]), "cycles_per_xcd": g,
                               "mfma_busy": a.get("SQ_VALU_MFMA_BUSY_CYCLES", 0.0) / (g * 1024),
                               "lds_bank_conflict_frac": a.get("SQ_LDS_BANK_CONFLICT", 0.0) / 256 / g,
                               "mfma_flops_executed": {t: v for t, v in mops.items() if v}}
    return out


def pmc_summary(dirs, frames: int) -> dict:
    """HBM bytes per product (build) or apply of the dominant kernels from two
    rocprofv3 counter runs of `bench.py --pmc-run` (FETCH_SIZE, WRITE_SIZE; KiB
    per dispatch, summed over a product's launches), scaled by what the same
    counters read for the plain 2 GiB copy it runs first."""
    import sqlite3
    import glob

    def read(d, counter):
        db = sorted(glob.glob(os.path.join(d, "**", "*results.db"), recursive=True))[0]
        con = sqlite3.connect(db)
        rows = con.execute("select kernel_name, value from counters_collection where counter_name = ?",
                           (counter,)).fetchall()
        con.close()
        return rows

    from paper_2410_06129_amd import synth
    w = synth.spiral_128x128_c8(F=1)
    N, M = w.enc.N, w.enc.M
    alg = algorithmic_bytes(N, M, frames)
    vals = {}
    for counter, d in zip(("FETCH_SIZE", "WRITE_SIZE"), dirs):
        rows = read(d, counter)
        copy = max(v for n, v in rows if "copyBuffer" in n or "elementwise_kernel" in n)
        per = {}
        for key, pat in PMC_KERNELS.items():
            # the run builds and applies each kind once; the BF16X3 W product is
            # one launch per conj(E) slab, summed to the product's bytes
            xs = [v for n, v in rows if pat in n]
            per[key] = sum(xs) if xs else None
        vals[counter] = (copy, per)
    copy_bytes = 2.0 ** 31
    fscale = copy_bytes / (vals["FETCH_SIZE"][0] * 1024.0)
    wscale = copy_bytes / (vals["WRITE_SIZE"][0] * 1024.0)
    rec = {"source_hash": kernel_source_hash(), "workload": w.name.replace("_f1", f"_f{frames}"),
           "commands": [f"rocprofv3 --pmc {c} -d <out> -o run -- python3 bench.py --pmc-run"
                        for c in ("FETCH_SIZE", "WRITE_SIZE")],
           "calibration": {"kernel": "2 GiB device copy", "fetch_kib": vals["FETCH_SIZE"][0],
                           "write_kib": vals["WRITE_SIZE"][0], "fetch_scale": fscale,
                           "write_scale": wscale},
           "kernels": {}}
    for key in PMC_KERNELS:
        fk, wk = vals["FETCH_SIZE"][1][key], vals["WRITE_SIZE"][1][key]
        if fk is None or wk is None:
            continue
        rec["kernels"][key] = {"fetch_kib": fk, "write_kib": wk, "fetch_bytes": fk * 1024.0 * fscale,
                               "write_bytes": wk * 1024.0 * wscale, "algorithmic_bytes": alg[key]}
    return rec


# ----------------------------------------------------------------------------
# helpers on the device
# ----------------------------------------------------------------------------

class Timer:
    """HIP events on the launch stream."""

    def __init__(self, stream):
        import torch
        self.stream = stream
        self.e0 = torch.cuda.Event(enable_timing=True)
        self.e1 = torch.cuda.Event(enable_timing=True)

    def __enter__(self):
        self.e0.record(self.stream)
        return self

    def __exit__(self, *exc):
        import torch
        self.e1.record(self.stream)
        torch.cuda.synchronize()
        self.ms = self.e0.elapsed_time(self.e1)


def stage_dict(st):
    return {"gram": float(st[0]), "chol_inv": float(st[1]), "trmm_w": float(st[2]),
            "trmm_r": float(st[3])}


def make_inputs(P, ctx, w, F, dev, seed=2026):
    """data = E x (FP64 GPU forward of the ground-truth frames) + complex
    Gaussian noise at the workload's SNR, drawn on the device from a seeded
    generator; and the reference images x_ref from a factor-only FP64 plan
    (L^-H L^-1 E^H d with one FP64 refinement step).  Returns d64, d32, x_ref."""
    import torch
    enc = w.enc
    N, M = enc.N, enc.M
    q = P.pinv_build(ctx, enc, w.rel_lambda, P.LAMBDA_REL_MEAN_DIAG, P.FP64,
                     P.FLAG_UNCACHED | P.FLAG_NO_R)
    P.pinv_plan_wait(q)
    x_true = torch.from_numpy(np.ascontiguousarray(w.images[:F])).to(dev)
    d64 = torch.empty((F, M), dtype=torch.complex128, device=dev)
    P.pinv_forward(ctx, q, x_true, d64)
    sigma = torch.sqrt(torch.mean(torch.abs(d64) ** 2)) * 10 ** (-w.snr_db / 20)
    if w.noise.shape[0] >= F:
        noise = torch.from_numpy(np.ascontiguousarray(w.noise[:F])).to(dev)
    else:
        g = torch.Generator(device=dev).manual_seed(seed)
        noise = torch.randn((F, M), dtype=torch.complex128, device=dev, generator=g)
    d64 += sigma * noise
    del noise, x_true
    x_ref = torch.empty((F, N), dtype=torch.complex128, device=dev)
    P.pinv_apply(ctx, q, d64, x_ref, refine_steps=1)
    torch.cuda.synchronize()
    P.pinv_plan_release(q)
    d32 = d64.to(torch.complex64)
    return d64, d32, x_ref


def rel_err(x, x_ref):
    import torch
    e = (torch.linalg.vector_norm(x.to(torch.complex128) - x_ref, dim=1)
         / torch.linalg.vector_norm(x_ref, dim=1))
    return float(e.max()), float(e.median())


def build_timed(P, ctx, enc, rel, prec, flags=0, **kw):
    p = P.pinv_build(ctx, enc, rel, P.LAMBDA_REL_MEAN_DIAG, prec, flags | P.FLAG_UNCACHED, **kw)
    P.pinv_plan_wait(p)
    return p, P.pinv_plan_info_get(p)["stage_ms"]


def apply_ms(P, ctx, plan, d, x, stream, refine=0, reps=3):
    ts = []
    for _ in range(reps):
        with Timer(stream) as t:
            P.pinv_apply(ctx, plan, d, x, refine_steps=refine)
        ts.append(t.ms)
    return float(np.median(ts))


def metric_timings(P, ctx, plan, enc, stream, dev, reps: int = 3) -> dict:
    """SRF (Eq. 9) and noise matrix (Eq. 10) of an FP32 plan: median HIP-event
    time per call on the launch stream, with the rate against each kernel's
    bound (HBM bytes 8NM for the maps, complex-equivalent flops for the full
    matrices: 8MN^2 for R E, 4MN^2 for the Hermitian R R^H)."""
    import torch
    N, M, C = enc.N, enc.M, enc.C
    rng = np.random.default_rng(99)
    a = rng.standard_normal((C, C)) + 1j * rng.standard_normal((C, C))
    psi_c = a @ a.conj().T + C * np.eye(C)
    out_d = torch.empty((N,), dtype=torch.complex64, device=dev)
    out_f = torch.empty((N, N), dtype=torch.complex64, device=dev)
    out_r = torch.empty((N,), dtype=torch.float32, device=dev)
    runs = {
        "srf_map": (lambda: P.pinv_srf(ctx, plan, out_d, P.METRIC_DIAG), "GB/s", 8.0 * N * M),
        "srf_matrix": (lambda: P.pinv_srf(ctx, plan, out_f, P.METRIC_FULL), "TFLOP/s", 8.0 * M * N * N),
        "noise_map_white": (lambda: P.pinv_noise(ctx, plan, out_r, mode=P.METRIC_DIAG), "GB/s",
                            8.0 * N * M),
        "noise_map_coils": (lambda: P.pinv_noise(ctx, plan, out_r, coil_cov=psi_c, mode=P.METRIC_DIAG),
                            "GB/s", 8.0 * N * M),
        "noise_matrix_white": (lambda: P.pinv_noise(ctx, plan, out_f, mode=P.METRIC_FULL), "TFLOP/s",
                               4.0 * M * N * N),
        "noise_matrix_coils": (lambda: P.pinv_noise(ctx, plan, out_f, coil_cov=psi_c,
                                                    mode=P.METRIC_FULL), "TFLOP/s", 4.0 * M * N * N),
    }
    res = {}
    for name, (fn, unit, work) in runs.items():
        fn()
        torch.cuda.synchronize()
        ts = []
        for _ in range(reps):
            with Timer(stream) as t:
                fn()
            ts.append(t.ms)
        ms = float(np.median(ts))
        rate = work / (ms * 1e-3) / (1e9 if unit == "GB/s" else 1e12)
        res[name] = {"ms": ms, unit: rate}
        log(f"metric {name}: {ms:.3f} ms, {rate:.1f} {unit}")
    return res


# ----------------------------------------------------------------------------
# the 64x64 / 8-coil workload (earlier headline; kept for continuity)
# ----------------------------------------------------------------------------

def config2_figures(P, ctx, stream, dev, tol) -> dict:
    import torch
    from paper_2410_06129_amd import synth
    w = synth.spiral_64x64_c8(F=1000)
    enc = w.enc
    N, M, F = enc.N, enc.M, 1000
    d64, d32, x_ref = make_inputs(P, ctx, w, F, dev)
    x32 = torch.empty((F, N), dtype=torch.complex64, device=dev)
    out = {"workload": w.name, "N": N, "M": M, "F": F}
    p, st = build_timed(P, ctx, enc, w.rel_lambda, P.FP32)
    refine = None
    errs = {}
    for r in range(3):
        P.pinv_apply(ctx, p, d32, x32, refine_steps=r)
        torch.cuda.synchronize()
        errs[str(r)] = rel_err(x32, x_ref)[0]
        if refine is None and errs[str(r)] <= tol:
            refine = r
    refine = 2 if refine is None else refine
    builds = []
    for _ in range(3):
        q, stq = build_timed(P, ctx, enc, w.rel_lambda, P.FP32)
        builds.append(sum(stq))
        P.pinv_plan_release(q)
    a0 = apply_ms(P, ctx, p, d32, x32, stream)
    ar = apply_ms(P, ctx, p, d32, x32, stream, refine=refine)
    out["fp32"] = {"build_ms": float(np.median(builds)), "stage_ms": stage_dict(st),
                   "apply_frames_per_s": F / (a0 * 1e-3),
                   "apply_refined_frames_per_s": F / (ar * 1e-3), "refine_steps": refine,
                   "rel_err_by_refine_steps": errs}
    out["metrics_fp32_plan"] = metric_timings(P, ctx, p, enc, stream, dev)
    P.pinv_plan_release(p)
    q, stq = build_timed(P, ctx, enc, w.rel_lambda, P.FP32, P.FLAG_R_FP64)
    P.pinv_apply(ctx, q, d32, x32)
    torch.cuda.synchronize()
    out["fp32_r_fp64"] = {"build_ms": float(sum(stq)), "rel_err_unrefined": rel_err(x32, x_ref)[0],
                          "apply_frames_per_s": F / (apply_ms(P, ctx, q, d32, x32, stream) * 1e-3)}
    P.pinv_plan_release(q)
    q, stq = build_timed(P, ctx, enc, w.rel_lambda, P.FP64)
    x64 = torch.empty((F, N), dtype=torch.complex128, device=dev)
    out["fp64_gpu"] = {"build_ms": float(sum(stq)),
                       "apply_frames_per_s": F / (apply_ms(P, ctx, q, d64, x64, stream) * 1e-3)}
    P.pinv_plan_release(q)
    log(f"64x64 workload: {out}")
    P.pinv_context_trim(ctx)
    return out


# ----------------------------------------------------------------------------
# other modes
# ----------------------------------------------------------------------------

class RequestArena:
    """Request buffers of the serving replay carved first-fit out of one device
    buffer, so that they never take more than its bytes whatever the mix of
    sizes (freed buffers in torch's cache would otherwise stay reserved beyond
    the data cap, beside the plans).  Ranges are 256-byte aligned."""

    def __init__(self, nbytes: int):
        import torch
        self.buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        self.free = [(0, nbytes)]   # (offset, size), sorted by offset, disjoint

    @staticmethod
    def _round(n: int) -> int:
        return (n + 255) & ~255

    def alloc(self, n: int):
        n = self._round(n)
        for i, (o, sz) in enumerate(self.free):
            if sz >= n:
                if sz == n:
                    del self.free[i]
                else:
                    self.free[i] = (o + n, sz - n)
                return o
        return None

    def release(self, o: int, n: int) -> None:
        n = self._round(n)
        i = 0
        while i < len(self.free) and self.free[i][0] < o:
            i += 1
        self.free.insert(i, (o, n))
        if i + 1 < len(self.free) and o + n == self.free[i + 1][0]:   # merge the next range
            self.free[i] = (o, n + self.free[i + 1][1])
            del self.free[i + 1]
        if i > 0 and self.free[i - 1][0] + self.free[i - 1][1] == o:   # and the previous one
            self.free[i - 1] = (self.free[i - 1][0], self.free[i - 1][1] + self.free[i][1])
            del self.free[i]

    def view(self, o: int, shape, dtype):
        import torch
        es = torch.empty((), dtype=dtype).element_size()
        n = es * int(np.prod(shape))
        return self.buf[o:o + n].view(dtype).view(shape)


def serving(args) -> dict:
    """Replay the seeded serving trace (Poisson arrivals; sizes 32^2..128^2 with
    probabilities .4/.3/.2/.1; 1, 8 or 16 coils; spiral of 2N samples per coil;
    70% of requests reuse an earlier encoding; frames uniform in [50, 2000])
    through the server, once per variant.  Request buffers (data and image)
    come first-fit from one device arena of the data cap; a request waits for
    room.  Latency = completion - scheduled arrival (queueing included).  A request that fails (its plan exceeds the
    budget) counts as never served: p50/p99 are over all requests, failures
    at infinite latency, and over the requests served by every variant."""
    import torch
    from paper_2410_06129_amd import pinv as P
    from paper_2410_06129_amd import synth

    trace = synth.serving_trace(rate_per_s=args.rate, duration_s=args.duration)
    encs = {}
    for r in trace:
        if r.enc_id not in encs:
            encs[r.enc_id] = synth.serving_encoding(r.n, r.coils, r.enc_id)
    res = {"requests": len(trace), "rate_per_s": args.rate, "duration_s": args.duration,
           "frames_range": [50, 2000]}
    variants = {"fp32_refined": (P.FP32, torch.complex64, args.serve_refine, 0),
                "fp32_r_fp64": (P.FP32, torch.complex64, 0, P.FLAG_R_FP64),
                "fp64": (P.FP64, torch.complex128, 0, 0),
                "fp32_unrefined": (P.FP32, torch.complex64, 0, 0),
                "bf16x3_refined": (P.BF16X3, torch.complex64, args.serve_refine, 0)}
    lat_by = {}
    for label in args.serve_variants.split(","):
        prec, cdt, refine, flags = variants[label]
        ctx = P.pinv_context_create(0)
        torch.cuda.reset_peak_memory_stats()
        free, total = torch.cuda.mem_get_info()
        srv = P.pinv_server_create(ctx, 0, hbm_budget_bytes=int(free * args.plan_frac),
                                   max_group=16, max_inflight=2, max_builds=1)
        data_cap = int(free * (0.85 - args.plan_frac))
        log(f"[{label}] device free {free / 2**30:.1f} of {total / 2**30:.1f} GiB; plan budget "
            f"{free * args.plan_frac / 2**30:.1f} GiB, data cap {data_cap / 2**30:.1f} GiB")
        arena = RequestArena(data_cap)
        live = {}
        sched = {}
        done = []
        t0 = time.perf_counter()

        def reap():
            for c in P.pinv_server_poll(srv, 1024):
                done.append((c, time.perf_counter() - t0))
                off, nb = live.pop(c["tag"])
                arena.release(off, nb)

        flops_offered = 0.0
        for r in trace:
            enc = encs[r.enc_id]
            N, M, F = enc.N, enc.M, r.frames
            while time.perf_counter() - t0 < r.arrival_s:
                reap()
                time.sleep(0.001)
            es = 8 if prec != P.FP64 else 16
            dbytes = RequestArena._round(M * F * es)
            nbytes = dbytes + N * F * es
            while True:        # back-pressure on request buffers (counts as queueing)
                reap()
                off = arena.alloc(nbytes)
                if off is not None:
                    break
                if not live:
                    raise RuntimeError(f"request {r.rid} ({nbytes} B) exceeds the data arena")
                time.sleep(0.002)
            g = torch.Generator(device="cuda").manual_seed(r.rid)
            d = arena.view(off, (F, M), cdt)
            x = arena.view(off + dbytes, (F, N), cdt)
            torch.randn((F, M), dtype=cdt, device="cuda", generator=g, out=d)
            torch.cuda.current_stream().synchronize()
            live[r.rid] = (off, nbytes)
            sched[r.rid] = r.arrival_s
            P.pinv_server_submit(srv, enc, d, x, 1e-3, P.LAMBDA_REL_MEAN_DIAG, prec, flags=flags,
                                 refine_steps=refine, tag=r.rid)
            flops_offered += 8.0 * N * M * F + (build_flops_standard(enc) if r.new_build else 0)
            log(f"[{label}] t={time.perf_counter() - t0:7.2f}s submitted {r.rid} n={r.n} C={r.coils} "
                f"F={F} new={r.new_build}; done {len(done)}")
        while len(done) < len(trace):
            reap()
            time.sleep(0.002)
        t_end = time.perf_counter() - t0
        st = P.pinv_server_stats_get(srv)
        torch_peak = torch.cuda.max_memory_reserved()   # request buffers held by torch's cache
        P.pinv_server_destroy(srv)
        live.clear()
        d = x = None   # the last request's views hold the arena's buffer
        del arena
        P.pinv_context_destroy(ctx)
        torch.cuda.empty_cache()
        lat = {c["tag"]: (tw - sched[c["tag"]] if c["status"] == P.OK else float("inf"))
               for c, tw in done}
        lat_by[label] = lat
        ok = np.array([v for v in lat.values() if np.isfinite(v)])
        allv = np.array(list(lat.values()))
        fails = {}
        for c, _ in done:
            if c["status"] != P.OK:
                k = P.pinv_status_string(c["status"])
                fails[k] = fails.get(k, 0) + 1
        def pct(v, q):
            # nearest-rank percentile; a failed request counts as never served,
            # so a percentile that falls on one is reported as "unserved"
            x = float(np.percentile(v, q, method="higher"))
            return x if np.isfinite(x) else "unserved"

        res[label] = {"p50_s": pct(allv, 50), "p99_s": pct(allv, 99),
                      "p50_served_s": float(np.percentile(ok, 50)),
                      "p99_served_s": float(np.percentile(ok, 99)),
                      "completed_ok": int(len(ok)), "failed": int(len(allv) - len(ok)),
                      "failures": fails, "refine_steps": refine,
                      "throughput_req_per_s": len(ok) / t_end, "makespan_s": t_end,
                      "offered_tflops_standard": flops_offered / args.duration / 1e12,
                      "served_tflops_standard": flops_offered / t_end / 1e12,
                      "builds": st["builds"], "hits": st["hits"], "evictions": st["evictions"],
                      "batches": st["batches"], "peak_plan_bytes": st["peak_used"],
                      "torch_peak_reserved_bytes": torch_peak,
                      "invariant_violations": st["invariant_violations"]}
        log(f"[{label}] {res[label]}")
    common = set.intersection(*[{t for t, v in l.items() if np.isfinite(v)} for l in lat_by.values()])
    res["common_requests"] = len(common)
    for label, lat in lat_by.items():
        v = np.array([lat[t] for t in common])
        if len(v):
            res[label]["p50_common_s"] = float(np.percentile(v, 50))
            res[label]["p99_common_s"] = float(np.percentile(v, 99))
    return res


def eigen_study(args) -> dict:
    """The eigenvalue route (Eq. 7; truncation, Eq. 4) at moderate N: FP64 plans
    of SIDE^2 images with 8 coils and a spiral of 2N samples per coil, built
    once uncached.  Per build: Jacobi sweeps, kept rank, stage times (Gram,
    eigendecomposition + truncation + Q^H, W, R).  The Jacobi stage's rate
    counts the rotation passes' compulsory bytes, 64 N^2 per step (A and V
    read and their rotated copies written, complex128) over np - 1 steps a
    sweep, against 8 TB/s; the stage time also holds the per-sweep norms and
    host check, the ranking and Q^H.  The spectrum is checked against
    numpy.linalg.eigvalsh of the plan's own FP64 Gram, and the plain
    Cholesky FP64 build of the same encoding is timed beside it."""
    import torch
    from paper_2410_06129_amd import pinv as P
    from paper_2410_06129_amd import synth

    ctx = P.pinv_context_create(0)
    out = {"coils": 8, "builds": []}
    for side in [int(x) for x in args.eigen_sides.split(",")]:
        enc = synth.serving_encoding(side, 8, 0)
        N, M = enc.N, enc.M
        rec = {"side": side, "N": N, "M": M}
        for label, kw in (("eigen_kappa100", dict(route=P.ROUTE_EIGEN, trunc=P.TRUNC_KAPPA,
                                                  trunc_value=100.0)),
                          ("cholesky", {})):
            t0 = time.perf_counter()
            p = P.pinv_build(ctx, enc, 1e-3, P.LAMBDA_REL_MEAN_DIAG, P.FP64, P.FLAG_UNCACHED, **kw)
            P.pinv_plan_wait(p)
            wall = (time.perf_counter() - t0) * 1e3
            info = P.pinv_plan_info_get(p)
            r = {"wall_ms": wall, "stage_ms": dict(zip(("gram", "factor", "trmm_w", "trmm_r"),
                                                       info["stage_ms"]))}
            if label.startswith("eigen"):
                sweeps = info["sweeps"]
                steps = sweeps * (N + N % 2 - 1)
                nbytes = 64.0 * N * N * steps
                ms = info["stage_ms"][1]
                spec = torch.empty((N,), dtype=torch.float64, device="cuda")
                P.pinv_spectrum(ctx, p, spec)
                G = torch.empty((N, N), dtype=torch.complex128, device="cuda")
                P.pinv_plan_copy_buffer(p, P.BUF_GRAM, G)
                torch.cuda.synchronize()
                ref = np.linalg.eigvalsh(G.cpu().numpy())
                got = np.sort(spec.cpu().numpy())
                del G
                r.update(sweeps=sweeps, rank=info["rank"], rotation_steps=steps,
                         jacobi_bytes=nbytes, jacobi_GBps=nbytes / (ms * 1e-3) / 1e9,
                         jacobi_hbm_frac=nbytes / (ms * 1e-3) / PEAK_HBM,
                         spectrum_max_abs_err_rel=float(np.abs(got - ref).max() / np.abs(ref).max()))
            rec[label] = r
            P.pinv_plan_release(p)
            P.pinv_context_trim(ctx)
            log(f"eigen study {side}^2 {label}: {r}")
        out["builds"].append(rec)
    P.pinv_context_destroy(ctx)
    return out


def precision_study(args) -> dict:
    """96x96, 16 coils, 8192-sample spiral per coil (M=131072), 500 frames:
    relative image error of FP32 plans (FP64 PSF Gram, and an FP32 Gram over
    all rows), FP32 plans with R formed in FP64 and BF16-split plans against
    the plain FP64 GPU path (itself checked against the oracle's residual at
    this shape) for lambda in {1e-4, 1e-3, 1e-2} * mean diag and 0-2
    refinement steps, with kappa(G_l) from power iteration on the FP64 Gram."""
    import torch
    from paper_2410_06129_amd import pinv as P
    from paper_2410_06129_amd import synth

    w = synth.spiral_96x96_c16(F=args.frames_study)
    enc = w.enc
    N, M, F = enc.N, enc.M, w.images.shape[0]
    dev = torch.device("cuda:0")
    ctx = P.pinv_context_create(0)
    out = {"workload": w.name, "N": N, "M": M, "F": F, "by_lambda": {}}
    d64 = d32 = None
    for rel in (1e-4, 1e-3, 1e-2):
        p64 = P.pinv_build(ctx, enc, rel, P.LAMBDA_REL_MEAN_DIAG, P.FP64, P.FLAG_UNCACHED)
        P.pinv_plan_wait(p64)
        if d64 is None:
            d64 = torch.empty((F, M), dtype=torch.complex128, device=dev)
            P.pinv_forward(ctx, p64, torch.from_numpy(w.images).to(dev), d64)
            noise = torch.from_numpy(w.noise).to(dev)
            d64 += torch.sqrt(torch.mean(torch.abs(d64) ** 2)) * 10 ** (-w.snr_db / 20) * noise
            del noise
            d32 = d64.to(torch.complex64)
        info = P.pinv_plan_info_get(p64)
        G = torch.empty((N, N), dtype=torch.complex128, device=dev)
        P.pinv_plan_copy_buffer(p64, P.BUF_GRAM, G)
        v = torch.randn((N, 1), dtype=torch.complex128, device=dev)
        for _ in range(30):
            v = G @ v
            v = v / torch.linalg.vector_norm(v)
        smax = float(torch.real(torch.vdot(v[:, 0], (G @ v)[:, 0])))
        del G
        kappa = (smax + info["lambda_abs"]) / info["lambda_abs"]
        x64 = torch.empty((F, N), dtype=torch.complex128, device=dev)
        P.pinv_apply(ctx, p64, d64, x64)
        torch.cuda.synchronize()
        entry = {"kappa": kappa, "fp64_build_ms": sum(info["stage_ms"])}
        for name, prec, kw in (("fp32", P.FP32, {}),
                               ("fp32_gram_fp32", P.FP32, {"gram": P.GRAM_FULL}),
                               ("fp32_r_fp64", P.FP32, {"flags": P.FLAG_R_FP64}),
                               ("bf16x3", P.BF16X3, {})):
            flags = kw.pop("flags", 0)
            p = P.pinv_build(ctx, enc, rel, P.LAMBDA_REL_MEAN_DIAG, prec, flags | P.FLAG_UNCACHED, **kw)
            P.pinv_plan_wait(p)
            entry[name + "_build_ms"] = sum(P.pinv_plan_info_get(p)["stage_ms"])
            x = torch.empty((F, N), dtype=torch.complex64, device=dev)
            errs = {}
            for r in range(3):
                P.pinv_apply(ctx, p, d32, x, refine_steps=r)
                torch.cuda.synchronize()
                errs[str(r)] = dict(zip(("max", "median"), rel_err(x, x64)))
            entry[name] = errs
            P.pinv_plan_release(p)
            log(f"lambda {rel:g} {name}: {errs}")
        P.pinv_plan_release(p64)
        out["by_lambda"][f"{rel:g}"] = entry
    P.pinv_context_destroy(ctx)
    return out


def build_only(args) -> dict:
    import torch  # noqa: F401
    from paper_2410_06129_amd import pinv as P
    from paper_2410_06129_amd import synth
    import dataclasses
    side, coils = args.build_only
    enc = synth.serving_encoding(side, coils, 0)
    K = args.samples_per_coil or enc.K
    if args.samples_per_coil:
        enc = dataclasses.replace(enc, k=synth.vd_spiral(side, K))
    if args.mask == "disc":   # unknowns: the voxels inside the inscribed circle
        enc = dataclasses.replace(enc, voxels=synth.circular_mask(side, side).astype(np.int32))
    N, M = enc.N, enc.M
    ctx = P.pinv_context_create(0)
    route = "right pseudoinverse" if M < N else "left pseudoinverse"
    out = {"metric": "R-build executed TFLOP/s", "unit": "TFLOP/s",
           "config": {"workload": f"{side}x{side} image, {coils} coils, spiral {K} per coil"
                                  + (", disc mask" if args.mask == "disc" else "") + f", {route}",
                      "N": N, "M": M}, "builds": {}}
    for name in args.precisions.split(","):
        prec, flags, kw = {"fp32": (P.FP32, 0, {}), "fp64": (P.FP64, 0, {}),
                           "fp64_3m": (P.FP64, 0, {"cprod": P.CPROD_3M}),
                           "fp32_r_fp64": (P.FP32, P.FLAG_R_FP64, {}),
                           "bf16x3": (P.BF16X3, 0, {}),
                           "fp32_shared_gram": (P.FP32, 0, {"gram": P.GRAM_SHARED})}[name]
        form = "shared" if kw.get("gram") == P.GRAM_SHARED else "psf"
        ex = build_flops_executed(enc, form)
        times = []
        for rep in range(max(1, args.steps)):
            log(f"build {name} rep {rep} N={N} M={M}")
            p, st = build_timed(P, ctx, enc, 1e-3, prec, flags, **kw)
            times.append(st)
            P.pinv_plan_release(p)
            P.pinv_context_trim(ctx)
        st = np.median(np.array(times), axis=0)
        total = float(st.sum())
        exec_total = sum(ex.values())
        peak = PEAK_FP64_MFMA
        # a BF16X3 build's products run on the BF16 pipe (see bf16_mfma), an FP32 build's on
        # the F16 pipe: their counted rate has no single peak
        b3 = prec == P.BF16X3
        mixed = not (prec == P.FP64 or flags)
        out["builds"][name] = {
            "stage_ms": stage_dict(st), "build_ms": total,
            "tflops_executed": exec_total / (total * 1e-3) / 1e12,
            "frac_of_peak_executed": None if mixed else exec_total / (total * 1e-3) / 1e12 / peak,
            "peak": None if mixed else peak,
            "bf16_mfma": bf16x3_mfma(ex, stage_dict(st)) if b3 else None,
            "tflops_standard_count_effective": build_flops_standard(enc) / (total * 1e-3) / 1e12,
            "stage_tflops_executed": {k: ex[k] / (st[i] * 1e-3) / 1e12 if st[i] > 0 else None
                                      for i, k in enumerate(("gram", "chol_inv", "trmm_w", "trmm_r"))}}
        if M < N:
            # the right route runs both products (and R = Z^H) inside the last
            # stage interval: one rate for the two
            sx = out["builds"][name]["stage_tflops_executed"]
            del sx["trmm_w"], sx["trmm_r"]
            sx["products"] = (ex["trmm_w"] + ex["trmm_r"]) / ((st[2] + st[3]) * 1e-3) / 1e12
        log(json.dumps(out["builds"][name]))
    out["value"] = out["builds"][next(iter(out["builds"]))]["tflops_executed"]
    P.pinv_context_destroy(ctx)
    return out


def pmc_run(args) -> None:
    """A short run for counter collection: a plain 2 GiB device copy (the
    counters' scale), then at the default workload one FP32 build and one
    apply of `frames` frames with one refinement step, one BF16-split build
    and apply, and one build and apply of an FP32 plan with R formed in FP64
    (random data: the counters do not depend on values)."""
    import torch
    from paper_2410_06129_amd import pinv as P
    from paper_2410_06129_amd import synth
    dev = torch.device("cuda:0")
    src = torch.ones((1 << 29,), dtype=torch.float32, device=dev)     # 2 GiB
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    del src, dst
    w = synth.spiral_128x128_c8(F=1)
    enc = w.enc
    ctx = P.pinv_context_create(0)
    g = torch.Generator(device=dev).manual_seed(5)
    d = torch.randn((args.frames, enc.M), dtype=torch.complex64, device=dev, generator=g)
    x = torch.empty((args.frames, enc.N), dtype=torch.complex64, device=dev)
    few = {"fp32": (1, 16, 32), "bf16x3": (16,), "fp32_r_fp64": ()}
    for name, prec, flags, refine in (("fp32", P.FP32, 0, 1), ("bf16x3", P.BF16X3, 0, 0),
                                      ("fp32_r_fp64", P.FP32, P.FLAG_R_FP64, 0)):
        # (4M: the applies of an FP64-formed R on FP32 instructions, not on the pieces'
        # kernels that the FP32 plan's apply counts)
        p = P.pinv_build(ctx, enc, w.rel_lambda, P.LAMBDA_REL_MEAN_DIAG, prec, flags | P.FLAG_UNCACHED,
                         cprod=P.CPROD_4M if flags else P.CPROD_AUTO)
        P.pinv_apply(ctx, p, d, x, refine_steps=refine)
        for f in few[name]:   # one pass over R each
            P.pinv_apply(ctx, p, d[:f].contiguous(), x[:f])
        torch.cuda.synchronize()
        P.pinv_plan_wait(p)
        log(f"pmc run {name}: stage ms {P.pinv_plan_info_get(p)['stage_ms']}")
        P.pinv_plan_release(p)
        P.pinv_context_trim(ctx)
    # the Gram on MFMA: the 5-species, B0 workload (32x32, 8 coils, M = 49152),
    # whose default Gram is the shared-trajectory product (FP64 3M), and the
    # all-rows FP32 Gram
    ws = synth.species5_32x32_c8(F=1)
    for gram in (P.GRAM_AUTO, P.GRAM_FULL):
        p = P.pinv_build(ctx, ws.enc, ws.rel_lambda, P.LAMBDA_REL_MEAN_DIAG, P.FP32,
                         P.FLAG_UNCACHED | P.FLAG_NO_R, gram=gram)
        P.pinv_plan_wait(p)
        log(f"pmc run gram {gram}: stage ms {P.pinv_plan_info_get(p)['stage_ms']}")
        P.pinv_plan_release(p)
    P.pinv_context_destroy(ctx)
    print(json.dumps({"pmc_run": "done"}), flush=True)


# ----------------------------------------------------------------------------
# default: the headline workload
# ----------------------------------------------------------------------------

def headline(args) -> dict:
    import torch
    from paper_2410_06129_amd import pinv as P
    from paper_2410_06129_amd import synth

    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    w = synth.spiral_128x128_c8(F=args.frames)
    enc = w.enc
    N, M, F = enc.N, enc.M, args.frames
    log(f"workload {w.name}: N={N} M={M} F={F}")
    ctx = P.pinv_context_create(0)
    d64, d32, x_ref = make_inputs(P, ctx, w, F, dev)
    log("inputs ready")
    P.pinv_context_trim(ctx)
    x32 = torch.empty((F, N), dtype=torch.complex64, device=dev)

    # --- refinement steps: the fewest that meet the tolerance ---
    p32, st32 = build_timed(P, ctx, enc, w.rel_lambda, P.FP32)
    err_table = {}
    refine = None
    for r in range(3):
        P.pinv_apply(ctx, p32, d32, x32, refine_steps=r)
        torch.cuda.synchronize()
        err_table[str(r)] = rel_err(x32, x_ref)[0]
        log(f"refine {r}: max rel err {err_table[str(r)]:.3e}")
        if refine is None and err_table[str(r)] <= args.tol:
            refine = r
    refine = 2 if refine is None else refine
    a0 = apply_ms(P, ctx, p32, d32, x32, stream)
    ar = apply_ms(P, ctx, p32, d32, x32, stream, refine=refine)
    def few_frames(plan):
        """Applies of 1-32 frames: one pass over R (8NM bytes, complex64 or
        split-packed), timed as fractions of the HBM peak."""
        out = {}
        for Fs in (1, 2, 3, 4, 8, 9, 16, 24, 32):
            ds = d32[:Fs].contiguous()
            xs = torch.empty((Fs, N), dtype=torch.complex64, device=dev)
            ms = apply_ms(P, ctx, plan, ds, xs, stream, reps=5)
            nbytes = 8.0 * (N * M + Fs * M + Fs * N)
            out[str(Fs)] = {"ms": ms, "GB/s": nbytes / (ms * 1e-3) / 1e9,
                            "hbm_frac": nbytes / (ms * 1e-3) / PEAK_HBM,
                            "path": "rows" if Fs <= ROW_APPLY_MAX_F else
                            "stream" if Fs <= STREAM_MAX_F else "tiles"}
        return out

    small_f = few_frames(p32)
    log(f"small-F applies: {small_f}")
    P.pinv_plan_release(p32)
    P.pinv_context_trim(ctx)

    # --- timed steps ---
    def step():
        p = P.pinv_build(ctx, enc, w.rel_lambda, P.LAMBDA_REL_MEAN_DIAG, P.FP32, P.FLAG_UNCACHED)
        P.pinv_apply(ctx, p, d32, x32, refine_steps=refine)
        return p

    def run_steps(n, stages=None):
        # A plan lives until the next step is enqueued: the host waits for its
        # build (the next step already queued behind it), reads its stage
        # times and releases it, stream-ordered after its apply.
        prev = None
        for i in range(n):
            p = step()
            log(f"step {i} enqueued")
            if prev is not None:
                P.pinv_plan_wait(prev)
                if stages is not None:
                    stages.append(P.pinv_plan_info_get(prev)["stage_ms"])
                P.pinv_plan_release(prev)
            prev = p
        return prev

    last = run_steps(args.warmup)
    torch.cuda.synchronize()
    if last is not None:
        P.pinv_plan_release(last)
    stages = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    last = run_steps(args.steps, stages)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    P.pinv_plan_wait(last)
    stages.append(P.pinv_plan_info_get(last)["stage_ms"])
    P.pinv_plan_release(last)
    stages = np.array(stages)
    st_mean = stages.mean(axis=0)
    err_final = rel_err(x32, x_ref)
    ms_step = 1e3 * dt / args.steps
    for i, st in enumerate(stages):
        log(f"step {i} stage ms (gram, chol+inv, W, R): {np.round(st, 2)}")
    P.pinv_context_trim(ctx)

    ex = build_flops_executed(enc, "psf")
    build_exec = sum(ex.values())
    step_exec = build_exec + 8.0 * N * M * F + refine_flops(enc, F, refine)
    step_std = build_flops_standard(enc) + 8.0 * N * M * F
    build_ms = float(st_mean.sum())
    value = step_exec / (ms_step * 1e-3) / 1e12

    # --- FP32 plan with R formed in FP64: no refinement needed ---
    q, stq = build_timed(P, ctx, enc, w.rel_lambda, P.FP32, P.FLAG_R_FP64)
    P.pinv_apply(ctx, q, d32, x32)
    torch.cuda.synchronize()
    rf_err = rel_err(x32, x_ref)
    rf_apply = apply_ms(P, ctx, q, d32, x32, stream)
    P.pinv_plan_release(q)
    P.pinv_context_trim(ctx)
    rf_build = float(sum(stq))
    gap = (ar - rf_apply) / F          # ms per frame the FP64-formed R saves
    r_fp64 = {"build_ms": rf_build, "stage_ms": stage_dict(stq),
              "apply_frames_per_s": F / (rf_apply * 1e-3),
              "rel_err_unrefined": {"max": rf_err[0], "median": rf_err[1]},
              "breakeven_frames_vs_fp32_refined": (rf_build - build_ms) / gap if gap > 0 else None}
    log(f"R formed in FP64: {r_fp64}")

    # --- BF16-split plan ---
    b3, stb = build_timed(P, ctx, enc, w.rel_lambda, P.BF16X3)
    b3_err = {}
    for r in range(3):
        P.pinv_apply(ctx, b3, d32, x32, refine_steps=r)
        torch.cuda.synchronize()
        b3_err[str(r)] = rel_err(x32, x_ref)[0]
    b3_apply = apply_ms(P, ctx, b3, d32, x32, stream)
    b3_refined = apply_ms(P, ctx, b3, d32, x32, stream, refine=1)
    b3_small = few_frames(b3)
    P.pinv_plan_release(b3)
    P.pinv_context_trim(ctx)
    exb = build_flops_executed(enc)
    bf16x3 = {"build_ms": float(sum(stb)), "stage_ms": stage_dict(stb),
              "apply_frames_per_s": F / (b3_apply * 1e-3),
              "apply_refined_1_frames_per_s": F / (b3_refined * 1e-3),
              "apply_small_frames": b3_small,
              "rel_err_by_refine_steps": b3_err,
              "bf16_mfma": bf16x3_mfma(exb, stage_dict(stb), b3_apply, F, enc),
              "speedup_vs_fp32": {"build": build_ms / float(sum(stb)),
                                  "trmm_w": st32[2] / stb[2], "trmm_r": st32[3] / stb[3],
                                  "apply": a0 / b3_apply},
              "step_ms_refined_1": float(sum(stb)) + b3_refined}
    log(f"bf16x3: {bf16x3}")

    # --- factor-only plan (no W, no R) ---
    fo, stf = build_timed(P, ctx, enc, w.rel_lambda, P.FP32, P.FLAG_NO_R)
    fo_apply = apply_ms(P, ctx, fo, d32, x32, stream, refine=refine)
    fo_err = rel_err(x32, x_ref)
    P.pinv_plan_release(fo)
    fo_build = float(sum(stf))
    per_frame_gap = (fo_apply - ar) / F
    factor_only = {"build_ms": fo_build, "apply_refined_frames_per_s": F / (fo_apply * 1e-3),
                   "rel_err": {"max": fo_err[0], "median": fo_err[1]},
                   "breakeven_frames": (build_ms - fo_build) / per_frame_gap if per_frame_gap > 0 else None}
    log(f"factor-only: {factor_only}")
    P.pinv_context_trim(ctx)

    # --- plain FP64 GPU comparator (R 69 GB, W 69 GB) ---
    f64, st64 = build_timed(P, ctx, enc, w.rel_lambda, P.FP64)
    x64 = torch.empty((F, N), dtype=torch.complex128, device=dev)
    f64_apply = apply_ms(P, ctx, f64, d64, x64, stream, reps=2)
    f64_err = rel_err(x64, x_ref)
    P.pinv_plan_release(f64)
    P.pinv_context_trim(ctx)
    f64_build = float(sum(st64))
    fp64_gpu = {"build_ms": f64_build, "stage_ms": stage_dict(st64),
                "build_tflops_executed": build_exec / (f64_build * 1e-3) / 1e12,
                "apply_frames_per_s": F / (f64_apply * 1e-3),
                "rel_err": {"max": f64_err[0], "median": f64_err[1]}}
    log(f"fp64: {fp64_gpu}")
    del d64, d32, x64, x32, x_ref
    P.pinv_context_destroy(ctx)
    torch.cuda.empty_cache()

    # --- roofline of the dominant kernel of the step (HIP-event stage times on
    # the build stream; W with the packing of its operands) ---
    # (rates in executed f16 flops of the pieces' products)
    kern = {"trmm_w": (float(st_mean[2]), F16_TRMM * ex["trmm_w"], PEAK_F16_MFMA),
            "trmm_r": (float(st_mean[3]), F16_TRMM * ex["trmm_r"], PEAK_F16_MFMA),
            "apply": (a0, F16_APPLY * 8.0 * N * M * F, PEAK_F16_MFMA)}
    name = max(kern, key=lambda k: kern[k][0])
    kms, kfl, kpeak = kern[name]
    achieved = kfl / (kms * 1e-3) / 1e12
    tr = measured_traffic(name, w.name)
    roof = {"kernel": name, "bound": "mfma", "achieved": achieved, "peak": kpeak, "unit": "TFLOP/s",
            "frac": achieved / kpeak, "traffic": tr["bytes_per_launch"] if tr else None,
            "traffic_detail": tr,
            "mfma_pipe_frac": achieved / kpeak, "pipe": "f16, products of two and three pieces",
            "per_kernel": {k: {"ms": v[0], "tflops": v[1] / (v[0] * 1e-3) / 1e12, "peak": v[2],
                               "frac": v[1] / (v[0] * 1e-3) / 1e12 / v[2]} for k, v in kern.items()}}

    out = {
        "metric": METRIC, "value": value, "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": w.name, "N": N, "M": M, "F": F, "coils": enc.C,
                   "precision": "fp32 products on f16 pieces, fp64 gram and factorisation",
                   "refine_steps": refine, "lambda_rel": w.rel_lambda},
        "value_basis": "executed complex-equivalent flops per step / step time",
        "step_tflops_standard_count_effective": step_std / (ms_step * 1e-3) / 1e12,
        "build": {"ms": build_ms, "stage_ms": stage_dict(st_mean),
                  "tflops_executed": build_exec / (build_ms * 1e-3) / 1e12,
                  # (the products' executed f16 flops against the F16 pipe, over the whole build)
                  "frac_f16_peak_executed": F16_TRMM * (ex["trmm_w"] + ex["trmm_r"]) / (build_ms * 1e-3)
                                            / 1e12 / PEAK_F16_MFMA,
                  "tflops_standard_count_effective":
                      build_flops_standard(enc) / (build_ms * 1e-3) / 1e12,
                  "executed_flops": ex},
        "apply_frames_per_s": F / (a0 * 1e-3),
        "apply_refined_frames_per_s": F / (ar * 1e-3),
        "apply_small_frames": small_f,
        "rel_err_vs_fp64": {"max": err_final[0], "median": err_final[1],
                            "by_refine_steps": err_table,
                            "reference": "factor-only FP64 GPU solve with one FP64 refinement step"},
        "fp32_r_fp64": r_fp64,
        "bf16x3": bf16x3,
        "factor_only_fp32": factor_only,
        "fp64_gpu": fp64_gpu,
        "speedup_vs_fp64_gpu": {"build": f64_build / build_ms, "apply": f64_apply / a0,
                                # the fastest FP32-class apply that meets the tolerance
                                "apply_at_tol": f64_apply / min(
                                    [ar] + ([rf_apply] if rf_err[0] <= args.tol else []))},
        "roofline": roof,
    }
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--frames", type=int, default=1000)
    ap.add_argument("--tol", type=float, default=1e-5)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-config2", action="store_true")
    ap.add_argument("--serving", action="store_true", help="run the serving-mix trace instead")
    ap.add_argument("--rate", type=float, default=4.0)
    ap.add_argument("--duration", type=float, default=120.0)
    ap.add_argument("--serve-refine", type=int, default=1)
    ap.add_argument("--plan-frac", type=float, default=0.6)
    ap.add_argument("--serve-variants", default="fp32_refined,fp32_r_fp64,fp64")
    ap.add_argument("--pmc-run", action="store_true",
                    help="a 2 GiB copy, one FP32 build and one refined apply (counter runs)")
    ap.add_argument("--pmc-summary", nargs=2, metavar=("FETCH_DIR", "WRITE_DIR"),
                    help="write profiles/pmc_traffic.json from two rocprofv3 --pmc output folders")
    ap.add_argument("--pmc-mfma-summary", metavar="DIR",
                    help="write profiles/pmc_mfma.json from a rocprofv3 --pmc run of the MFMA counters")
    ap.add_argument("--build-only", type=int, nargs=2, metavar=("SIDE", "COILS"),
                    help="build plans for a SIDE^2 image with COILS coils (spiral 2N per coil)")
    ap.add_argument("--precisions", default="fp32,fp64")
    ap.add_argument("--samples-per-coil", type=int, default=0,
                    help="--build-only: spiral samples per coil (default 2N; fewer than N/C "
                         "gives the right pseudoinverse)")
    ap.add_argument("--mask", choices=("none", "disc"), default="none",
                    help="--build-only: restrict the unknowns to the inscribed disc")
    ap.add_argument("--precision-study", action="store_true")
    ap.add_argument("--eigen-study", action="store_true",
                    help="time the eigenvalue route (Jacobi) at moderate N beside the Cholesky route")
    ap.add_argument("--eigen-sides", default="32,48,64")
    ap.add_argument("--frames-study", type=int, default=500)
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (--gpus {args.gpus} requested); the multi-GPU "
              "sharding of this path is a design note, not a measured configuration.",
              file=sys.stderr)
        sys.exit(2)
    if args.pmc_mfma_summary:
        rec = pmc_mfma_summary(args.pmc_mfma_summary)
        with open(os.path.join(ROOT, "profiles", "pmc_mfma.json"), "w") as fh:
            json.dump(rec, fh, indent=1)
        print(json.dumps(rec), flush=True)
        return
    if args.pmc_summary:
        rec = pmc_summary(args.pmc_summary, args.frames)
        with open(os.path.join(ROOT, "profiles", "pmc_traffic.json"), "w") as fh:
            json.dump(rec, fh, indent=1)
        print(json.dumps(rec), flush=True)
        return

    import torch
    torch.cuda.init()
    # a dedicated (default-priority) stream: the library and torch's own work are
    # issued on it, and HIP events time it
    torch.cuda.set_stream(torch.cuda.Stream(device=torch.device("cuda:0")))
    if args.pmc_run:
        pmc_run(args)
        return
    if args.precision_study:
        res = precision_study(args)
        print(json.dumps({"metric": "relative image error vs plain FP64 GPU path", "unit": "rel",
                          "higher_is_better": False, "data": "synthetic",
                          "config": {"workload": res["workload"]}, "study": res}), flush=True)
        return
    if args.build_only:
        print(json.dumps(build_only(args)), flush=True)
        return
    if args.eigen_study:
        res = eigen_study(args)
        print(json.dumps({"metric": "eigenvalue-route build stages (ms) and Jacobi HBM rate",
                          "unit": "ms", "higher_is_better": False, "data": "synthetic",
                          "config": {"workload": "spiral 2N per coil, 8 coils, sides "
                                                 + args.eigen_sides}, "study": res}), flush=True)
        return
    if args.serving:
        res = serving(args)
        first = args.serve_variants.split(",")[0]
        p99 = res[first]["p99_s"]
        out = {"metric": "serving p50/p99 latency (s) and throughput",
               "value": p99 if isinstance(p99, float) else res[first]["p99_served_s"],
               "unit": "s", "n_gpus": 1, "higher_is_better": False, "data": "synthetic",
               "dtype": "f32", "config": {"workload": f"serving mix, Poisson {args.rate}/s over "
                                                      f"{args.duration} s"}, "serving": res}
        print(json.dumps(out), flush=True)
        return
    from paper_2410_06129_amd import pinv as P
    out = headline(args)
    if not args.no_config2:
        ctx = P.pinv_context_create(0)
        out["workload_64x64_c8"] = config2_figures(P, ctx, torch.cuda.current_stream(),
                                                   torch.device("cuda:0"), args.tol)
        P.pinv_context_destroy(ctx)
    if not args.no_cpu_baseline:
        from paper_2410_06129_amd import synth
        log("cpu baseline (oracle) ...")
        out["cpu_baseline"] = cpu_baseline(synth.spiral_128x128_c8(F=1).enc)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
