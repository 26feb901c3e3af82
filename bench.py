"""Benchmark of the differentiable Poisson solver on one MI355X.

A step is one forward + backward solve (every stage of the hot path: binning,
splat + r2c, the axis FFT passes, the fused spectral operator, c2r + gather,
the FP64 reductions, normalisation, and the whole adjoint) over one resident
synthetic oriented point cloud. Inputs, the loss gradient and all buffers are
in HBM before the timed region starts.

Default workload: 256^3 grid, 100,000 points on a random superellipsoid
(seed 2), normals perturbed by N(0, 0.05^2) and renormalised, sigma = 2 cells;
the loss is mean((chi - chi_t)^2) with chi_t from the clean normals.

Printed: ONE JSON line with solves/s, the dominant kernel's roofline
(algorithmic bytes / HIP-event duration, against 8 TB/s), two whole-step
rates (dense-equivalent: B_stage = 128 r^3 + 72 P over the step time, which
counts planes and row tiles the kernels skip; skip-aware: the bytes of the
stages actually run), secondary lines (128^3 fwd+bwd and forward only, 256^3
forward only, 256^3 with half the points uniform outliers so that nothing can
be skipped, 32^3 forward only, the 64-shape batch, a compact serving run with
p50/p99 latency), and the FP64 oracle timed on one host core on the headline
workload together with the GPU's error against that oracle run.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import re
import subprocess
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "PSR fwd+bwd solves/sec at 128^3/256^3 + %HBM roofline; p50/p99 latency in serving"
HBM_PEAK_GBS = 8000.0


# --------------------------------------------------------------------------- byte model
def half_spec_bytes(r: int) -> int:
    """One complex64 half-spectrum channel: r * r * (r/2 + 1) * 8 bytes."""
    return r * r * (r // 2 + 1) * 8


def tile_rows(r: int) -> int:
    """Rows of a binning tile (the library's row-pass geometry: 512-thread row
    workgroups, 256 at 256^3; 16 elements per thread of a half-length row)."""
    return min(r, (256 if r == 256 else 512) // max(1, (r // 2) // 16))


def live_fractions(points, r: int):
    """Fractions of the j0 planes and of the (j0, row-tile) tiles that some
    point's trilinear corners reach. The passes skip the rest (their splat is
    zero and nothing is gathered from them), so they set the bytes those
    passes must move."""
    import numpy as np
    t = np.asarray(points, dtype=np.float32).astype(np.float64)
    u = t - np.floor(t)
    u[u >= 1.0] = 0.0
    b = np.clip(np.floor(u * r).astype(np.int64), 0, r - 1)
    planes = np.zeros(r, dtype=bool)
    planes[b[:, 0]] = True
    planes[(b[:, 0] + 1) % r] = True
    tr = tile_rows(r)
    tiles = np.zeros((r, r // tr), dtype=bool)
    for o0 in (0, 1):
        for o1 in (0, 1):
            tiles[(b[:, 0] + o0) % r, ((b[:, 1] + o1) % r) // tr] = True
    return float(planes.mean()), float(tiles.mean())


def stage_bytes(r: int, P: int, fp: float = 1.0, ft: float = 1.0) -> dict:
    """Algorithmic bytes per launch of each stage: every array the stage must
    read once and write once (points, spectra, grids), nothing counted twice.
    fp / ft: fractions of planes / row tiles that points reach; spectra lines
    of the other planes and tiles are neither written nor read where the
    method leaves them zero or unused."""
    S = half_spec_bytes(r)
    N4 = 4 * r ** 3
    slots = 2 if r <= 128 else 4  # gather partials per point and channel (16 bytes each)
    return {
        "bin": 24 * P + 32 * P * 2 + 8 * P,
        "P1_splat_r2c": 32 * P + 3 * S * ft,           # sorted points in, 3 half-spectra of touched row tiles out
        "P2_fft_j1": 3 * S * ft + 2 * S * fp,          # touched tile segments of 3 channels in, v~_0 and merged W of live planes out
        # live planes of the 2 in, chi~ (after the k0 inverse) out; at 32-128 the plane pass hands over 3 channels
        # (v~_0, kappa_1 v~_1, kappa_2 v~_2)
        "P3_fft_j0_spectral_ifft_j0": (3 if 32 <= r <= 128 else 2) * S * fp + S,
        "P4_ifft_j1": 2 * S,
        "P5_c2r_gather": S + N4 + 32 * P + 16 * slots * P,  # chi' written, gather partials
        "fwd_reduce": 64 * P + 16 * P,
        "normalize": 2 * N4 + (16 * slots * P + 16 * P if r <= 256 else 0),  # the points' gradients ride along up to 256
        "bwd_reduce": 2 * N4,
        "B1a_reduce_r2c": 2 * N4 + S * (1 - ft),      # G and chi in (FP64 partials), H = sG spectra of point-free tiles out
        "B1_cotangent_r2c": N4 * ft + 32 * P + S * ft, # the tiles with points: G in, splat of W, spectra out
        "B2_fft_j1": 2 * S,
        # 1 in (after a plane pass W^ of the live planes too); kappa_0 channel and U out on live planes
        "B3_fft_j0_conjop_ifft_j0": S + (S * fp if 32 <= r <= 128 else 0) + 2 * S * fp,
        "B4_ifft_j1": 2 * S * fp + 3 * S * ft,         # live planes in, touched tiles out
        "B5_c2r_gather": 3 * S * ft + 32 * P + 48 * slots * P,
        "bwd_finalize": 48 * slots * P + 16 * P + 32 * P + 24 * P,
        # plane passes (two axes per kernel; 32^3 to 256^3)
        "P12_splat_r2c_fft_j1": 32 * P + 3 * S * fp,   # sorted points in, v~_0, kappa_1 v~_1, kappa_2 v~_2 of live planes out
        "P45_ifft_j1_c2r_gather": S + N4 + 32 * P + 16 * slots * P,
        "B12_cotangent_r2c_fft_j1": 2 * N4 + 32 * P + S + S * fp,  # G and chi in (FP64 sums), (sG)^ and live W^ out
        "B45_ifft_j1_c2r_gather": 2 * S * fp + 32 * P + 48 * slots * P,  # upper bound: plane parts without points are skipped
    }


def path_stages(r: int, backward: bool = True) -> list:
    """The stages one solve runs at grid size r (plane passes at 32-128, the
    plane inverse pass also at 256, two-pass row/column kernels elsewhere)."""
    plane, p45 = 32 <= r <= 128, 32 <= r <= 256
    f = ["bin"] + (["P12_splat_r2c_fft_j1"] if plane else ["P1_splat_r2c", "P2_fft_j1"])
    f += ["P3_fft_j0_spectral_ifft_j0"] + (["P45_ifft_j1_c2r_gather"] if p45 else ["P4_ifft_j1", "P5_c2r_gather"])
    f += (["fwd_reduce"] if r >= 512 else []) + ["normalize"]
    b = ["B12_cotangent_r2c_fft_j1"] if plane else ["B1a_reduce_r2c", "B1_cotangent_r2c", "B2_fft_j1"]
    b += ["B3_fft_j0_conjop_ifft_j0"] + (["B45_ifft_j1_c2r_gather"] if plane else ["B4_ifft_j1", "B5_c2r_gather"])
    b += ["bwd_finalize"]
    return f + (b if backward else [])


def skip_aware_bytes(r: int, P: int, fp: float, ft: float, backward: bool = True) -> float:
    """Algorithmic bytes of the stages a solve actually runs, with the
    point-free planes and row tiles that the kernels skip left out."""
    sb = stage_bytes(r, P, fp, ft)
    return float(sum(sb[st] for st in path_stages(r, backward)))


def b_stage(r: int, P: int) -> int:
    """Whole-step algorithmic bytes of forward+backward: 128 r^3 + 72 P (every
    named array written once and read once in FP32; each 3D transform one
    read + one write)."""
    return 128 * r ** 3 + 72 * P


# Kernel of each single-kernel stage, as rocprofv3 names it (res substituted).
KERNEL_STAGES = [
    (r"k_splat_r2c<{r}, 0,", "P1_splat_r2c"),
    (r"k_axis1_fwd<{r}, true,", "P2_fft_j1"),
    (r"k_fwd_axis0<{r},", "P3_fft_j0_spectral_ifft_j0"),
    (r"k_axis1_inv<{r}, false,", "P4_ifft_j1"),
    (r"k_c2r_gather<{r}, 0,", "P5_c2r_gather"),
    (r"k_normalize<{r},", "normalize"),
    (r"k_splat_r2c<{r}, 1,", "B1_cotangent_r2c"),
    (r"k_splat_r2c<{r}, 4,", "B1a_reduce_r2c"),
    (r"k_axis1_fwd<{r}, false,", "B2_fft_j1"),
    (r"k_bwd_axis0<{r},", "B3_fft_j0_conjop_ifft_j0"),
    (r"k_axis1_inv<{r}, true,", "B4_ifft_j1"),
    (r"k_c2r_gather<{r}, 1,", "B5_c2r_gather"),
    (r"k_plane_fwd<{r}, 0,", "P12_splat_r2c_fft_j1"),
    (r"k_plane_inv<{r}, 0,", "P45_ifft_j1_c2r_gather"),
    (r"k_plane_fwd<{r}, 3,", "B12_cotangent_r2c_fft_j1"),
    (r"k_plane_inv<{r}, 1,", "B45_ifft_j1_c2r_gather"),
]


SOLVER_SOURCES = ["fft_device.h", "psr_geometry.h", "psr_internal.h", "psr_device.h", "psr_kernels.hip"]


def kernel_source_hash() -> str:
    """Hash of the sources the solver's kernels are built from (the counters
    of profiles/ stay valid while it is unchanged)."""
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2106_03452_amd", "csrc")
    for name in SOLVER_SOURCES:
        with open(os.path.join(csrc, name), "rb") as fh:
            h.update(name.encode() + fh.read())
    return h.hexdigest()[:16]


def traffic_from_profiles(kernel_stage: str, workload: str):
    """HBM bytes per launch of the dominant kernel from the committed rocprofv3
    counter summary, if it was taken on the current kernel sources."""
    path = os.path.join(ROOT, "profiles", "hbm_traffic_" + workload + ".json")
    if not os.path.exists(path):
        return None
    try:
        d = json.load(open(path))
    except Exception:
        return None
    if d.get("kernel_source_hash") != kernel_source_hash():
        return None
    st = d.get("stages", {}).get(kernel_stage)
    if not st:
        return None
    return st.get("hbm_bytes_per_launch")


def _counter_means(path: str) -> dict:
    """Mean Counter_Value (KiB) per kernel name of a rocprofv3 --pmc CSV."""
    import csv
    acc = {}
    with open(path) as fh:
        for row in csv.DictReader(fh):
            a = acc.setdefault(row["Kernel_Name"], [0.0, 0])
            a[0] += float(row["Counter_Value"])
            a[1] += 1
    return {k: v[0] / v[1] for k, v in acc.items()}


def ingest_counters(fetch_csv, write_csv, copy_fetch_csv, copy_write_csv, workload="c3_256"):
    """HBM bytes per launch of each stage kernel from two rocprofv3 --pmc runs
    (FETCH_SIZE, WRITE_SIZE; KiB per dispatch), each scaled by what the same
    counter reads for a plain 1 GiB device copy (bench.py --calibrate-copy).
    Writes profiles/hbm_traffic_<workload>.json, tagged with the kernel source
    hash so that a later kernel change voids it."""
    gib = float(1 << 30)
    cf, cw = _counter_means(copy_fetch_csv), _counter_means(copy_write_csv)
    # the copy kernel is the one launch whose counters are ~1 GiB-sized
    copy_f = max(cf.values()) * 1024.0
    copy_w = max(cw.values()) * 1024.0
    kf, kw = gib / copy_f, gib / copy_w
    fe, wr = _counter_means(fetch_csv), _counter_means(write_csv)
    import psr_synth as S
    shape = S.config_c3()
    r, P = shape.res, shape.P
    sb = stage_bytes(r, P, *live_fractions(shape.points, r))
    stages = {}
    for pat, stage in KERNEL_STAGES:
        rx = re.compile(re.escape(pat.format(r=r)).replace(r"\ ", r"\s*"))
        names = [k for k in fe if rx.search(k)]
        if len(names) != 1:
            continue
        f = fe[names[0]] * 1024.0 * kf
        w = wr.get(names[0], 0.0) * 1024.0 * kw
        stages[stage] = {"kernel": names[0], "fetch_bytes": round(f), "write_bytes": round(w),
                         "hbm_bytes_per_launch": round(f + w), "algorithmic_bytes": round(sb[stage]),
                         "ratio_to_algorithmic": round((f + w) / sb[stage], 3)}
    out = {"workload": workload, "kernel_source_hash": kernel_source_hash(),
           "copy_calibration": {"fetch_counter_bytes_per_GiB_copy": round(copy_f),
                                "write_counter_bytes_per_GiB_copy": round(copy_w),
                                "fetch_scale": round(kf, 4), "write_scale": round(kw, 4)},
           "stages": stages}
    path = os.path.join(ROOT, "profiles", "hbm_traffic_" + workload + ".json")
    with open(path, "w") as fh:
        json.dump(out, fh, indent=1)
        fh.write("\n")
    return out


# --------------------------------------------------------------------------- CPU baseline
CPU_SNIPPET = r"""
import json, os, sys, time
sys.path.insert(0, {root!r})
import numpy as np
import oracle, psr_synth as S
sh = S.config_c3()
chi_t, _ = oracle.forward(sh.points_clean, sh.normals_clean, sh.res, sh.sigma)
secs = []
for _ in range(3):
    t0 = time.perf_counter()
    chi, aux = oracle.forward(sh.points, sh.normals, sh.res, sh.sigma)
    G = 2.0 * (chi - chi_t) / chi.size
    dc, dn = oracle.backward(aux, G)
    secs.append(time.perf_counter() - t0)
np.savez({out!r}, chi=chi, dc=dc, dn=dn)
print(json.dumps(dict(seconds=sorted(secs)[1])))
"""


def cpu_baseline(gpu_result=None):
    """The FP64 oracle timed on one host core over three full solves of the
    headline workload; with ``gpu_result`` = (chi, dpoints, dnormals) of the
    GPU on the same workload, also the GPU's error against this oracle run
    (e_chi = max|dchi| / max|chi|, e_g = relative L2 per gradient)."""
    import tempfile
    import numpy as np
    env = dict(os.environ, OMP_NUM_THREADS="1", OPENBLAS_NUM_THREADS="1", MKL_NUM_THREADS="1",
               NUMEXPR_NUM_THREADS="1")
    with tempfile.TemporaryDirectory() as td:
        npz = os.path.join(td, "oracle_c3.npz")
        out = subprocess.run([sys.executable, "-c", CPU_SNIPPET.format(root=ROOT, out=npz)], env=env,
                             capture_output=True, text=True, timeout=900)
        if out.returncode != 0:
            sys.stderr.write(out.stderr[-2000:])
            return None
        sec = json.loads(out.stdout.strip().splitlines()[-1])["seconds"]
        res = {"value": round(1.0 / sec, 5), "unit": "solves/s", "cores": 1, "kind": "oracle",
               "sample": f"three full forward+backward solves of the same 256^3 / 100k-point workload, median "
                         f"{sec:.1f} s (FP64 NumPy oracle, single thread; the loss target chi_t is computed "
                         f"outside the timed samples)"}
        if gpu_result is not None:
            ref = np.load(npz)
            chi, dp, dn = (np.asarray(a, dtype=np.float64) for a in gpu_result)
            rel2 = lambda a, b: float(np.linalg.norm(a - b) / np.linalg.norm(b))
            res["parity"] = {"e_chi": float(np.abs(chi - ref["chi"]).max() / np.abs(ref["chi"]).max()),
                             "e_dpoints": rel2(dp, ref["dc"]), "e_dnormals": rel2(dn, ref["dn"]),
                             "bars": {"e_chi": 1e-5, "e_dpoints": 1e-4, "e_dnormals": 1e-4},
                             "note": "GPU forward+backward of the timed workload (FP32 bulk, FP64 reductions; "
                                     "each side forms its own loss gradient) against this FP64 oracle run"}
    return res


def step_times(step, reps, torch, scrub=None):
    """Per-repetition durations (ms) of one step from HIP events on the current
    stream; with scrub, a 512 MiB device write runs before each repetition
    (outside the events) so the step starts with cold caches."""
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(reps)]
    for a, b in ev:
        if scrub is not None:
            scrub.fill_(1.0)
        a.record()
        step()
        b.record()
    torch.cuda.synchronize()
    t = sorted(a.elapsed_time(b) for a, b in ev)
    q = lambda f: round(t[min(len(t) - 1, int(f * len(t)))], 4)
    return {"median_ms": q(0.5), "p10_ms": q(0.1), "p90_ms": q(0.9), "reps": reps}


# --------------------------------------------------------------------------- GPU runs
def prepare(shape, dev, torch, F):
    pts = torch.from_numpy(shape.points).to(dev)
    nrm = torch.from_numpy(shape.normals).to(dev)
    r, P = shape.res, shape.P
    chi, saved = F.forward(pts, nrm, r, shape.sigma)
    if shape.points_clean is not None:
        chi_t, _ = F.forward(torch.from_numpy(shape.points_clean).to(dev),
                             torch.from_numpy(shape.normals_clean).to(dev), r, shape.sigma)
        G = (2.0 * (chi - chi_t) / chi.numel()).contiguous()
    else:  # forward-only workloads: the backward is never run
        G = torch.zeros_like(chi)
    from paper_2106_03452_amd import _lib
    ws = torch.empty(_lib.workspace_bytes(r, P), dtype=torch.uint8, device=dev)
    dp = torch.empty((P, 3), dtype=torch.float32, device=dev)
    dn = torch.empty((P, 3), dtype=torch.float32, device=dev)
    torch.cuda.synchronize()
    return dict(pts=pts, nrm=nrm, chi=chi, saved=saved, G=G, ws=ws, dp=dp, dn=dn, r=r, P=P, sigma=shape.sigma)


def make_step(b, ctx, backward: bool = True):
    import ctypes
    import torch
    from paper_2106_03452_amd import _lib
    L = _lib.lib()
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    wsb = ctypes.c_size_t(b["ws"].numel())
    args_f = (ctx.handle, p(b["pts"]), p(b["nrm"]), b["P"], b["r"], b["sigma"], p(b["chi"]), p(b["saved"]),
              p(b["ws"]), wsb, stream)
    args_b = (ctx.handle, b["P"], b["r"], b["sigma"], p(b["chi"]), p(b["saved"]), p(b["G"]), p(b["dp"]),
              p(b["dn"]), p(b["ws"]), wsb, stream)

    def step():
        rc = L.psr_forward(*args_f)
        if rc:
            raise RuntimeError(f"psr_forward failed: {rc}")
        if backward:
            rc = L.psr_backward(*args_b)
            if rc:
                raise RuntimeError(f"psr_backward failed: {rc}")
    return step


def batch_c4(dev, torch, steps=10, warmup=3):
    """64 shapes (res 64/128, P log-uniform 1e3..5e4, seed 3), fwd+bwd with
    G = 2 chi / N (loss mean chi^2): one psr_run_batched call vs the same
    solves as sequential psr_forward/psr_backward calls on one stream."""
    import psr_synth as S
    from paper_2106_03452_amd import _lib
    from paper_2106_03452_amd import function as F
    from paper_2106_03452_amd.batch import BatchPlan, Job
    shapes = S.config_c4()
    jobs = []
    for sh in shapes:
        p = torch.from_numpy(sh.points).to(dev)
        n = torch.from_numpy(sh.normals).to(dev)
        chi, _ = F.forward(p, n, sh.res, sh.sigma)
        jobs.append(Job(p, n, sh.res, sh.sigma, (2.0 * chi / chi.numel()).contiguous()))
    plan = BatchPlan(jobs)
    dt_b = timed(plan.run, steps, warmup, torch)
    ctx = _lib.context(0)
    steps_seq = []
    for i, j in enumerate(jobs):
        b = dict(pts=j.points, nrm=j.normals, chi=plan.chi[i], saved=plan.saved[i], G=j.dchi, ws=plan.ws[i],
                 dp=plan.dp[i], dn=plan.dn[i], r=j.res, P=int(j.points.shape[0]), sigma=j.sigma)
        steps_seq.append(make_step(b, ctx))

    def seq():
        for st in steps_seq:
            st()
    dt_s = timed(seq, steps, warmup, torch)
    total_bytes = sum(b_stage(j.res, int(j.points.shape[0])) for j in jobs)
    t_b = dt_b / steps
    return {"workload": "64 shapes, res 64/128, P log-uniform [1e3, 5e4] (seed 3), fwd+bwd",
            "shapes_per_s_batched": round(len(jobs) / t_b, 1),
            "shapes_per_s_sequential": round(len(jobs) / (dt_s / steps), 1),
            "ms_per_batch": round(t_b * 1e3, 4), "ms_sequential": round(dt_s / steps * 1e3, 4),
            "step_roofline_frac": round(total_bytes / t_b / 1e9 / HBM_PEAK_GBS, 4)}


def batch_c2(dev, torch, copies=24, steps=10, warmup=3):
    """The 128^3 workload (20k points, fwd+bwd) as one batch of `copies`
    solves (one launch per stage for all of them), against the same number
    of single solves one after the other: a single 128^3 solve leaves most of
    the 256 CUs idle between its dependent passes, a batch fills them."""
    import psr_synth as S
    from paper_2106_03452_amd import function as F
    from paper_2106_03452_amd.batch import BatchPlan, Job
    sh = S.config_c2()
    p = torch.from_numpy(sh.points).to(dev)
    n = torch.from_numpy(sh.normals).to(dev)
    chi_t, _ = F.forward(torch.from_numpy(sh.points_clean).to(dev), torch.from_numpy(sh.normals_clean).to(dev),
                         128, sh.sigma)
    chi, _ = F.forward(p, n, 128, sh.sigma)
    G = (2.0 * (chi - chi_t) / chi.numel()).contiguous()
    plan = BatchPlan([Job(p, n, 128, sh.sigma, G) for _ in range(copies)])
    dt = timed(plan.run, steps, warmup, torch)
    t = dt / steps
    return {"workload": f"{copies} copies of the 128^3 / 20k-point solve, fwd+bwd, one batched call",
            "solves_per_s": round(copies / t, 1), "ms_per_batch": round(t * 1e3, 4),
            "dense_equivalent_frac": round(copies * b_stage(128, int(p.shape[0])) / t / 1e9 / HBM_PEAK_GBS, 4)}


def slab_bytes(r, P):
    """Algorithmic bytes of each stage of the slab forward (grid traffic with
    every plane counted, plus the point records): sp = one channel of the
    half spectrum, r^2 (r/2 + 1) complex64."""
    sp = r * r * (r // 2 + 1) * 8
    return {"slab_bin": 112 * P, "S1_splat_r2c": 3 * sp + 192 * P, "S2_fft_j1_exchange": 5 * sp,
            "S3_pencil_fft_j0_spectral": 3 * sp, "S4_ifft_k1": 2 * sp, "S5_c2r_halo": sp + 4 * r ** 3,
            "slab_gather_mean": P * (32 + 32 + 8 + 8), "slab_normalize": 8 * r ** 3}


def slab_leg(dev, torch, steps=3, warmup=1, slabs=8):
    """The large-scene form: a 1M-point scene of 16 objects on a 1024^3 grid
    (sigma 2), forward only, solved in `slabs` slabs of 128 planes; stage
    times from HIP events on the solve stream. Also the C3 cloud at 256^3
    through the slab path, beside the single-grid forward of the same cloud."""
    import psr_synth as S
    from paper_2106_03452_amd import _lib
    from paper_2106_03452_amd import slab as SL
    ctx = _lib.context(0)
    sh = S.config_scene()
    r, P = sh.res, sh.P
    pts = torch.from_numpy(sh.points).to(dev)
    nrm = torch.from_numpy(sh.normals).to(dev)
    ws = torch.empty(SL.workspace_bytes(r, P, slabs), dtype=torch.uint8, device=dev)
    chi = torch.empty((r, r, r), dtype=torch.float32, device=dev)
    rb = torch.zeros(48, dtype=torch.uint8, device=dev)

    def step():
        SL.forward_raw(pts, nrm, r, sh.sigma, slabs, chi, rb, ws, ctx)
    dt = timed(step, steps, warmup, torch)
    ms = dt / steps * 1e3
    ctx.set("timers", 1)
    ctx.reset_timers()
    timed(step, steps, 0, torch)
    st = {k: v[0] / v[1] for k, v in ctx.stage_times().items() if v[1] > 0}
    ctx.set("timers", 0)
    sb = slab_bytes(r, P)
    total = sum(sb.values())
    stages = {k: {"ms": round(st[k], 4), "GBs": round(sb[k] / (st[k] * 1e-3) / 1e9, 1),
                  "frac": round(sb[k] / (st[k] * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)} for k in sb if k in st}
    status = SL.read_result(rb)["status"]
    del ws, chi
    # the same path on the 256^3 cloud, beside the single-grid forward
    from paper_2106_03452_amd import function as F
    c3 = S.config_c3()
    p3, n3 = torch.from_numpy(c3.points).to(dev), torch.from_numpy(c3.normals).to(dev)
    ws3 = torch.empty(SL.workspace_bytes(256, c3.P, slabs), dtype=torch.uint8, device=dev)
    chi3 = torch.empty((256, 256, 256), dtype=torch.float32, device=dev)
    d3 = timed(lambda: SL.forward_raw(p3, n3, 256, c3.sigma, slabs, chi3, rb, ws3, ctx), 20, 3, torch)
    wsf = torch.empty(_lib.workspace_bytes(256, c3.P), dtype=torch.uint8, device=dev)
    d4 = timed(lambda: F.forward(p3, n3, 256, c3.sigma, ctx, wsf), 20, 3, torch)
    return {"workload": f"1024^3, 1M points on 16 objects (seed 5), sigma 2, forward only, {slabs} slabs of "
                        f"{r // slabs} planes", "status": status,
            "ms_per_solve": round(ms, 3), "solves_per_s": round(1e3 / ms, 2),
            "dense_bytes": total, "dense_GBs": round(total / (ms * 1e-3) / 1e9, 1),
            "dense_frac": round(total / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4), "stages": stages,
            "c3_256_slab_ms": round(d3 / 20 * 1e3, 4), "c3_256_single_grid_fwd_ms": round(d4 / 20 * 1e3, 4)}


def sweep(dev, torch):
    """Sizes beyond the named workloads: the C3 superellipsoid (seed 2) with
    10^4, 10^5 and 10^6 points at 64^3 to 512^3 (forward + backward, the loss
    gradient a dense standard normal field, and forward alone), and the
    1M-point scene at 1024^3 through the slab forward with 2, 8 and 32 slabs."""
    import psr_synth as S
    from paper_2106_03452_amd import _lib
    from paper_2106_03452_amd import function as F
    from paper_2106_03452_amd import slab as SL
    ctx = _lib.context(0)
    rows = []
    for P in (10_000, 100_000, 1_000_000):
        base = S.config_c3(P=P)
        for r in (64, 128, 256, 512):
            sh = S.Shape(r, 2.0, base.points, base.normals, kind="superellipsoid")
            b = prepare(sh, dev, torch, F)
            b["G"] = torch.from_numpy(S.loss_gradient(r, 11)).to(dev)
            n = 20 if r <= 256 else 5
            t_fb = timed(make_step(b, ctx), n, 3, torch) / n
            t_f = timed(make_step(b, ctx, backward=False), n, 3, torch) / n
            rows.append({"res": r, "npoints": P, "fwd_bwd_ms": round(t_fb * 1e3, 4), "fwd_ms": round(t_f * 1e3, 4),
                         "fwd_bwd_solves_per_s": round(1.0 / t_fb, 1),
                         "dense_equivalent_frac": round(b_stage(r, P) / t_fb / 1e9 / HBM_PEAK_GBS, 4)})
            print(json.dumps(rows[-1]), flush=True)
            del b
    sc = S.config_scene()
    p, n = torch.from_numpy(sc.points).to(dev), torch.from_numpy(sc.normals).to(dev)
    chi = torch.empty((sc.res,) * 3, dtype=torch.float32, device=dev)
    rb = torch.zeros(48, dtype=torch.uint8, device=dev)
    slabs = []
    for g in (2, 8, 32):
        ws = torch.empty(SL.workspace_bytes(sc.res, sc.P, g), dtype=torch.uint8, device=dev)
        t = timed(lambda: SL.forward_raw(p, n, sc.res, sc.sigma, g, chi, rb, ws, ctx), 3, 1, torch) / 3
        slabs.append({"res": sc.res, "npoints": sc.P, "slabs": g, "fwd_ms": round(t * 1e3, 3)})
        print(json.dumps(slabs[-1]), flush=True)
        del ws
    return {"grid": rows, "slab_1024": slabs}


def serve_mode(dev, torch, n_requests, levels=(0.5, 0.8, 1.0, 1.5)):
    """Poisson request stream (seed 4): res in {64,128,256}, P log-uniform in
    [3e3, 2e5], 50/50 forward vs forward+backward. lambda_seq = throughput of
    sequential plain solves over the stream; then, at QPS = level x
    lambda_seq, the continuous-batching engine and the sequential baseline
    serve the same arrivals; p50/p99 latency skip the first 100 requests."""
    import numpy as np
    import psr_synth as S
    from paper_2106_03452_amd import _lib
    from paper_2106_03452_amd.serve import Engine, GpuBackend, Request, SequentialBaseline, drive, latency_stats
    print(f"serve: generating {n_requests} requests", file=sys.stderr, flush=True)
    reqs_spec, arrivals_unit = S.config_c5(n_requests=n_requests, workers=min(16, os.cpu_count() or 1))
    classes = {64: 200000, 128: 200000, 256: 200000}
    data = []
    rng = np.random.Generator(np.random.PCG64(44))
    G = {r: torch.from_numpy((rng.standard_normal((r, r, r)) * 1e-6).astype(np.float32)).to(dev) for r in classes}
    for sh, bwd in reqs_spec:
        data.append((sh.res, sh.P, bwd, torch.from_numpy(sh.points).to(dev), torch.from_numpy(sh.normals).to(dev)))
    torch.cuda.synchronize()

    def make(arr):
        return [Request(i, res, P, bwd, float(a), p, n, G[res] if bwd else None)
                for i, ((res, P, bwd, p, n), a) in enumerate(zip(data, arr))]

    seq = SequentialBaseline(0)
    # warm up and measure lambda_seq: everything available at t = 0, one solve at a time
    seq.run(make([0.0] * min(50, len(data))), classes)
    rs = make([0.0] * len(data))
    t0 = seq.run(rs, classes)
    lam = len(rs) / (max(r.done for r in rs) - t0)
    be = GpuBackend(0, num_streams=4)
    budget = 48 << 30
    warm = Engine(be, classes, budget)
    drive(warm, make([0.0] * min(100, len(data))))
    out = {"workload": f"{len(data)} requests, res 64/128/256, P log-uniform [3e3, 2e5], 50/50 fwd vs fwd+bwd, "
                       "Poisson arrivals (seed 4)",
           "lambda_seq_solves_per_s": round(lam, 1), "levels": []}
    print(f"serve: lambda_seq = {lam:.1f} solves/s", file=sys.stderr, flush=True)
    for f in levels:
        print(f"serve: level {f}", file=sys.stderr, flush=True)
        qps = f * lam
        arr = np.cumsum(arrivals_unit[:len(data)]) / qps
        eng = Engine(be, classes, budget)
        eng.classes = warm.classes  # resident slots carried over
        eng.used = warm.used
        r_e = make(arr)
        t0e = drive(eng, r_e)
        r_s = make(arr)
        t0s = seq.run(r_s, classes)
        thr = lambda rr, t0: len(rr) / (max(r.done for r in rr) - t0)
        out["levels"].append({"qps_factor": f, "qps": round(qps, 1),
                              "engine": {"solves_per_s": round(thr(r_e, t0e), 1), **latency_stats(r_e, 100)},
                              "sequential": {"solves_per_s": round(thr(r_s, t0s), 1), **latency_stats(r_s, 100)}})
    return out


def mc_bytes(r: int, nv: int, nt: int, backward: bool = False) -> int:
    """Algorithmic bytes of the Marching Cubes layer: the grid read once and
    the mesh written once (positions, normals, edge ids: 28 B per vertex;
    triangles 12 B), or for the backward the grid read, dL/dchi written and
    dL/dverts and the normals read (24 B per vertex). Counted densely: the
    backward's workgroups without surface write zeros and read nothing."""
    n = r ** 3
    return 8 * n + 24 * nv if backward else 4 * n + 28 * nv + 12 * nt


def marching_cubes_leg(dev, torch, chi, steps=20, warmup=3):
    """Marching Cubes of a solver output (level 0) and its backward, timed
    with HIP events around the library calls on the current stream."""
    import ctypes
    from paper_2106_03452_amd import _lib
    from paper_2106_03452_amd import mesh as M
    L = _lib.lib()
    ctx = _lib.context(0)
    m = M.marching_cubes(chi)
    r = int(chi.shape[0])
    nv, nt = int(m.verts.shape[0]), int(m.faces.shape[0])
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    verts = torch.empty((nv, 3), dtype=torch.float32, device=dev)
    nrm = torch.empty((nv, 3), dtype=torch.float32, device=dev)
    edges = torch.empty((nv,), dtype=torch.int32, device=dev)
    tris = torch.empty((nt, 3), dtype=torch.int32, device=dev)
    state = torch.empty_like(m.state)
    dv = torch.randn((nv, 3), dtype=torch.float32, device=dev)
    dchi = torch.empty_like(chi)

    def fwd():
        _lib.check(L.psr_marching_cubes(ctx.handle, p(chi), r, 0.0, p(verts), p(nrm), p(edges), nv, p(tris), nt,
                                        p(state), st), "psr_marching_cubes")

    def bwd():
        _lib.check(L.psr_marching_cubes_backward(ctx.handle, p(chi), r, 0.0, p(state), p(nrm), p(dv), nv, p(dchi),
                                                 st), "psr_marching_cubes_backward")
    out = {"res": r, "vertices": nv, "triangles": nt}
    for name, fn, back in (("forward", fwd, False), ("backward", bwd, True)):
        for _ in range(warmup):
            fn()
        ms = step_times(fn, steps, torch)["median_ms"]
        b = mc_bytes(r, nv, nt, back)
        out[name] = {"ms": ms, "algorithmic_bytes": b, "GBs": round(b / (ms * 1e-3) / 1e9, 1),
                     "hbm_frac": round(b / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)}
    return out


def optimisation_leg(dev, torch, iters=40, npoints=20000):
    """The optimisation loop of main Sec. 3.2 on a synthetic target (a rotated
    torus, 20k points): ms per iteration (solve, Marching Cubes, sampling,
    Chamfer, every backward and the Adam step) at each grid size of the
    paper's schedule, a resampling from the largest component included every
    `iters // 2` iterations, and the whole schedule's time from them; each
    iteration one psr_opt_step call, and beside it the same loop through the
    autograd Functions and PyTorch's Adam."""
    import psr_synth as S
    from paper_2106_03452_amd import optimize as O
    target = torch.from_numpy(S.tiny_case(8, 256, npoints, kind="torus").points).to(dev)
    out = {"workload": f"{npoints}-point torus target, {npoints} source points and samples, "
                       f"{iters} iterations per grid size", "ms_per_iter": {}}
    out["ms_per_iter_autograd"] = {}
    for lev in O.PAPER_SCHEDULE:
        for native, key in ((True, "ms_per_iter"), (False, "ms_per_iter_autograd")):
            # a short untimed run first: first-use costs (tables, allocator) stay out
            O.optimise(target, [O.Level(lev.res, lev.sigma, 5)], npoints=npoints, resample_every=100, log_every=0,
                       native=native)
            r = O.optimise(target, [O.Level(lev.res, lev.sigma, iters)], npoints=npoints,
                           resample_every=iters // 2, log_every=0, native=native)
            out[key][str(lev.res)] = round(r.ms_per_iter[lev.res], 3)
    full = sum(out["ms_per_iter"][str(l.res)] * l.iters for l in O.PAPER_SCHEDULE) / 1e3
    out["schedule_s"] = round(full, 2)
    out["schedule"] = "32^3 x1000, 64^3 x1000, 128^3 x1000, 256^3 x200 (sigma 2, 2, 3, 3)"
    out["paper_gtx1080ti_s"] = "326-380 per object (its Table: Thingi10K, SRB, D-FAUST)"
    return out


def training_leg(dev, torch, batch=8, steps=10, warmup=3, res=128):
    """One DPSR-loss training step (main Sec. 3.3): the point network, the
    batched solve of all shapes, the MSE against the ground-truth grids,
    every backward and the Adam step; 3,000 noisy input points per shape and
    k = 7 offsets (21,000 oriented points per shape) at 128^3."""
    import numpy as np
    import psr_synth as S
    from paper_2106_03452_amd import function as F
    from paper_2106_03452_amd import learn
    rng = np.random.default_rng(7)
    c_in, gt = [], []
    for _ in range(batch):
        sh = S.random_shape(rng, res, 20000)
        c_in.append(sh.points[:3000] + rng.normal(0, 0.005, (3000, 3)).astype(np.float32))
        chi, _ = F.forward(torch.from_numpy(sh.points).to(dev), torch.from_numpy(sh.normals).to(dev), res, 2.0)
        gt.append(chi)
    c = torch.from_numpy(np.stack(c_in)).to(dev)
    torch.manual_seed(0)
    model = learn.OffsetNormalNet(k=7).to(dev)
    opt = torch.optim.Adam(model.parameters(), lr=1e-4, fused=True)
    for _ in range(warmup):
        learn.train_step(model, opt, c, gt, res)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        loss = learn.train_step(model, opt, c, gt, res)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) / steps * 1e3
    return {"workload": f"batch of {batch} shapes, 3,000 input points x 7 offsets, {res}^3, sigma 2",
            "ms_per_step": round(ms, 3), "shapes_per_s": round(batch / ms * 1e3, 1), "loss": float(loss),
            "paper_context": "about 0.58 s per step of batch 32 on 2 GTX 1080Ti (2 days for 300k steps, whole model)"}


def timed(step, steps, warmup, torch):
    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        step()
    torch.cuda.synchronize()
    return time.perf_counter() - t0


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-secondary", action="store_true", help="skip the 128^3 and forward-only lines")
    ap.add_argument("--mode", choices=["solve", "serve"], default="solve",
                    help="solve: the fwd+bwd throughput line (default); serve: the request-stream measurement")
    ap.add_argument("--requests", type=int, default=2000, help="serve mode: requests per QPS level")
    ap.add_argument("--serve-requests", type=int, default=600,
                    help="requests of the compact serving leg of the default run (levels 1.0 and 1.5 x lambda_seq)")
    ap.add_argument("--no-serve", action="store_true", help="skip the compact serving leg")
    ap.add_argument("--no-loops", action="store_true", help="skip the optimisation-loop and training-step legs")
    ap.add_argument("--workload", choices=["c3", "c2", "c4", "mc", "slab", "sweep", "opt"], default="c3",
                    help="profiling runs: c3 = the headline line (default); c2 = only the 128^3 fwd+bwd steps; "
                         "c4 = only the 64-shape batch; mc = only Marching Cubes of the 256^3 solve; "
                         "slab = only the 1024^3 slab forward; sweep = grid sizes 64-512 x 1e4-1e6 points "
                         "and the 1024^3 slab forward at 2, 8, 32 slabs; opt = only the optimisation loop "
                         "(--steps iterations per grid size)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="only run a plain device copy of 1 GiB five times (scale reference for HBM counters)")
    ap.add_argument("--ingest-counters", nargs=4, metavar=("FETCH_CSV", "WRITE_CSV", "COPY_FETCH_CSV", "COPY_WRITE_CSV"),
                    help="host only: turn rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE CSVs of this bench and of "
                         "--calibrate-copy into profiles/hbm_traffic_c3_256.json")
    args = ap.parse_args()
    if args.ingest_counters:
        print(json.dumps(ingest_counters(*args.ingest_counters), indent=1))
        return
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: the solver runs on a single MI355X (a multi-GPU slab "
              "decomposition is described, not implemented). Run with --gpus 1.", file=sys.stderr)
        sys.exit(2)

    import torch
    dev = torch.device("cuda", 0)
    if args.calibrate_copy:
        n = 1 << 28  # 2^28 float32 = 1 GiB
        src = torch.ones(n, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        dt = (time.perf_counter() - t0) / 5
        print(json.dumps({"copy_bytes_read": 4 * n, "copy_bytes_written": 4 * n, "ms": round(dt * 1e3, 4),
                          "GBs_read_plus_write": round(8 * n / dt / 1e9, 1)}), flush=True)
        return

    if args.mode == "serve":
        print(json.dumps(serve_mode(dev, torch, args.requests)), flush=True)
        return

    import psr_synth as S
    from paper_2106_03452_amd import _lib
    from paper_2106_03452_amd import function as F

    ctx = _lib.context(0)
    if args.workload != "c3":
        # profiling runs of one secondary workload (no JSON contract line)
        if args.workload == "c2":
            b2 = prepare(S.config_c2(), dev, torch, F)
            dt = timed(make_step(b2, ctx), args.steps, args.warmup, torch)
            print(json.dumps({"workload": "c2", "ms_per_step": round(dt / args.steps * 1e3, 4)}), flush=True)
        elif args.workload == "sweep":
            print(json.dumps({"workload": "sweep", **sweep(dev, torch)}), flush=True)
        elif args.workload == "slab":
            print(json.dumps({"workload": "slab", **slab_leg(dev, torch, args.steps, args.warmup)}), flush=True)
        elif args.workload == "c4":
            print(json.dumps({"workload": "c4", **batch_c4(dev, torch, args.steps, args.warmup)}), flush=True)
        elif args.workload == "opt":
            print(json.dumps({"workload": "opt", **optimisation_leg(dev, torch, iters=max(2, args.steps))}),
                  flush=True)
        else:
            b3 = prepare(S.config_c3(), dev, torch, F)
            print(json.dumps({"workload": "mc", **marching_cubes_leg(dev, torch, b3["chi"], args.steps)}), flush=True)
        return
    shape = S.config_c3()
    b = prepare(shape, dev, torch, F)
    r, P = b["r"], b["P"]

    # main timed region: forward + backward, no per-kernel events
    step = make_step(b, ctx)
    dt = timed(step, args.steps, args.warmup, torch)
    ms = dt / args.steps * 1e3
    value = args.steps / dt

    # per-stage durations (HIP events on the solve stream) to find the dominant kernel
    ctx.set("timers", 1)
    ctx.reset_timers()
    timed(step, max(5, args.steps // 3), 1, torch)
    times = ctx.stage_times()
    per_launch = {k: (v[0] / v[1]) for k, v in times.items() if v[1] > 0}
    dom = max(per_launch, key=lambda k: per_launch[k])
    # time the dominant kernel alone inside a timed region identical to the main one
    names = [_lib.lib().psr_stage_name(i).decode() for i in range(_lib.lib().psr_num_stages())]
    ctx.set("timer_mask", 1 << names.index(dom))
    ctx.reset_timers()
    dt2 = timed(step, args.steps, 1, torch)
    t_dom = ctx.stage_times()[dom]
    ctx.set("timers", 0)
    dom_ms = t_dom[0] / t_dom[1]
    fp, ft = live_fractions(shape.points, r)
    sb = stage_bytes(r, P, fp, ft)
    achieved = sb[dom] / (dom_ms * 1e-3) / 1e9
    traffic = traffic_from_profiles(dom, "c3_256")
    roof = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
            "kernel": dom, "algorithmic_bytes_per_launch": round(sb[dom]), "avg_launch_ms": round(dom_ms, 5),
            "live_plane_fraction": round(fp, 4), "live_tile_fraction": round(ft, 4)}
    step_bytes = b_stage(r, P)
    rate = lambda nbytes, ms_: nbytes / (ms_ * 1e-3) / 1e9
    # B_stage counts every plane and row tile; the kernels skip the point-free
    # ones, so this is a dense-equivalent rate, not bytes moved over HBM
    step_dense = {"bytes": step_bytes, "achieved_GBs": round(rate(step_bytes, ms), 1),
                  "frac": round(rate(step_bytes, ms) / HBM_PEAK_GBS, 4),
                  "model": "B_stage = 128 r^3 + 72 P (fwd+bwd), every plane and row tile counted: a "
                           "dense-equivalent rate (the kernels skip point-free planes and tiles)",
                  "B_min": 56 * r ** 3 + 72 * P,
                  "B_min_frac": round(rate(56 * r ** 3 + 72 * P, ms) / HBM_PEAK_GBS, 4)}
    sk = skip_aware_bytes(r, P, fp, ft)
    step_skip = {"bytes": round(sk), "achieved_GBs": round(rate(sk, ms), 1),
                 "frac": round(rate(sk, ms) / HBM_PEAK_GBS, 4),
                 "model": "sum of the algorithmic bytes of the stages run, point-free planes and row tiles left out",
                 "live_plane_fraction": round(fp, 4), "live_tile_fraction": round(ft, 4)}
    breakdown = {k: round(v, 4) for k, v in sorted(per_launch.items(), key=lambda kv: -kv[1])}
    tr = json.load(open(os.path.join(ROOT, "profiles", "hbm_traffic_c3_256.json"))) if traffic is not None else None
    if tr is not None:
        cb = sum(v["hbm_bytes_per_launch"] for v in tr["stages"].values())
        step_skip["counter_bytes_large_kernels"] = cb
        step_skip["counter_frac_large_kernels"] = round(rate(cb, ms) / HBM_PEAK_GBS, 4)
    # warm (back-to-back) and cold (caches scrubbed by a 512 MiB write) repetitions
    scrub = torch.empty(1 << 27, dtype=torch.float32, device=dev)
    timing = {"warm": step_times(step, 50, torch), "cold": step_times(step, 50, torch, scrub)}
    del scrub

    secondary = {}
    if not args.no_secondary:
        fwd = make_step(b, ctx, backward=False)
        dtf = timed(fwd, args.steps, 2, torch)
        secondary["fwd_only_256"] = {"solves_per_s": round(args.steps / dtf, 2), "ms": round(dtf / args.steps * 1e3, 4),
                                     "paper_gtx1080ti_ms": 140.0}
        sh2 = S.config_c2()
        b2 = prepare(sh2, dev, torch, F)
        s2 = make_step(b2, ctx)
        d2 = timed(s2, args.steps * 3, args.warmup, torch)
        ms2 = d2 / (args.steps * 3) * 1e3
        scrub = torch.empty(1 << 27, dtype=torch.float32, device=dev)
        secondary["fwd_bwd_128"] = {"solves_per_s": round(args.steps * 3 / d2, 2), "ms": round(ms2, 4),
                                    "step_roofline_frac": round(b_stage(128, sh2.P) / (ms2 * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
                                    "workload": "128^3, 20k points torus+sphere, sigma 2",
                                    "step_timing_200": {"warm": step_times(s2, 200, torch),
                                                        "cold": step_times(s2, 200, torch, scrub)}}
        del scrub
        f2 = make_step(b2, ctx, backward=False)
        d3 = timed(f2, args.steps * 3, 2, torch)
        secondary["fwd_only_128"] = {"solves_per_s": round(args.steps * 3 / d3, 2),
                                     "ms": round(d3 / (args.steps * 3) * 1e3, 4), "paper_gtx1080ti_ms": 12.0}
        del b2
        # the dense worst case: half of the C3 cloud replaced by uniform outliers,
        # so every plane and row tile is live and nothing can be skipped
        sh3 = S.config_c3_outliers()
        b3 = prepare(sh3, dev, torch, F)
        s3 = make_step(b3, ctx)
        d3 = timed(s3, args.steps, args.warmup, torch)
        ms3 = d3 / args.steps * 1e3
        ctx.set("timers", 1)
        ctx.reset_timers()
        timed(s3, max(5, args.steps // 3), 1, torch)
        st3 = {k: round(v[0] / v[1], 4) for k, v in ctx.stage_times().items() if v[1] > 0}
        ctx.set("timers", 0)
        fp3, ft3 = live_fractions(sh3.points, 256)
        sk3 = skip_aware_bytes(256, sh3.P, fp3, ft3)
        secondary["fwd_bwd_256_no_skip"] = {
            "workload": "the 256^3 cloud with 50% of its 100k points replaced by uniform outliers "
                        "(|n| ~ U[0, 0.05]): every plane and row tile holds points",
            "solves_per_s": round(args.steps / d3, 2), "ms": round(ms3, 4),
            "live_plane_fraction": round(fp3, 4), "live_tile_fraction": round(ft3, 4),
            "algorithmic_bytes": round(sk3), "hbm_frac": round(rate(sk3, ms3) / HBM_PEAK_GBS, 4),
            "dense_equivalent_frac": round(rate(b_stage(256, sh3.P), ms3) / HBM_PEAK_GBS, 4),
            "stage_ms": dict(sorted(st3.items(), key=lambda kv: -kv[1]))}
        del b3
        sh1 = S.config_c1()
        b1 = prepare(sh1, dev, torch, F)
        f1 = make_step(b1, ctx, backward=False)
        d1 = timed(f1, args.steps * 10, args.warmup, torch)
        secondary["fwd_only_32"] = {"workload": "32^3, 3,000 points on a sphere, sigma 2, forward only",
                                    "solves_per_s": round(args.steps * 10 / d1, 1),
                                    "ms": round(d1 / (args.steps * 10) * 1e3, 4)}
        del b1
        secondary["batch_c4"] = batch_c4(dev, torch)
        secondary["batch_128"] = batch_c2(dev, torch)
        secondary["marching_cubes_256"] = marching_cubes_leg(dev, torch, b["chi"])
        secondary["slab_1024"] = slab_leg(dev, torch)
        if not args.no_loops:
            secondary["optimisation_loop"] = optimisation_leg(dev, torch)
            secondary["training_step_128"] = training_leg(dev, torch)
        if not args.no_serve:
            secondary["serve_c5"] = serve_mode(dev, torch, args.serve_requests, levels=(1.0, 1.5))

    gpu_result = None
    if not args.no_cpu_baseline:
        step()
        torch.cuda.synchronize()
        gpu_result = tuple(t.detach().cpu().numpy() for t in (b["chi"], b["dp"], b["dn"]))
    cpu = None if args.no_cpu_baseline else cpu_baseline(gpu_result)
    out = {
        "metric": METRIC, "value": round(value, 3), "unit": "solves/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms, 4), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "fwd+bwd 256^3, 100k points on a superellipsoid (seed 2), noisy normals, sigma 2",
                   "res": r, "npoints": P, "sigma": shape.sigma, "precision": "FP32 grid, FP64 reductions",
                   "parallelism": "single GPU"},
        "roofline": roof, "step_roofline_dense_equivalent": step_dense, "step_roofline_skip_aware": step_skip,
        "step_timing_50": timing, "stage_ms": breakdown,
        "dominant_kernel_region_ms_per_step": round(dt2 / args.steps * 1e3, 4),
        "secondary": secondary, "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
