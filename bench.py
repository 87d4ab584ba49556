"""Benchmark of the solution-transfer DD hot path on one MI355X.

Workload: the 2D variable-coefficient convection-diffusion problem on a
1023 x 1023 interior grid cut into 32 slabs of 32 cells (31 interfaces of
1023 nodes), kappa = exp(0.5 G) from 16 seeded Fourier modes, b = (10, 0),
f ~ N(0,1), g = 0 -- synthetic inputs generated on the host and resident in
HBM before the timed region.

One step = one pass of the hot path: build every transfer block by batched
elimination (FP32 on the matrix cores) + solve the equilibrium system by
GMRES inside FP64 iterative refinement, to a predicted relative error of
1e-9 (target 1e-8).  value = N / (seconds per step), N = 1023^2 DOFs.  The
FP64 plain path (FP64 build, same solver) is timed beside it, and the
adjoint of a sensor loss (factors recomputed) is timed once, and so is the
matrix-free alternative (S applied by sweeps with the stored slab factors,
set-up without the transfer blocks) beside the dense-block form, and one
solve of 8 right-hand sides together beside single solves.  The two
largest workloads (2D oscillatory 2047^2 on 64 slabs, 3D variable
coefficient 127^3 on 16 slabs) are each timed once end to end by two
routes: the dense transfer blocks compressed as HODLR, and the paper's
sampled construction (Algorithm 1) without dense blocks, compressed as HBS.
Hardware counters of the dominant kernel (HBM bytes, executed matrix-core
flops) come from rocprofv3 passes over child runs of this same script,
before the timed runs.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu] [--no-pmc]
                       [--no-large]
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

PEAK = {"fp32_mfma_tflops": 157.3, "fp64_mfma_tflops": 78.6, "bf16_mfma_tflops": 2500.0,
        "hbm_gbs": 8000.0}
# The FP32 products of the build run on the BF16 matrix cores: each FP32
# operand is split into three BF16 parts and every 16x16x32 FP32 tile
# product costs six BF16 products, so the ceiling of that arithmetic is the
# dense BF16 peak / 6 (FP32-equivalent flops).
X6_PRODUCTS = 6
PEAK["fp32_via_bf16x6_tflops"] = PEAK["bf16_mfma_tflops"] / X6_PRODUCTS
# width of the pivot blocks of the library's Gauss-Jordan inversion (the rank
# of each update step)
GJ_RANK = 128


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle leg")
    ap.add_argument("--no-fp64", action="store_true", help="skip the FP64 plain path")
    ap.add_argument("--no-adjoint", action="store_true")
    ap.add_argument("--no-matfree", action="store_true",
                    help="skip the matrix-free comparison (untimed, after the timed steps)")
    ap.add_argument("--no-many", action="store_true",
                    help="skip the many-right-hand-side solve (untimed, after the timed steps)")
    ap.add_argument("--n", type=int, default=None, help="reduced grid (debug only)")
    ap.add_argument("--slabs", type=int, default=None)
    ap.add_argument("--copy-bytes", type=int, default=0,
                    help="run one device-to-device copy of this many bytes first (a kernel of "
                         "known traffic, to calibrate hardware byte counters)")
    ap.add_argument("--no-pmc", action="store_true",
                    help="skip the hardware-counter passes (rocprofv3 over child runs)")
    ap.add_argument("--no-large", action="store_true",
                    help="skip the 2047^2 and 127^3 workloads (timed once each)")
    ap.add_argument("--only-large", action="store_true",
                    help="run only the 2047^2 and 127^3 workloads and print their JSON object")
    ap.add_argument("--pmc-child", action="store_true",
                    help="internal: one calibration copy and one step, nothing printed")
    return ap.parse_args()


def step(dd, dev, precision, opts):
    op = dd.Operator(2, dev["n"], dev["n_slabs"], kappa=dev["kappa"], bvec=dev["bvec"],
                     precision=precision)
    u, _, st = op.solve(dev["f"], opts=opts, want_gamma=False, allow_notconv=True)
    op.close()
    return u, st


def timed(dd, torch, dev, precision, opts, steps, warmup, profile):
    """Warm-up, then (with profile) one untimed step with every kernel class
    timed, which gives the per-step kernel mix and names the dominant class,
    then `steps` timed steps with per-launch HIP events on that class only
    (events attached to its dispatches: about 0.3% of step time, where
    timing every class costs about 4%)."""
    for _ in range(warmup):
        step(dd, dev, precision, opts)
    torch.cuda.synchronize()
    mix = None
    if profile:
        dd.profile_enable(True)
        step(dd, dev, precision, opts)
        torch.cuda.synchronize()
        mix = dd.profile_read()
        dominant = max(mix.items(), key=lambda kv: kv[1][1])[0]
        dd.profile_enable(True, kinds=[dominant])
    stats = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    u = None
    for _ in range(steps):
        u, st = step(dd, dev, precision, opts)
        stats.append(st)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    prof = dd.profile_read() if profile else None
    if profile:
        busy = dd.profile_busy()
        prof = {k: v + (busy[k],) for k, v in prof.items()}
        dd.profile_enable(False)
    return (t1 - t0) / steps, stats, u, prof, mix


PMC_COPY_BYTES = 256 << 20  # calibration copy of the counter passes
# the kernels of the update class: rank-128 updates, and the products of the
# outer blocks
PMC_KERNELS = ("k_gj_update", "k_gj_left", "k_gj_right")


def _pmc_rows(outdir):
    """Rows of every rocprofv3 counter-collection CSV under outdir."""
    import csv
    import glob
    rows = []
    for f in glob.glob(os.path.join(outdir, "**", "*counter_collection.csv"), recursive=True):
        with open(f, newline="") as fh:
            rows.extend(csv.DictReader(fh))
    return rows


def _per_dispatch(rows, kernel_subs, counter):
    """{dispatch id: summed counter value} of the dispatches whose kernel name
    contains one of kernel_subs."""
    out = {}
    for r in rows:
        name = r.get("Kernel_Name", "")
        if not any(k in name for k in kernel_subs) or r.get("Counter_Name") != counter:
            continue
        d = r.get("Dispatch_Id") or r.get("Correlation_Id")
        out[d] = out.get(d, 0.0) + float(r.get("Counter_Value", 0.0))
    return out


def pmc_measure(root):
    """Hardware counters of the dominant kernel, measured now: three rocprofv3
    passes (one counter set each, as the profiler requires) over a child run
    of this script (one 256 MiB device copy, then one step).  Byte counters
    are calibrated by the copy kernel (its true traffic is known):
    bytes = raw KiB x 1024 x (copy bytes / copy's raw bytes).  Returns a dict
    (entries None when a pass fails)."""
    import shutil
    import subprocess
    import tempfile
    res = {"traffic_bytes_per_launch": None, "fetch_scale": None, "write_scale": None,
           "mfma_flops_per_launch": None, "mfma_bf16_flops_per_launch": None,
           "mfma_busy_serialised": None, "launches": None,
           "error": None}
    prof = shutil.which("rocprofv3")
    if prof is None:
        res["error"] = "rocprofv3 not found"
        return res
    passes = {"fetch": ["FETCH_SIZE"], "write": ["WRITE_SIZE"],
              "mfma": ["SQ_INSTS_VALU_MFMA_MOPS_BF16", "SQ_INSTS_VALU_MFMA_MOPS_F32",
                       "SQ_VALU_MFMA_BUSY_CYCLES", "GRBM_GUI_ACTIVE"]}
    rows = {}
    tmp = tempfile.mkdtemp(prefix="ddst_pmc_", dir="/tmp")
    env = dict(os.environ, TMPDIR="/tmp")
    for name, counters in passes.items():
        out = os.path.join(tmp, name)
        cmd = ["timeout", "-s", "KILL", "150", prof, "--pmc", *counters, "-f", "csv", "-d", out,
               "-o", name, "--", sys.executable, os.path.join(root, "bench.py"), "--pmc-child"]
        print(f"[bench] counter pass {name}: {' '.join(counters)}", file=sys.stderr, flush=True)
        try:
            r = subprocess.run(cmd, cwd="/tmp", env=env, capture_output=True, text=True,
                               timeout=170)
            rows[name] = _pmc_rows(out)
            if not rows[name]:
                res["error"] = f"pass {name}: no counter rows (rc {r.returncode}): " + \
                    (r.stderr or "")[-300:]
        except Exception as e:  # noqa: BLE001 - reported, never fatal
            rows[name] = []
            res["error"] = f"pass {name}: {e}"
    shutil.rmtree(tmp, ignore_errors=True)

    def scale(counter, rws):
        copy = _per_dispatch(rws, ("copyBuffer",), counter)
        big = [v for v in copy.values() if v * 1024 > PMC_COPY_BYTES / 4]
        return PMC_COPY_BYTES / (big[0] * 1024) if big else None

    f = _per_dispatch(rows.get("fetch", []), PMC_KERNELS, "FETCH_SIZE")
    w = _per_dispatch(rows.get("write", []), PMC_KERNELS, "WRITE_SIZE")
    fs, ws = scale("FETCH_SIZE", rows.get("fetch", [])), scale("WRITE_SIZE", rows.get("write", []))
    res["fetch_scale"], res["write_scale"] = fs, ws
    if f and w and fs and ws:
        res["launches"] = len(f)
        res["traffic_bytes_per_launch"] = (sum(f.values()) / len(f) * fs
                                           + sum(w.values()) / len(w) * ws) * 1024.0
    mr = rows.get("mfma", [])
    mops = _per_dispatch(mr, PMC_KERNELS, "SQ_INSTS_VALU_MFMA_MOPS_F32")
    mops16 = _per_dispatch(mr, PMC_KERNELS, "SQ_INSTS_VALU_MFMA_MOPS_BF16")
    busy = _per_dispatch(mr, PMC_KERNELS, "SQ_VALU_MFMA_BUSY_CYCLES")
    act = _per_dispatch(mr, PMC_KERNELS, "GRBM_GUI_ACTIVE")
    # the counters count matrix-core operations in units of 512 flops
    if mops:
        res["mfma_flops_per_launch"] = 512.0 * sum(mops.values()) / len(mops)
    if mops16:
        res["mfma_bf16_flops_per_launch"] = 512.0 * sum(mops16.values()) / len(mops16)
    if busy and act and sum(act.values()) > 0:
        # busy cycles summed over the SIMDs; active cycles summed over the
        # 8 XCDs: fraction = busy / (active / 8 x 1024 SIMDs)
        res["mfma_busy_serialised"] = sum(busy.values()) / (sum(act.values()) / 8.0 * 1024.0)
    return res


def pmc_child():
    """One calibration copy and one step of the benchmark workload (run under
    rocprofv3 by pmc_measure)."""
    import torch
    from problems import make_config
    from paper_2510_25991_amd import ddst as dd
    src = torch.ones(PMC_COPY_BYTES // 4, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    del src, dst
    prob = make_config("cfg2")
    dev = {"n": prob.n, "n_slabs": prob.n_slabs, "bvec": prob.bvec,
           "kappa": torch.tensor(prob.kappa, dtype=torch.float64, device="cuda"),
           "f": torch.tensor(prob.f, dtype=torch.float64, device="cuda")}
    step(dd, dev, "fp32", dd.SolveOptions(tol=1e-9, max_outer=6))
    torch.cuda.synchronize()


def outer_blocks(nmat, M, symmetric):
    """Whether FP32 matrices are eliminated in outer blocks (the rule and its
    constants: csrc/rules.h)."""
    import re
    text = open(os.path.join(ROOT, "paper_2510_25991_amd", "csrc", "rules.h")).read()
    rows, tiles = (int(re.search(r"constexpr int %s = (\d+);" % k, text).group(1))
                   for k in ("kOuterRows", "kOuterTiles"))
    ld = (M + 127) // 128 * 128
    return ld >= rows and nmat * (ld / 256.0) ** 2 >= tiles * (2 if symmetric else 1)


def gj_update_bytes_per_flop(M, esz, outer):
    """Algorithmic bytes per flop of the Gauss-Jordan updates of one M x M
    inverse.  One level: every step is a rank-r update (r = GJ_RANK) of the
    M - r rows outside the pivot block, 2 r M (M - r) flops; it reads and writes
    those rows once, writes the r pivot rows and reads the two panels,
    esz (2 M^2 + r M - r^2) bytes.  Outer blocks of w <= 512: the steps of one
    level on the w x w block, the rank-w update of the other rows and columns
    (2 w (M - w)^2 flops; they are read and written, the panels read), and the
    products of both panels with the block's inverse (2 w^2 (M - w) flops each;
    the panel is read and written, the inverse read)."""
    def level(m):  # m rows in all their steps
        steps = (m + GJ_RANK - 1) // GJ_RANK
        r = GJ_RANK
        return (steps * 2.0 * r * m * max(m - r, 0),
                steps * esz * (2.0 * m * m + r * m - r * r))
    if not outer:
        f, b = level(M)
        return b / f
    f = b = 0.0
    for p0 in range(0, M, 512):
        w = min(512, M - p0)
        o = M - w
        fi, bi = level(w)
        f += fi + 2.0 * w * o * o + 4.0 * w * w * o
        b += bi + esz * (2.0 * o * o + 2.0 * w * o + 2 * (2.0 * w * o + w * w))
    return b / f


def roofline(prof, precision, M, pmc=None, outer=False):
    """Dominant kernel class (the only class timed in the timed region, else
    the longest); achieved = algorithmic work per launch / average launch
    duration (HIP events on the stream each launch runs on).

    The bound of the Gauss-Jordan updates (gj_update_bytes_per_flop) is
    whichever floor is higher: HBM (algorithmic bytes / 8 TB/s) or the matrix
    cores (flops / dense MFMA peak of the precision).  At M = 1023 the
    intensity is about 26.5 flop/B in FP32 by one level, 51 by outer blocks,
    and 13.3 in FP64, above the ridges of the FP32 and FP64 instructions (157.3
    / 8 and 78.6 / 8).  The FP32 products run as six BF16 products each
    (three-part split), so the matrix-core ceiling of the FP32 path is the BF16
    dense peak / 6 = 416.7 TFLOP/s of FP32 work, ridge 52 flop/B: at M = 1023
    the FP32 updates are HBM-bound by one level, and near both bounds by outer
    blocks; the FP64 ones are MFMA-bound.
    The rate against the FP32 instruction's own peak is given beside it.
    Launches
    of the look-ahead schedule cover subsets of the tiles; their work is
    summed, so the figures are averages over all update launches.  Two of
    them run at once on different streams, so the average launch duration
    counts shared time twice: achieved_union divides the same work by the
    union of the launch intervals instead."""
    name, (n, ms, work, busy_ms) = max(prof.items(), key=lambda kv: kv[1][1])
    avg_s = ms / 1e3 / max(n, 1)
    esz = 4 if precision == "fp32" else 8
    mpeak = (PEAK["fp32_via_bf16x6_tflops"] if precision == "fp32"
             else PEAK["fp64_mfma_tflops"])
    base = {"kernel": name, "launches": n, "avg_launch_us": round(avg_s * 1e6, 2)}
    if busy_ms > 0 and name in ("gj_update", "gemm", "gj_panel"):
        ach_u = work / (busy_ms / 1e3) / 1e12
        base.update({"union_ms": round(busy_ms, 3), "overlap": round(ms / busy_ms, 3),
                     "achieved_union": round(ach_u, 3), "frac_union": round(ach_u / mpeak, 4)})
    if name == "gj_update":
        flops_per_launch = work / max(n, 1)
        bytes_per_flop = gj_update_bytes_per_flop(M, esz, outer)
        bytes_per_launch = flops_per_launch * bytes_per_flop
        hbm_floor = bytes_per_launch / (PEAK["hbm_gbs"] * 1e9)
        mfma_floor = flops_per_launch / (mpeak * 1e12)
        pm = pmc if (pmc and precision == "fp32") else {}
        tr = pm.get("traffic_bytes_per_launch")
        ex = pm.get("mfma_flops_per_launch")
        extra = {"traffic": tr, "bytes_per_launch": bytes_per_launch,
                 "traffic_ratio": round(tr / bytes_per_launch, 3) if tr else None,
                 "flops_per_launch": flops_per_launch,
                 # executed matrix-core flops from SQ_INSTS_VALU_MFMA_MOPS_F32
                 "flops_executed_per_launch": ex,
                 "executed_over_algorithmic": round(ex / flops_per_launch, 3) if ex else None,
                 # executed BF16 matrix-core flops (SQ_INSTS_VALU_MFMA_MOPS_BF16):
                 # six BF16 products per FP32 product
                 "bf16_flops_executed_per_launch": pm.get("mfma_bf16_flops_per_launch"),
                 "bf16_executed_over_algorithmic": (
                     round(pm["mfma_bf16_flops_per_launch"] / flops_per_launch, 3)
                     if pm.get("mfma_bf16_flops_per_launch") else None),
                 "peak_basis": ("BF16 dense peak 2500 TFLOP/s / 6 BF16 products per FP32 "
                                "product" if precision == "fp32" else "FP64 dense MFMA peak"),
                 "frac_vs_fp32_instruction_peak": (
                     round(flops_per_launch / avg_s / 1e12 / PEAK["fp32_mfma_tflops"], 4)
                     if precision == "fp32" else None),
                 "hbm_gbs": round(bytes_per_launch / avg_s / 1e9, 1),
                 # matrix-core busy fraction of the same launches when rocprofv3
                 # serialises them (the two look-ahead halves otherwise overlap,
                 # which lengthens each launch's duration above)
                 "mfma_busy_serialised": (round(pm["mfma_busy_serialised"], 4)
                                          if pm.get("mfma_busy_serialised") else None),
                 "counters": ({"launches": pm.get("launches"), "fetch_scale": pm.get("fetch_scale"),
                               "write_scale": pm.get("write_scale"), "error": pm.get("error")}
                              if pm else None),
                 "mfma_tflops": round(flops_per_launch / avg_s / 1e12, 3),
                 "frac_mfma": round(flops_per_launch / avg_s / 1e12 / mpeak, 4)}
        if mfma_floor >= hbm_floor:
            achieved = flops_per_launch / avg_s / 1e12
            return name, {"bound": "mfma", "achieved": round(achieved, 3), "peak": mpeak,
                          "unit": "TFLOP/s", "frac": round(achieved / mpeak, 4),
                          **extra, **base}
        achieved = bytes_per_launch / avg_s / 1e9
        return name, {"bound": "hbm", "achieved": round(achieved, 1), "peak": PEAK["hbm_gbs"],
                      "unit": "GB/s", "frac": round(achieved / PEAK["hbm_gbs"], 4),
                      **extra, **base}
    if name in ("gemm", "gj_panel"):
        achieved = work / max(n, 1) / avg_s / 1e12
        peak = mpeak
        return name, {"bound": "mfma", "achieved": round(achieved, 3), "peak": peak,
                      "unit": "TFLOP/s", "frac": round(achieved / peak, 4), "traffic": None,
                      "flops_per_launch": work / max(n, 1), **base}
    achieved = work / max(n, 1) / avg_s / 1e9
    return name, {"bound": "hbm", "achieved": round(achieved, 1), "peak": PEAK["hbm_gbs"],
                  "unit": "GB/s", "frac": round(achieved / PEAK["hbm_gbs"], 4), "traffic": None,
                  "bytes_per_launch": work / max(n, 1), **base}


def cpu_leg(prob, u_mixed, u_fp64):
    """The FP64 oracle on a bounded sample of the same workload, plus the
    accuracy of both GPU paths against the oracle's global direct solve."""
    import numpy as np
    from oracle import dd as odd
    from oracle import fd as ofd
    try:
        from threadpoolctl import threadpool_info
        blas_threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        blas_threads = os.cpu_count() or 1
    o = odd.DDOracle(prob)
    b = o.rhs()
    sample_ds = [prob.n_ds // 2, prob.n_ds // 2 + 1]
    t0 = time.perf_counter()
    for j in sample_ds:
        for jp in (j - 1, j + 1):
            if 1 <= jp <= prob.n_ds:
                o.transfer_block(j, jp)
    t_blocks = (time.perf_counter() - t0) / len(sample_ds)
    t0 = time.perf_counter()
    _ = o.loads(b)
    t_loads = time.perf_counter() - t0
    ug = np.zeros((prob.n_ds, prob.M))
    t0 = time.perf_counter()
    _ = o.reconstruct(b, ug)
    t_recon = time.perf_counter() - t0
    t_total = t_blocks * prob.n_ds + t_loads + t_recon
    t0 = time.perf_counter()
    ref = ofd.solve_global(prob)
    t_direct = time.perf_counter() - t0
    scale = float(np.abs(ref).max())
    errs = {}
    for k, u in (("mixed", u_mixed), ("fp64", u_fp64)):
        if u is not None:
            errs[k] = float(np.abs(u.cpu().numpy().ravel() - ref).max() / scale)
    return {
        "value": round(prob.N / t_total, 1), "unit": "DOF/s", "cores": 1,
        "kind": "oracle",
        "sample": (f"the oracle's DD route: transfer blocks of double slabs {sample_ds} "
                   f"(sparse LU + {2 * prob.M} dense solves each), scaled x{prob.n_ds}/"
                   f"{len(sample_ds)}, + all loads + all slab reconstructions; the dense "
                   f"interface solve is left out (favours the CPU). SuperLU runs on one "
                   f"thread; BLAS threads {blas_threads}"),
        "seconds_extrapolated": round(t_total, 2),
        # the oracle's plain global sparse direct solve of the same problem
        # (its reference solution), timed in full on the same host
        "global_direct_s": round(t_direct, 2),
        "global_direct_dof_per_s": round(prob.N / t_direct, 1),
        "host": host_info(),
    }, errs


def host_info():
    """The host the CPU leg ran on: logical CPUs, the CPUs this process may
    use, and the processor model."""
    import subprocess
    model = None
    try:
        out = subprocess.run(["lscpu"], capture_output=True, text=True, timeout=10).stdout
        for line in out.splitlines():
            if line.startswith("Model name:"):
                model = line.split(":", 1)[1].strip()
    except Exception:  # noqa: BLE001 - informational only
        pass
    if model is None:
        try:
            for line in open("/proc/cpuinfo"):
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
        except OSError:
            pass
    try:
        allowed = len(os.sched_getaffinity(0))
    except AttributeError:
        allowed = None
    return {"nproc": os.cpu_count(), "cpus_allowed": allowed, "model": model}


def large_leg(dd, torch, name):
    """One end-to-end run of a large workload by two routes: the dense
    transfer blocks compressed as HODLR (the workload's definition), and the
    sampled construction without dense blocks compressed as HBS (the paper's
    Algorithm 1).  FP32 build, FP64 refinement to a predicted relative error
    of 1e-9; times from the host clock around the calls (inputs resident in
    HBM), the library's own phase times beside them.  Compressed factors in
    BF16 (the workloads' definition).  For the 2D oscillatory workload, whose
    near-resonant conditioning turns the BF16 factors' rounding into 5
    (HODLR) and 7 (HBS) refinement passes, each route is also solved again
    with the FP32 Krylov basis (the solve option basis_fp32: `fp32_basis`,
    timed as the route's set-up, compression and that solve) and compressed
    again with FP32 factors and solved (4 passes, FP64 basis: `fp32_factors`,
    timed as the route's set-up plus that compression and solve)."""
    from problems import make_config
    p = make_config(name)
    t = lambda a: None if a is None else torch.tensor(a, dtype=torch.float64, device="cuda")
    kap, c, f = t(p.kappa), t(p.c), t(p.f)
    F_build = p.n_ds * (2 * p.m - 1) * (14.0 / 3.0) * float(p.M) ** 3
    M3, steps = float(p.M) ** 3, p.m - 1
    # algorithmic work of each route's build: Gauss-Jordan inverses 2 M^3,
    # or M^3 by the symmetric elimination (lower triangle only) when the
    # operator has no convection (left-to-right sweeps of every slab,
    # right-to-left sweeps of the interior ones, the interface blocks),
    # transfer chains 2 M^3 per step of the interior slabs' two sweeps and
    # the blocks S = Sigma^{-1} R (dense route) or the sampling chains
    # 2 M^2 s per step of four chains per interior slab plus the final and W
    # products (sampled route)
    n_inv = (p.n_slabs + p.n_ds) * steps + p.n_ds
    chain = (2 * (p.n_slabs - 2) * steps + 2 * (p.n_ds - 1)) * 2.0 * M3
    flops = {}
    out = {"workload": f"{p.dim}D {name} {p.n}^{p.dim}, {p.n_slabs} slabs, M={p.M}, N_ds={p.n_ds}",
           "N": p.N, "s_build_nominal_flops": F_build}
    opts = dd.SolveOptions(tol=1e-9, max_iter=3000, max_outer=12)
    fdt = "bf16"
    out["factor_dtype"] = fdt
    for route in ("dense_hodlr", "sampled_hbs"):
        print(f"[bench] {name} route {route}", file=sys.stderr, flush=True)
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        t0 = time.perf_counter()
        op = dd.Operator(p.dim, p.n, p.n_slabs, kappa=kap, bvec=p.bvec, c=c, precision="fp32",
                         transfer_blocks=(route == "dense_hodlr"))
        torch.cuda.synchronize()
        t_setup = time.perf_counter() - t0
        sym = bool(op.build_stats()["symmetric"])
        inv = n_inv * (1.0 if sym else 2.0) * M3
        if route == "dense_hodlr":
            # symmetric: the chains of one direction serve both
            flops[route] = inv + chain - ((p.n_slabs - 2) * steps * 2.0 * M3 if sym else 0.0)
            info = op.compress(tol=1e-8 if p.dim == 2 else 1e-7, leaf=128, oversample=10,
                               max_rank=118, factor_dtype=fdt)
            o = dataclasses_replace(opts, use_hodlr=True)
        else:
            k = 32 if p.dim == 2 else 64
            info = op.compress_hbs(rank=k, oversample=10, factor_dtype=fdt, seed=11)
            o = dataclasses_replace(opts, use_hbs=True)
            smp = (4 * (p.n_slabs - 2) * steps + 2 * (p.n_ds - 1) + p.n_ds) * 2.0 * p.M ** 2 * (
                3 * k + 10)
            flops["sampled_hbs"] = inv + smp
        torch.cuda.synchronize()
        held = (free0 - torch.cuda.mem_get_info()[0]) / 1e9
        u, _, st = op.solve(f, opts=o, want_gamma=False, allow_notconv=True)
        torch.cuda.synchronize()
        total = time.perf_counter() - t0
        bs = op.build_stats()
        del u
        v32 = vb32 = None
        if p.dim == 2:
            # the same form, FP32 Krylov basis
            ob = dataclasses_replace(o, basis_fp32=True)
            ub, _, sb = op.solve(f, opts=ob, want_gamma=False, allow_notconv=True)
            torch.cuda.synchronize()
            del ub
            tb = total - st["t_solve_ms"] / 1e3 + sb["t_solve_ms"] / 1e3
            vb32 = {"total_s": round(tb, 3), "dof_per_s": round(p.N / tb, 1),
                    "solve_ms": round(sb["t_solve_ms"], 1), "outer_iters": sb["outer_iters"],
                    "gmres_iters": sb["gmres_iters"], "fd_residual_rel": sb["residual_rel"],
                    "converged": bool(sb["status"] == 0)}
            # the same route with FP32 compressed factors
            t1 = time.perf_counter()
            if route == "dense_hodlr":
                i32 = op.compress(tol=1e-8, leaf=128, oversample=10, max_rank=118,
                                  factor_dtype="fp32")
            else:
                i32 = op.compress_hbs(rank=k, oversample=10, factor_dtype="fp32", seed=11)
            torch.cuda.synchronize()
            t_c = time.perf_counter() - t1
            u32, _, s32 = op.solve(f, opts=o, want_gamma=False, allow_notconv=True)
            torch.cuda.synchronize()
            t_s = time.perf_counter() - t1 - t_c
            del u32
            tot32 = t_setup + t_c + t_s
            v32 = {"total_s": round(tot32, 3), "dof_per_s": round(p.N / tot32, 1),
                   "compress_s": round(t_c, 3), "solve_ms": round(s32["t_solve_ms"], 1),
                   "outer_iters": s32["outer_iters"], "gmres_iters": s32["gmres_iters"],
                   "fd_residual_rel": s32["residual_rel"],
                   "converged": bool(s32["status"] == 0), "compressed_bytes": i32["bytes"]}
        op.close()
        bt = bs["t_build_ms"] / 1e3
        r = {"total_s": round(total, 3), "dof_per_s": round(p.N / total, 1),
             "build_ms": round(bs["t_build_ms"], 1),
             # the workload's nominal S-build work (forming S) over this
             # route's build time; the sampled route does less than that
             "s_build_tflops_nominal": round(F_build / bt / 1e12, 2),
             "build_flops": flops[route],
             "symmetric_elimination": sym,
             "build_tflops": round(flops[route] / bt / 1e12, 2)
             if route == "dense_hodlr" else None,
             "solve_ms": round(st["t_solve_ms"], 1), "outer_iters": st["outer_iters"],
             "gmres_iters": st["gmres_iters"], "fd_residual_rel": st["residual_rel"],
             "correction_rel": st["correction_rel"], "converged": bool(st["status"] == 0),
             "device_gb_held": round(held, 2),
             "bytes_dense_blocks": bs["bytes_transfer"], "bytes_factors": bs["bytes_factors"],
             "compressed_bytes": info["bytes"]}
        if route == "dense_hodlr":
            r.update({"compress_ms": round(info["ms"], 1), "ranks": [info["min_rank"],
                                                                     info["max_rank"]]})
        else:
            # sampling runs in ddst_compress_hbs: the build's work over the
            # build and sampling times together
            r.update({"sample_ms": round(info["sample_ms"], 1),
                      "compress_ms": round(info["compress_ms"], 1), "rank": info["rank"],
                      "build_tflops": round(flops[route] / (bt + info["sample_ms"] / 1e3) / 1e12,
                                            2)})
        if vb32 is not None:
            r["fp32_basis"] = vb32
        if v32 is not None:
            r["fp32_factors"] = v32
        out[route] = r
        torch.cuda.empty_cache()
    return out


def dataclasses_replace(o, **kw):
    import dataclasses
    return dataclasses.replace(o, **kw)


def matfree_leg(dd, torch, dev, prob, opts):
    """Dense transfer blocks vs the matrix-free form (the comparison of the
    paper's Section 5.1): device memory, set-up time, one product with S
    (host-timed C-ABI call, mean of 10) and one refined solve, FP32 factors."""
    full = dd.Operator(2, dev["n"], dev["n_slabs"], kappa=dev["kappa"], bvec=dev["bvec"],
                       precision="fp32")
    lite = dd.Operator(2, dev["n"], dev["n_slabs"], kappa=dev["kappa"], bvec=dev["bvec"],
                       precision="fp32", transfer_blocks=False)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(prob.n_ds * full.M, dtype=torch.float64, device="cuda", generator=g)

    def apply_ms(op, which):
        for _ in range(2):
            op.apply(x, which=which)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(10):
            op.apply(x, which=which)
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / 10 * 1e3

    a_dense, a_free = apply_ms(full, "dense"), apply_ms(lite, "matfree")
    _, _, sd = full.solve(dev["f"], opts=opts, want_gamma=False, allow_notconv=True)
    _, _, sm = lite.solve(dev["f"], opts=opts, want_gamma=False, allow_notconv=True)
    full.close()
    lite.close()
    return {"memory_gb": {"transfer_blocks": round(sd["bytes_transfer"] / 1e9, 3),
                          "slab_factors": round(sd["bytes_factors"] / 1e9, 3)},
            "setup_ms": {"dense": round(sd["t_build_ms"], 2), "matfree": round(sm["t_build_ms"], 2)},
            "apply_ms": {"dense": round(a_dense, 3), "matfree": round(a_free, 3)},
            "solve_ms": {"dense": round(sd["t_solve_ms"], 2), "matfree": round(sm["t_solve_ms"], 2)},
            "gmres_iters": {"dense": sd["gmres_iters"], "matfree": sm["gmres_iters"]},
            "converged": {"dense": bool(sd["status"] == 0), "matfree": bool(sm["status"] == 0)}}


def many_leg(dd, torch, dev, prob, opts, nrhs=8):
    """nrhs seeded N(0,1) loads on the benchmark operator solved together
    (ddst_solve_many) beside one solve of the first alone (library solve
    times, the solve's own HIP events)."""
    op = dd.Operator(2, dev["n"], dev["n_slabs"], kappa=dev["kappa"], bvec=dev["bvec"],
                     precision="fp32")
    g = torch.Generator(device="cuda").manual_seed(7)
    F = torch.randn(nrhs, prob.n, prob.n, dtype=torch.float64, device="cuda", generator=g)
    op.solve(F[0], opts=opts, want_gamma=False, allow_notconv=True)
    _, _, s1 = op.solve(F[0], opts=opts, want_gamma=False, allow_notconv=True)
    op.solve_many(F, opts=opts, allow_notconv=True)
    # the multi-vector products timed live (HIP events on their stream)
    dd.profile_enable(True, kinds=["gemv_many"])
    _, sm = op.solve_many(F, opts=opts, allow_notconv=True)
    n, ms, work = dd.profile_read()["gemv_many"]
    dd.profile_enable(False)
    op.close()
    gbs = work / (ms / 1e3) / 1e9 if ms > 0 else 0.0
    return {"nrhs": nrhs, "solve_ms_together": round(sm["t_solve_ms"], 2),
            "solve_ms_per_rhs": round(sm["t_solve_ms"] / nrhs, 2),
            "solve_ms_single": round(s1["t_solve_ms"], 2),
            "throughput_gain": round(s1["t_solve_ms"] * nrhs / sm["t_solve_ms"], 2),
            "gmres_iters": {"together": sm["gmres_iters"], "single": s1["gmres_iters"]},
            "converged": bool(sm["status"] == 0),
            # k_gemv_nv: matrix bytes (one read per group of 8 vectors; interface
            # products count one of their two blocks, so a lower bound) per launch
            "gemv_many": {"launches": n, "avg_launch_us": round(ms / max(n, 1) * 1e3, 2),
                          "matrix_bytes_per_launch": work / max(n, 1),
                          "achieved_gbs": round(gbs, 1),
                          "frac_hbm": round(gbs / PEAK["hbm_gbs"], 4)}}


def main():
    args = parse()
    if args.pmc_child:
        pmc_child()
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only: --gpus {args.gpus} is not supported "
              f"(the multi-GPU slab sharding is a design, not part of this build)",
              file=sys.stderr)
        sys.exit(2)
    if args.only_large:
        import torch
        from paper_2510_25991_amd import ddst as dd
        print(json.dumps({"oscillatory_2d_2047": large_leg(dd, torch, "cfg3"),
                          "var_kappa_3d_127": large_leg(dd, torch, "cfg4")}), flush=True)
        return
    # hardware counters first, in child processes, before this one uses the GPU
    pmc = None if args.no_pmc else pmc_measure(ROOT)
    import numpy as np
    import torch
    from problems import make_config
    from paper_2510_25991_amd import ddst as dd

    prob = make_config("cfg2", n=args.n, n_slabs=args.slabs)
    dev = {"n": prob.n, "n_slabs": prob.n_slabs, "bvec": prob.bvec,
           "kappa": torch.tensor(prob.kappa, dtype=torch.float64, device="cuda"),
           "f": torch.tensor(prob.f, dtype=torch.float64, device="cuda")}
    torch.cuda.synchronize()
    if args.copy_bytes > 0:
        src = torch.ones(args.copy_bytes // 4, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    opts = dd.SolveOptions(tol=1e-9, max_outer=6)
    M, m, nds = prob.M, prob.m, prob.n_ds
    F_build = nds * (2 * m - 1) * (14.0 / 3.0) * float(M) ** 3

    print(f"[bench] mixed path: {args.warmup} warmup + {args.steps} timed steps "
          f"(n={prob.n}, slabs={prob.n_slabs})", file=sys.stderr, flush=True)
    t_mix, st_mix, u_mix, prof_mix, mix = timed(dd, torch, dev, "fp32", opts, args.steps,
                                                args.warmup, True)
    tb = float(np.mean([s["t_build_ms"] for s in st_mix])) / 1e3
    ts = float(np.mean([s["t_solve_ms"] for s in st_mix])) / 1e3
    # every sweep's matrices at once: left-to-right of all slabs, right-to-left
    # of all but the first
    outer = outer_blocks(2 * prob.n_slabs - 1, M, not any(prob.bvec))
    kname, roof = roofline(prof_mix, "fp32", M, pmc, outer)
    out_fp64 = None
    u64 = None
    if not args.no_fp64:
        print("[bench] FP64 plain path", file=sys.stderr, flush=True)
        t64, st64, u64, prof64, _ = timed(dd, torch, dev, "fp64", opts,
                                          max(1, args.steps // 2), 1, True)
        tb64 = float(np.mean([s["t_build_ms"] for s in st64])) / 1e3
        _, roof64 = roofline(prof64, "fp64", M)
        out_fp64 = {"ms_per_step": round(t64 * 1e3, 2), "dof_per_s": round(prob.N / t64, 1),
                    "build_ms": round(tb64 * 1e3, 2),
                    "s_build_tflops": round(F_build / tb64 / 1e12, 3),
                    "outer_iters": st64[-1]["outer_iters"],
                    "gmres_iters": st64[-1]["gmres_iters"], "roofline": roof64,
                    "speedup_mixed_over_fp64": round(t64 / t_mix, 3)}
    adj = None
    if not args.no_adjoint:
        print("[bench] adjoint (factors recomputed)", file=sys.stderr, flush=True)
        from problems import sensor_nodes
        op = dd.Operator(2, prob.n, prob.n_slabs, kappa=dev["kappa"], bvec=prob.bvec,
                         precision="fp32")
        u, _, _ = op.solve(dev["f"], opts=opts, want_gamma=False, allow_notconv=True)
        op.release_factors()
        gbar = torch.zeros(prob.N, dtype=torch.float64, device="cuda")
        gbar[torch.tensor(sensor_nodes(2, prob.n, 256, seed=1003), device="cuda")] = 1.0
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        dk, sta = op.adjoint(u.reshape(-1), gbar, opts=opts, allow_notconv=True)
        torch.cuda.synchronize()
        adj = {"ms": round((time.perf_counter() - t0) * 1e3, 2),
               "outer_iters": sta["outer_iters"], "gmres_iters": sta["gmres_iters"],
               "converged": bool(sta["status"] == 0)}
        op.close()
    mfree = None
    if not args.no_matfree:
        print("[bench] matrix-free comparison", file=sys.stderr, flush=True)
        mfree = matfree_leg(dd, torch, dev, prob, opts)
    many = None
    if not args.no_many:
        print("[bench] many right-hand sides", file=sys.stderr, flush=True)
        many = many_leg(dd, torch, dev, prob, opts)
    large = None
    if not args.no_large:
        large = {"oscillatory_2d_2047": large_leg(dd, torch, "cfg3"),
                 "var_kappa_3d_127": large_leg(dd, torch, "cfg4")}
    cpu, errs = (None, {})
    if not args.no_cpu:
        print("[bench] CPU oracle leg", file=sys.stderr, flush=True)
        cpu, errs = cpu_leg(prob, u_mix, u64)
    result = {
        "metric": "DOF/s end-to-end + S-build TFLOP/s; mixed vs FP64 GPU at rel err <=1e-8",
        "value": round(prob.N / t_mix, 1),
        "unit": "DOF/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(t_mix * 1e3, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32 build / f64 refinement",
        "data": "synthetic",
        "config": {"workload": f"2D conv-diff FD {prob.n}^2, {prob.n_slabs} slabs of {m} cells, "
                               f"M={M}, N_ds={nds}, variable kappa, b=(10,0), dense S",
                   "N": prob.N, "n": prob.n, "n_slabs": prob.n_slabs, "M": M, "N_ds": nds},
        "build_ms": round(tb * 1e3, 2),
        "solve_ms": round(ts * 1e3, 2),
        "s_build_tflops": round(F_build / tb / 1e12, 3),
        "s_build_nominal_flops": F_build,
        "outer_iters": st_mix[-1]["outer_iters"],
        "gmres_iters": st_mix[-1]["gmres_iters"],
        "converged": bool(st_mix[-1]["status"] == 0),
        "correction_rel": st_mix[-1]["correction_rel"],
        "rel_err_vs_oracle": errs or None,
        "fp64_plain": out_fp64,
        "adjoint": adj,
        "matrix_free": mfree,
        "many_rhs": many,
        "large_workloads": large,
        # every class timed over one extra step (untimed)
        "kernel_profile_per_step": {k: {"launches": v[0], "ms": round(v[1], 3)}
                                    for k, v in mix.items()},
        "roofline": roof,
        "cpu_baseline": cpu,
    }
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
