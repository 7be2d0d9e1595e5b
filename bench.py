#!/usr/bin/env python3
"""Benchmark of the Brillouin-kernel overlap hot path on one MI355X.

Workload (the metric's configuration): a 32^3x64 lattice, links exp(0.7 i A) + 3 APE steps at
alpha 0.6 (seeded), the 12 spin-colour point sources at the origin, D_ov = rho (1 + gamma5 sign(H))
with the Kenney-Laub [16/16] partial fractions (16 shifts), rho = 1, per-shift CG tolerance 1e-12.

Step (the timed unit behind `value`) = one pass of the whole hot path over the 12 sources:
bri_build_links (U -> FP64 off-axis links, and the FP32 links of the inner solve) + one batched
mixed-precision ov_apply (FP64 multi-shift CG whose iterations switch to FP32 links and vectors
once the residual has fallen to where their rounding no longer reaches the tolerance; FP64 final
apply).

value        overlap applies (right-hand sides) per second of that step.  Gated: every source with
             a stored FP64 oracle output (tests/golden/overlap_32x32x32x64_point*.npz) must match
             it to 1e-10 of its norm (stored sites, norm, two projections), else value = 0.
extra        the same workload through the plain FP64 single-source path (the speedup's
             denominator) and the FP64 batched path, with the speedups; a 16^4 line.
roofline     dominant kernel family, the FP64 stencil bri_apply at 32^3x64 (1 RHS, default launch),
             timed live with HIP events on the stream it runs on: algorithmic bytes per launch
             (6144 B/site: the 40 stored links, spinor in and out) / average launch time, against
             the 8 TB/s HBM peak; `traffic` from the committed rocprofv3 counter summary while the
             kernel sources match it.  The FP32 stencil and the multi-RHS kernels (% of peak
             flops) are reported beside it.
cpu_baseline the FP64 CPU oracle (every shift solved on its own) on the host: its stencil timed on
             a 16^4 field (same per-site work), scaled to the 32^3x64 volume and to the CG
             iterations the oracle itself needed on this workload (stored with its outputs).

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu] [--extras]
       python bench.py --stencil-only [--stencil-rhs 12] [--stencil-cols 2,4]
                                                            (copy calibration + stencil launches, for counters)
       python bench.py --survey                             (tuned stencil and overlap timings, 3 lattices)
"""

from __future__ import annotations

import argparse
import glob
import hashlib
import json
import os
import subprocess
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0
FP64_PEAK_TFLOPS = 78.6
FP32_PEAK_TFLOPS = 157.3
L_BENCH = (32, 32, 32, 64)
NSRC = 12
KL_N = 16
RHO = 1.0
CG_TOL = 1e-12  # per-shift residual tolerance of the 16^4 extras and the NEXT-row tables
# the benchmark's stopping rule: the result bound sum_i omega_i |r_i| / (2 sqrt(sigma_i)) <= 1e-11
# |psi| bounds the error of D_ov psi by rho 1e-11 |psi|, 10x inside the 1e-10 result criterion
RESULT_TOL = 1e-11
GATE_TOL = 1e-10
LINK_EPS, APE_ALPHA, APE_STEPS = 0.7, 0.6, 3
LINK_SEED = 1701 + 4
L_SMALL = (16, 16, 16, 16)  # the 16^4 line: exp(0.5 i A) + 3 APE, Gaussian source
SMALL_EPS, SMALL_SEED, SMALL_SRC_SEED = 0.5, 1701 + 2, 726 + 2
MASS = 0.05  # bare quark mass of the massive solve (extras)
OUTER_TOL = 1e-10
LINK_SEED_16 = SMALL_SEED
SRC_SEED = SMALL_SRC_SEED
GOLDEN = os.path.join(ROOT, "tests", "golden")
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "stencil_f64_32x32x32x64_counters.txt")
FLOP_PER_SITE_RHS = 2 * 18648  # FMA count of the kernels per site and right-hand side, x2


def stencil_bytes_per_site(spinor_bytes_per_real: int, link_bytes_per_real: int, nrhs: int = 1) -> int:
    """Algorithmic bytes of one stencil apply per site: 24 reals in and 24 out per
    right-hand side, and the 40 stored 3x3 complex links (720 reals)."""
    return (24 + 24) * nrhs * spinor_bytes_per_real + 720 * link_bytes_per_real


STENCIL_SOURCES = ("common.hpp", "stencil.hpp", "stencil_core.hpp", "stencil_kernels.hpp", "stencil.hip",
                   "stencil_f64_bri.hip", "tune.hip")


def kernel_source_digest() -> str:
    """Hash of the sources that define the FP64 stencil kernel and its launch configuration."""
    h = hashlib.sha256()
    for name in STENCIL_SOURCES:
        with open(os.path.join(ROOT, "paper_1701_00726_amd", "csrc", name), "rb") as f:
            h.update(name.encode() + f.read())
    return h.hexdigest()[:16]


def measured_traffic():
    """HBM bytes per launch of the FP64 stencil at 32^3x64 from the committed counter summary
    (FETCH_SIZE and WRITE_SIZE, each scaled by its copy-kernel factor), or None when the kernel
    sources changed since the counters were taken."""
    if not os.path.exists(TRAFFIC_FILE):
        return None
    vals = {}
    with open(TRAFFIC_FILE) as f:
        for ln in f:
            if "=" in ln and not ln.startswith("#"):
                k, v = ln.split("=", 1)
                vals[k.strip()] = v.strip()
    if vals.get("kernel_src_sha") != kernel_source_digest():
        return None
    try:
        return float(vals["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def golden_cases(L):
    """Stored oracle outputs for lattice L: list of dicts (tests/golden/overlap_<L>_*.npz)."""
    tag = "x".join(str(v) for v in L)
    out = []
    for path in sorted(glob.glob(os.path.join(GOLDEN, f"overlap_{tag}_*.npz"))):
        d = np.load(path, allow_pickle=False)
        out.append({k: d[k] for k in d.files} | {"name": os.path.basename(path)})
    return out


def gate(torch, bri, synth, out, cases):
    """Compare columns of `out` (nsrc, 4, 3, V) with the stored oracle outputs of point sources:
    the worst of (stored sites, norm, projections) relative to the oracle norm, per case."""
    rows = []
    for g in cases:
        if str(g["source_kind"]) != "point":
            continue
        col = out[int(g["source_arg"])]
        ref_norm = float(g["norm"])
        sites = torch.from_numpy(g["sites"]).to(col.device)
        es = float(np.abs(col[:, :, sites].permute(2, 0, 1).cpu().numpy() - g["out_sites"]).max()) / ref_norm
        en = abs(float(torch.linalg.vector_norm(col)) - ref_norm) / ref_norm
        L = tuple(int(v) for v in g["L"])
        host = bri.spinor_to_host(col[None])[0].ravel()
        ep = max(abs(np.vdot(synth.gaussian_source(L, int(s))[0].ravel(), host) - p) / ref_norm
                 for s, p in zip(g["proj_seeds"], g["proj"]))
        rows.append({"case": g["name"], "source": int(g["source_arg"]), "err_sites": es, "err_norm": en,
                     "err_proj": float(ep), "pass": max(es, en, ep) <= GATE_TOL})
    return rows


def cpu_info():
    model, phys = None, set()
    try:
        with open("/proc/cpuinfo") as f:
            cur = {}
            for ln in f:
                if ":" in ln:
                    k, v = (t.strip() for t in ln.split(":", 1))
                    cur[k] = v
                    if k == "model name" and model is None:
                        model = v
                elif cur:
                    phys.add((cur.get("physical id"), cur.get("core id")))
                    cur = {}
            if cur:
                phys.add((cur.get("physical id"), cur.get("core id")))
    except OSError:
        pass
    return {"model": model, "physical_cores": len(phys) or None, "logical_cpus": os.cpu_count(),
            "affinity_cpus": len(os.sched_getaffinity(0))}


_ONE_CORE = r"""
import sys, time
sys.path.insert(0, sys.argv[1])
import oracle, synth
L = (8, 8, 8, 8)
W = oracle.links(L, synth.random_links(L, 0.5, 1))
b = synth.gaussian_source(L, 2)[0]
oracle.dirac(L, W, -1.0, b)
t0 = time.perf_counter(); n = 0
while time.perf_counter() - t0 < 2.0:
    oracle.dirac(L, W, -1.0, b); n += 1
print((time.perf_counter() - t0) / n / 4096, oracle.num_threads())
"""


def cpu_baseline(shift_iters_per_source, iters_note, budget_s):
    """The oracle's stencil timed on a 16^4 field (per-site cost identical at every volume: the
    same 81 terms), scaled to one 12-source overlap apply at 32^3x64 with the per-shift CG
    iterations the oracle needs there (each CG iteration = 2 stencils, plus 2 per restart and
    final residual check, plus the final X y)."""
    import oracle
    import synth

    V16, V32 = int(np.prod(L_SMALL)), int(np.prod(L_BENCH))
    U = synth.random_links(L_SMALL, SMALL_EPS, SMALL_SEED)
    t0 = time.perf_counter()
    Wo = oracle.links(L_SMALL, U)
    t_links = time.perf_counter() - t0
    b = synth.gaussian_source(L_SMALL, SMALL_SRC_SEED)[0]
    oracle.dirac(L_SMALL, Wo, -RHO, b)
    n, t0 = 0, time.perf_counter()
    while n < 3 or (time.perf_counter() - t0 < budget_s / 2 and n < 50):
        oracle.dirac(L_SMALL, Wo, -RHO, b)
        n += 1
    t_site = (time.perf_counter() - t0) / n / V16
    applies = [sum(2 * (int(i) + 2) for i in its) + 1 for its in shift_iters_per_source]
    per_src = float(np.mean(applies)) * V32 * t_site
    t_total = t_links / V16 * V32 + NSRC * per_src
    one = None
    try:
        r = subprocess.run([sys.executable, "-c", _ONE_CORE, ROOT], capture_output=True, text=True, timeout=120,
                           env=dict(os.environ, OMP_NUM_THREADS="1"))
        one = float(r.stdout.split()[0])
    except Exception:  # noqa: BLE001 - the one-core figure is informative only
        pass
    info = cpu_info()
    return {
        "value": NSRC / t_total,
        "unit": "overlap applies/s",
        "cores": oracle.num_threads(),
        "kind": "oracle",
        "sample": (
            f"oracle stencil (direct 81-term sum, stored 81 links per site) timed {n}x on a 16^4 field: "
            f"{t_site * 1e9:.0f} ns/site ({oracle.num_threads()} threads); oracle links {t_links:.2f} s at 16^4. "
            f"Scaled to 32^3x64 and to {np.mean(applies):.0f} stencil applies per source ({iters_note}; every "
            f"shift solved by its own CG): {per_src:.0f} s per source, {t_total:.0f} s for the 12 sources"
        ),
        "cpu": info,
        "one_thread_ns_per_site": None if one is None else one * 1e9,
        "one_thread_applies_per_s": None if one is None else NSRC / (t_links / V16 * V32 * oracle.num_threads() +
                                                                       NSRC * float(np.mean(applies)) * V32 * one),
    }


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--stencil-reps", type=int, default=50)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU-oracle baseline")
    ap.add_argument("--no-extra", action="store_true", help="skip the FP64 comparison paths and kernel extras")
    ap.add_argument("--extras", action="store_true",
                    help="also the 16^4 gradient, kernel and rational variants, massive solve, cascade and Sec. 7 tables")
    ap.add_argument("--tune", action="store_true", help="autotune the stencil launches before timing")
    ap.add_argument("--survey", action="store_true",
                    help="stencil (tuned, FP64/FP32/BF16-link, 1 and 12 RHS) and overlap timings at 16^4, 24^3x48, 32^3x64")
    ap.add_argument("--variants", action="store_true",
                    help="time the stencil kernel variants at 32^3x64 (FP64 / FP32 / bfloat16 links, 1 and 12 RHS)")
    ap.add_argument("--stencil-only", action="store_true", help="copy calibration + stencil launches only")
    ap.add_argument("--stencil-rhs", type=int, default=1,
                    help="with --stencil-only: also launch the multi-RHS kernel on this many RHS (FP64 and FP32)")
    ap.add_argument("--stencil-cols", type=str, default="",
                    help="with --stencil-only: also launch the FP64 1-RHS default kernel and traversal over each of "
                         "these numbers of columns (comma-separated), the columns of a tile back to back, to split "
                         "the 1-RHS traffic into its link and spinor parts")
    ap.add_argument("--inner", default="f32", choices=["f32", "bf16w"], help="inner precision of the timed path")
    ap.add_argument("--cpu-seconds", type=float, default=12.0, help="budget of the CPU-oracle sample")
    return ap.parse_args()


def survey(torch, bri, synth):
    """Tuned stencil and overlap timings at the three workload lattices (links
    exp(i eps A) + 3 APE(0.6) built on the device; one JSON line per lattice)."""
    cfgs = [((16, 16, 16, 16), 0.5, 1703), ((24, 24, 24, 48), 0.7, 1704), ((32, 32, 32, 64), 0.7, 1705)]
    name = {bri.F64: "f64", bri.F32: "f32", bri.F32_BF16W: "bf16w"}
    bps = {bri.F64: 8, bri.F32: 4, bri.F32_BF16W: 4}
    bpl = {bri.F64: 8, bri.F32: 4, bri.F32_BF16W: 2}
    for L, eps, seed in cfgs:
        V = int(np.prod(L))
        U = synth.smeared_links_torch(L, eps, seed, APE_ALPHA, APE_STEPS, device="cuda", chunk=1 << 18)
        U = U.permute(0, 2, 3, 1).contiguous()
        W = {p: bri.build_links(L, U, p) for p in (bri.F64, bri.F32, bri.F32_BF16W)}
        del U
        rec = {"lattice": list(L), "link_eps": eps}
        g = torch.randn((12, 4, 3, V), dtype=torch.complex128, device="cuda")
        for p in (bri.F64, bri.F32, bri.F32_BF16W):
            for nr in (1, 12):
                x = g[:nr].to(bri.spinor_dtype(p)).contiguous()
                best, us = bri.autotune(L, W[p], p, x, reps=3)
                key = f"stencil_{name[p]}_{nr}rhs"
                rec[key] = {"us": us, "GBps_alg": stencil_bytes_per_site(bps[p], bpl[p], nr) * V / us / 1e3,
                            "config": best.as_dict()}
                print(f"[survey] {L} {key} {us:.1f} us", file=sys.stderr, flush=True)
        b1 = bri.spinor_to_device(synth.gaussian_source(L, SRC_SEED), bri.F64)
        b12 = bri.spinor_to_device(synth.point_sources_12(L), bri.F64)
        # the last row keeps every (shift, source) solution in FP64 for the refinement: 16 x 12 columns,
        # 77 GB at 32^3x64, ~210 GB of HBM with the FP32 multi-shift and the link arrays
        for nm, inner, b in (("fp64_1src", bri.F64, b1), ("fp64_12src", bri.F64, b12), ("mixed_f32_1src", bri.F32, b1),
                             ("mixed_f32_12src", bri.F32, b12)):
            op = bri.OverlapOp(L, W[bri.F64], kl_n=KL_N, rho=RHO, tol=CG_TOL, max_iter=5000,
                               Wlo=None if inner == bri.F64 else W[inner], inner=inner, nrhs=b.shape[0])
            op.apply(b)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, st = op.apply(b)
            torch.cuda.synchronize()
            dt = time.perf_counter() - t0
            rec["overlap_" + nm] = {"ms_per_call": dt * 1e3, "applies_per_s": b.shape[0] / dt, "cg_iters": st.iters,
                                    "refine_passes": st.refine}
            print(f"[survey] {L} overlap {nm} {dt * 1e3:.1f} ms", file=sys.stderr, flush=True)
            del op
            torch.cuda.empty_cache()
        print(json.dumps(rec), flush=True)
        del W, g
        torch.cuda.empty_cache()


# the cascaded-preconditioning measurement: the 16^3x32 volume of the paper's timing table,
# links exp(0.5 iA) + 7 APE(0.6) steps, am = 0.03, rho = 1, exit |r|/|b| <= 1e-9
CASCADE_L = (16, 16, 16, 32)
CASCADE_MASS, CASCADE_TOL, CASCADE_APE = 0.03, 1e-9, 7
# rows: (Kenney-Laub order, name, preconditioner levels as (kl_n, tol, max_iter, ms_tol, precision),
# sources side by side); the first four are the paper's table, then the preconditioners in FP32
# (their accuracy does not reach the result) and the 12-source batch
CASCADE_ROWS = (
    (1, "none", (), 1),
    (1, "1-level", ((0, 0.03, 50, 0.0, 0),), 1),
    (4, "none", (), 1),
    (4, "2-level", ((1, 0.03, 30, 1e-4, 0), (0, 0.1, 30, 0.0, 0)), 1),
    (1, "1-level, FP32 level", ((0, 0.03, 50, 0.0, 1),), 1),
    (4, "2-level, FP32 levels", ((1, 0.03, 30, 1e-4, 1), (0, 0.1, 30, 0.0, 1)), 1),
    (1, "1-level, FP32 level, 12 sources", ((0, 0.03, 50, 0.0, 1),), 12),
    (4, "2-level, FP32 kernel level, 12 sources", ((1, 0.03, 30, 1e-4, 0), (0, 0.1, 30, 0.0, 1)), 12),
)


# the operator-quality comparison of Sec. 7: the f_{1,1} overlap (rho = 1) with Brillouin or Wilson
# kernel, 1 or 3 APE steps (alpha = 0.72, the paper's), c_SW = 0 or 1, on a 16^3x32 field
QUALITY_L = (16, 16, 16, 32)
QUALITY_APE_ALPHA = 0.72


def quality_table(dev):
    """Normality and Ginsparg-Wilson defects (mean over 4 Gaussian vectors) and the locality decay
    rate delta (mean over 2 point sources) for each kernel setting."""
    import torch

    import paper_1701_00726_amd as bri
    import synth
    from paper_1701_00726_amd import quality

    L = QUALITY_L
    V = int(np.prod(L))
    rows = []
    eta = bri.spinor_to_device(synth.gaussian_source(L, SRC_SEED + 40, nrhs=4), bri.F64, dev)
    for ape in (1, 3):
        U = synth.smeared_links_torch(L, SMALL_EPS, SMALL_SEED + 40, QUALITY_APE_ALPHA, ape, device=dev, chunk=1 << 18)
        U = U.permute(0, 2, 3, 1).contiguous()
        for csw in (0.0, 1.0):
            W = bri.build_links(L, U, bri.F64, csw=csw)
            for kname, kernel in (("brillouin", bri.KERNEL_BRILLOUIN), ("wilson", bri.KERNEL_WILSON)):
                op = bri.OverlapOp(L, W, kl_n=1, rho=1.0, tol=1e-12, max_iter=20000, kernel=kernel, nrhs=4)
                t0 = time.perf_counter()
                nd = quality.normality_defect(op, eta)
                gw = quality.gw_defect(op, eta)
                deltas = []
                for seed in (1, 2):
                    r, mag = quality.locality_profile(op, L, quality.point_source(L, seed, dev))
                    deltas.append(quality.decay_rate(r, mag, rmin=2.0, rmax=8.0))
                torch.cuda.synchronize()
                rows.append({"kernel": kname, "ape_steps": ape, "csw": csw, "normality": float(np.mean(nd)),
                             "gw_defect": float(np.mean(gw)), "locality_delta": float(np.mean(deltas)),
                             "seconds": time.perf_counter() - t0})
                del op
            del W
        del U
    return {"lattice": list(L), "operator": "f_{1,1} overlap, rho = 1", "ape_alpha": QUALITY_APE_ALPHA,
            "rows": rows}


def cascade_table(dev):
    """Outer BiCGstab iterations and seconds per right-hand side for f_{1,1} and f_{4,4}, without
    and with cascaded preconditioning (complete massive form), one Gaussian source."""
    import torch

    import paper_1701_00726_amd as bri
    import synth

    L = CASCADE_L
    U = synth.smeared_links_torch(L, SMALL_EPS, SMALL_SEED + 30, APE_ALPHA, CASCADE_APE, device=dev, chunk=1 << 18)
    U = U.permute(0, 2, 3, 1).contiguous()
    W = bri.build_links(L, U, bri.F64)
    W32 = bri.build_links(L, U, bri.F32)
    del U
    b1 = bri.spinor_to_device(synth.gaussian_source(L, SRC_SEED + 30), bri.F64, dev)
    b12 = bri.spinor_to_device(synth.point_sources_12(L), bri.F64, dev)
    rows, ref = [], {}
    for n, name, levels, nsrc in CASCADE_ROWS:
        b = b1 if nsrc == 1 else b12
        prec = [bri.Level(k, tol=t, max_iter=mi, ms_tol=ms, inner=ip) for k, t, mi, ms, ip in levels]
        op = bri.OverlapOp(L, W, kl_n=n, rho=RHO, tol=CG_TOL, max_iter=5000, Wlo=W32)
        op.solve(b, CASCADE_MASS, tol=1e-3, prec=prec)  # warm caches and workspace
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        x, st = op.solve(b, CASCADE_MASS, complete=True, tol=CASCADE_TOL, max_iter=2000, prec=prec)
        torch.cuda.synchronize()
        sec = (time.perf_counter() - t0) / nsrc
        row = {"f": f"{n},{n}", "precond": name, "n_iter": st.iters, "s_per_rhs": sec, "sources": nsrc,
               "level_iters": st.level_iters, "true_rel_resid": st.rel_resid}
        key = (n, nsrc)
        if key in ref:
            row["rel_diff_vs_first_row"] = float(torch.linalg.vector_norm(x - ref[key]) /
                                                 torch.linalg.vector_norm(ref[key]))
        else:
            ref[key] = x
        rows.append(row)
        del op
    return {"lattice": list(L), "mass": CASCADE_MASS, "tol": CASCADE_TOL, "ape_steps": CASCADE_APE, "rows": rows}




# (name, tile, col_z, nsplit, rpt, xcd, variant) of the launches compared by --variants
VARIANTS_1RHS = (  # name, tile, col_z, nsplit, rpt, xcd, variant, col_y
    ("standard 16x4 column traversal", (16, 4, 0, 0), 8, 4, 0, 1, 0, 0),
    ("t-streaming 32x8x1, chunks of 4", (32, 8, 1, 4), 0, 1, 0, 1, 1, 0),
    ("x-line 32x2, lexicographic", (32, 2, 1, 1), 0, 4, 0, 0, 2, 0),
    ("x-line 32x2, columns 8 rows x 4 z (FP64 default)", (32, 2, 1, 1), 4, 4, 0, 1, 2, 8),
    ("x-line 32x2, columns 16 rows x 4 z (FP32 default)", (32, 2, 1, 1), 4, 4, 0, 1, 2, 16),
    ("matrix cores (FP32 / bf16 links)", (16, 4, 1, 1), 2, 4, 1, 0, 3, 0),
)
VARIANTS_12RHS = (
    ("standard multi-RHS 16x4, 4 per thread", (16, 4, 0, 0), 8, 4, 4, 1, 0, 0),
    ("standard multi-RHS 32x2, 2 per thread, 1 row (FP64 default)", (32, 2, 1, 1), 4, 4, 2, 1, 0, 1),
    ("standard multi-RHS 32x2, 3 per thread, 2 rows (FP32 default)", (32, 2, 1, 1), 4, 4, 3, 1, 0, 2),
    ("x-line, 1 per thread, 2 rows (bf16-link default)", (32, 2, 1, 1), 4, 4, 0, 1, 2, 2),
    ("x-line, 1 per thread, 8 rows", (32, 2, 1, 1), 4, 4, 0, 1, 2, 8),
    ("x-line multi-RHS, 3 per thread, 2 rows", (32, 2, 1, 1), 4, 4, 3, 1, 2, 2),
    ("matrix cores, 4 per thread (FP32 / bf16 links)", (16, 4, 1, 1), 2, 4, 4, 0, 3, 0),
)


def variants(torch, bri, synth, dev):
    """HIP-event times of the stencil kernel variants on the 32^3x64 workload field (the same
    random input for every launch of a precision; each variant's output checked against the
    first), one JSON line per launch."""
    L = L_BENCH
    V = int(np.prod(L))
    U = synth.smeared_links_torch(L, LINK_EPS, LINK_SEED, APE_ALPHA, APE_STEPS, device=dev, chunk=1 << 18)
    U = U.permute(0, 2, 3, 1).contiguous()
    bpr = {bri.F64: (8, 8), bri.F32: (4, 4), bri.F32_BF16W: (4, 2)}
    for prec, pname in ((bri.F64, "f64"), (bri.F32, "f32"), (bri.F32_BF16W, "bf16w")):
        W = bri.build_links(L, U, prec)
        for nr, table in ((1, VARIANTS_1RHS), (NSRC, VARIANTS_12RHS)):
            x = torch.randn((nr, 4, 3, V), dtype=bri.spinor_dtype(prec), device=dev)
            ref = None
            for name, t, cz, ns, rpt, xcd, var, cy in table:
                if var == 3 and prec == bri.F64:
                    continue
                cfg = bri.StencilCfg(t[0], t[1], t[2], t[3], cz, ns, rpt, xcd, var, cy)
                us = bri.stencil_time(L, W, prec, x, cfg=cfg, reps=10 if nr == 1 else 3)
                bri.set_stencil_cfg(L, prec, nr, cfg)
                y = bri.apply(L, W, prec, -RHO, x)
                bri.set_stencil_cfg(L, prec, nr, None)
                if ref is None:
                    ref = y
                diff = float(torch.linalg.vector_norm(y - ref) / torch.linalg.vector_norm(ref))
                alg = stencil_bytes_per_site(*bpr[prec], nr) * V
                print(json.dumps({"prec": pname, "nrhs": nr, "variant": name, "us": us,
                                  "alg_GBps": alg / (us * 1e-6) / 1e9, "frac_hbm": alg / (us * 1e-6) / 1e9 / HBM_PEAK_GBPS,
                                  "TFLOPs": FLOP_PER_SITE_RHS * V * nr / (us * 1e-6) / 1e12, "rel_diff": diff,
                                  "config": cfg.as_dict()}), flush=True)
            del x, ref, y
        del W
        torch.cuda.empty_cache()


def small_line(torch, bri, synth, dev, timed):
    """The former headline: 16^4 FP64 overlap apply of one Gaussian source and of the 12 point
    sources (links exp(0.5 i A) + 3 APE), HIP-event timed."""
    L = L_SMALL
    U = bri.links_to_device(synth.smeared_links(L, SMALL_EPS, SMALL_SEED, APE_ALPHA, APE_STEPS), dev)
    W = bri.build_links(L, U, bri.F64)
    b = bri.spinor_to_device(synth.gaussian_source(L, SMALL_SRC_SEED), bri.F64, dev)
    op = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, tol=CG_TOL, max_iter=5000)
    o = torch.empty_like(b)
    _, st = op.apply(b, out=o)
    ms = timed(lambda: op.apply(b, out=o), 10)
    b12 = bri.spinor_to_device(synth.point_sources_12(L), bri.F64, dev)
    op12 = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, tol=CG_TOL, max_iter=5000, nrhs=12)
    o12 = torch.empty_like(b12)
    op12.apply(b12, out=o12)
    ms12 = timed(lambda: op12.apply(b12, out=o12), 3)
    return {"fp64_1src_applies_per_s": 1e3 / ms, "fp64_12src_applies_per_s": 12e3 / ms12,
            "cg_iterations": st.iters, "stencil_config": bri.get_stencil_cfg(L, bri.F64, 1).as_dict()}


def extras_16(torch, bri, synth, dev, timed, stencil_reps):
    """Gradient, Wilson kernel, relaxed stopping, upper diagonal, clover, massive solves, cascade and
    Sec. 7 quality tables on the 16^4 field (the NEXT rows and the differentiation growth)."""
    L = L_SMALL
    V = int(np.prod(L))
    U = bri.links_to_device(synth.smeared_links(L, SMALL_EPS, SMALL_SEED, APE_ALPHA, APE_STEPS), dev)
    W = bri.build_links(L, U, bri.F64)
    b = bri.spinor_to_device(synth.gaussian_source(L, SMALL_SRC_SEED), bri.F64, dev)
    op = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, tol=CG_TOL, max_iter=5000)
    ref64 = op.apply(b)[0].clone()
    ms_ov = timed(lambda: op.apply(b), 5)
    t_in, t_out = b.clone(), torch.empty_like(b)
    bri.apply(L, W, bri.F64, -RHO, t_in, out=t_out)
    us_st = timed(lambda: bri.apply(L, W, bri.F64, -RHO, t_in, out=t_out), stencil_reps) * 1e3
    ex = {}
    chi = bri.spinor_to_device(synth.gaussian_source(L, SMALL_SRC_SEED + 1), bri.F64, dev)
    op.grad(U, chi[0], b[0])
    ms_g = timed(lambda: op.grad(U, chi[0], b[0]), 2)
    ex["grad_fp64_1src"] = {"ms_per_call": ms_g, "ratio_to_apply": ms_g / ms_ov}
    for _ in range(3):
        bri.wilson_apply(L, W, bri.F64, -RHO, t_in, out=t_out)
    ms_w = timed(lambda: bri.wilson_apply(L, W, bri.F64, -RHO, t_in, out=t_out), stencil_reps)
    opw = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, tol=CG_TOL, max_iter=20000, kernel=bri.KERNEL_WILSON)
    _, stw = opw.apply(b)
    ms_ow = timed(lambda: opw.apply(b), 3)
    ex["wilson_kernel_fp64_1src"] = {"stencil_us": ms_w * 1e3, "stencil_GBps_alg": 960 * V / (ms_w * 1e-3) / 1e9,
                                     "overlap_applies_per_s": 1e3 / ms_ow, "cg_iterations": stw.iters,
                                     "brillouin_stencil_us": us_st}
    del opw
    opr = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, tol=CG_TOL, max_iter=5000, relax=True)
    orl, str_ = opr.apply(b)
    ms_r = timed(lambda: opr.apply(b), 5)
    ex["relaxed_fp64_1src"] = {"applies_per_s": 1e3 / ms_r, "cg_iterations": str_.iters,
                               "rel_diff_vs_strict": float(torch.linalg.vector_norm(orl - ref64) /
                                                           torch.linalg.vector_norm(ref64))}
    opu = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, tol=CG_TOL, max_iter=5000, kind=bri.KL_UPPER)
    ou, stu = opu.apply(b)
    ms_u = timed(lambda: opu.apply(b), 5)
    ex["upper_diagonal_fp64_1src"] = {"applies_per_s": 1e3 / ms_u, "cg_iterations": stu.iters,
                                      "rel_diff_vs_diagonal": float(torch.linalg.vector_norm(ou - ref64) /
                                                                    torch.linalg.vector_norm(ref64))}
    Wc = bri.build_links(L, U, bri.F64, csw=1.0)
    bri.apply(L, Wc, bri.F64, -RHO, t_in, out=t_out)
    ms_c = timed(lambda: bri.apply(L, Wc, bri.F64, -RHO, t_in, out=t_out), stencil_reps)
    opc = bri.OverlapOp(L, Wc, kl_n=KL_N, rho=RHO, tol=CG_TOL, max_iter=5000)
    _, stc = opc.apply(b)
    ms_oc = timed(lambda: opc.apply(b), 5)
    ex["clover_fp64_1src"] = {"csw": 1.0, "stencil_us": ms_c * 1e3, "stencil_GBps_alg": 7296 * V / (ms_c * 1e-3) / 1e9,
                              "overlap_applies_per_s": 1e3 / ms_oc, "cg_iterations": stc.iters}
    del Wc, opc
    _, sts = op.solve(b, MASS, complete=True, tol=OUTER_TOL)
    ms_s = timed(lambda: op.solve(b, MASS, complete=True, tol=OUTER_TOL), 1)
    ex["massive_solve_fp64_1src"] = {"mass": MASS, "outer_tol": OUTER_TOL, "outer_iters": sts.iters,
                                     "ov_applies": sts.applies, "ms_per_solve": ms_s,
                                     "ms_per_ov_apply": ms_s / sts.applies, "true_rel_resid": sts.rel_resid}
    # the low-precision phase and the result bound on this field (one Gaussian source; 12 point sources)
    W32 = bri.build_links(L, U, bri.F32)
    b12 = bri.spinor_to_device(synth.point_sources_12(L), bri.F64, dev)
    for name, kw in (("result_bound_fp64", dict(tol=RESULT_TOL, relax=bri.RELAX_BOUND)),
                     ("mixed_f32", dict(tol=CG_TOL, Wlo=W32, inner=bri.F32)),
                     ("mixed_f32_result_bound", dict(tol=RESULT_TOL, relax=bri.RELAX_BOUND, Wlo=W32, inner=bri.F32))):
        row = {}
        for nr, src in ((1, b), (12, b12)):
            opx = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, max_iter=5000, nrhs=nr, **kw)
            ox, stx = opx.apply(src)
            msx = timed(lambda: opx.apply(src), 3)
            row[f"{nr}src"] = {"applies_per_s": nr * 1e3 / msx, "cg_iterations": stx.iters,
                               "low_precision_iterations": stx.refine}
            if nr == 1:
                row["rel_diff_vs_fp64_1e-12"] = float(torch.linalg.vector_norm(ox - ref64) /
                                                      torch.linalg.vector_norm(ref64))
            del opx, ox
        ex[name] = row
    del W32, b12
    ex["cascaded_16x16x16x32"] = cascade_table(dev)
    ex["kernel_quality_16x16x16x32"] = quality_table(dev)
    return ex


def main():
    args = parse()
    if args.gpus != 1:
        print(
            "bench.py measures one GPU only: the library has no multi-GPU path "
            "(the work would shard by sources, or by domain decomposition of the lattice in t).",
            file=sys.stderr,
        )
        sys.exit(2)

    import torch

    import paper_1701_00726_amd as bri
    import synth

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)
    if args.survey:
        survey(torch, bri, synth)
        return
    if args.variants:
        variants(torch, bri, synth, torch.device("cuda:0"))
        return
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    stream = torch.cuda.current_stream()
    L = L_BENCH
    V = int(np.prod(L))
    inner = {"f32": bri.F32, "bf16w": bri.F32_BF16W}[args.inner]

    def timed(fn, reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(reps):
            fn()
        e1.record(stream)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps  # ms

    print(f"[bench] links {L} exp({LINK_EPS} i A) + {APE_STEPS} APE({APE_ALPHA}) on the device", file=sys.stderr,
          flush=True)
    U = synth.smeared_links_torch(L, LINK_EPS, LINK_SEED, APE_ALPHA, APE_STEPS, device=dev, chunk=1 << 18)
    U = U.permute(0, 2, 3, 1).contiguous()
    W = torch.empty((40, 3, 3, V), dtype=torch.complex128, device=dev)
    Wlo = torch.empty((40, 3, 3, V), dtype=bri.link_dtype(inner), device=dev)
    bri.build_links(L, U, bri.F64, out=W)
    bri.build_links(L, U, inner, out=Wlo)
    b12 = bri.spinor_to_device(synth.point_sources_12(L), bri.F64, dev)
    if args.tune:
        for p, Wp in ((bri.F64, W), (inner, Wlo)):
            x = b12[:1].to(bri.spinor_dtype(p)).contiguous()
            cfg, us = bri.autotune(L, Wp, p, x, reps=3)
            print(f"[bench] tuned stencil prec {p}: {us:.1f} us {cfg.as_dict()}", file=sys.stderr, flush=True)

    if args.stencil_only:
        # calibration copy of 1 GiB (beyond the 256 MB Infinity Cache), then the stencil
        a = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
        c = torch.empty_like(a)
        c.copy_(a)
        del a, c
        torch.cuda.synchronize()
        t_in = b12[:1].clone()
        t_out = torch.empty_like(t_in)
        for _ in range(args.stencil_reps):
            bri.apply(L, W, bri.F64, -RHO, t_in, out=t_out)
        torch.cuda.synchronize()
        rec = {"stencil_only": True, "lattice": list(L), "launches": args.stencil_reps, "copy_bytes": 1 << 30,
               "alg_bytes_per_launch": stencil_bytes_per_site(8, 8) * V, "kernel_src_sha": kernel_source_digest(),
               "config": bri.get_stencil_cfg(L, bri.F64, 1).as_dict()}
        for nc in [int(v) for v in args.stencil_cols.split(",") if v.strip()]:
            # the 1-RHS launch over nc columns: a tile's columns run in consecutive blocks, so the
            # columns after the first find the tile's links in L2 and add mostly spinor traffic
            one = bri.get_stencil_cfg(L, bri.F64, 1)
            if one.variant == bri.VARIANT_LIBRARY:  # not a launch that can be installed for nc columns
                rec[f"cols_{nc}"] = {"skipped": "the 1-RHS default of this lattice is the library's own"}
                continue
            xc = b12[:nc].clone()
            yc = torch.empty_like(xc)
            bri.set_stencil_cfg(L, bri.F64, nc, one)
            try:
                for _ in range(args.stencil_reps):
                    bri.apply(L, W, bri.F64, -RHO, xc, out=yc)
                torch.cuda.synchronize()
            finally:
                bri.set_stencil_cfg(L, bri.F64, nc, None)
            rec[f"cols_{nc}"] = {"launches": args.stencil_reps, "config": one.as_dict()}
            del xc, yc
        if args.stencil_rhs > 1:
            nr = args.stencil_rhs
            for prec, Wp, name in ((bri.F64, W, "f64"), (bri.F32, bri.build_links(L, U, bri.F32), "f32")):
                xm = torch.randn((nr, 4, 3, V), dtype=bri.spinor_dtype(prec), device=dev)
                ym = torch.empty_like(xm)
                bri.apply(L, Wp, prec, -RHO, xm, out=ym)
                ms = timed(lambda: bri.apply(L, Wp, prec, -RHO, xm, out=ym), 5)
                rec[f"mrhs_{name}_{nr}rhs"] = {"us": ms * 1e3, "config": bri.get_stencil_cfg(L, prec, nr).as_dict()}
                del xm, ym
        print(json.dumps(rec), flush=True)
        return

    cases = golden_cases(L)
    o12 = torch.empty_like(b12)
    stop = dict(tol=RESULT_TOL, relax=bri.RELAX_BOUND)
    opm = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, max_iter=5000, Wlo=Wlo, inner=inner, nrhs=NSRC, **stop)

    def step():
        bri.build_links(L, U, bri.F64, out=W)
        bri.round_links(L, W, inner, out=Wlo)
        _, st = opm.apply(b12, out=o12)
        return st

    for _ in range(args.warmup):
        st = step()
    torch.cuda.synchronize()
    print(f"[bench] warmup done, {st.iters} CG iterations ({st.refine} in low precision)", file=sys.stderr,
          flush=True)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    e0.record(stream)
    stats = []
    for _ in range(args.steps):
        stats.append(step())
    e1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms_step = e0.elapsed_time(e1) / args.steps
    print(f"[bench] {args.steps} steps, {ms_step:.1f} ms/step (host wall {wall:.2f} s)", file=sys.stderr, flush=True)
    gate_rows = gate(torch, bri, synth, o12, cases)
    gate_ok = bool(gate_rows) and all(r["pass"] for r in gate_rows)
    rate = NSRC / (ms_step / 1e3)
    print(f"[bench] gate against stored oracle outputs: {gate_rows}", file=sys.stderr, flush=True)
    last = stats[-1]
    opm = None  # its workspace (~200 GB at 32^3x64) goes before the comparison paths allocate theirs
    torch.cuda.empty_cache()

    # dominant kernel family: the FP64 stencil at 32^3x64, timed live on the stream it runs on
    t_in, t_out = b12[:1].clone(), torch.empty_like(b12[:1])
    for _ in range(3):
        bri.apply(L, W, bri.F64, -RHO, t_in, out=t_out)
    us_launch = timed(lambda: bri.apply(L, W, bri.F64, -RHO, t_in, out=t_out), args.stencil_reps) * 1e3
    alg_bytes = stencil_bytes_per_site(8, 8) * V
    achieved = alg_bytes / (us_launch * 1e-6) / 1e9
    traffic = measured_traffic()
    print(f"[bench] bri_apply FP64 {us_launch:.1f} us/launch, {achieved:.0f} GB/s", file=sys.stderr, flush=True)

    result = {
        "metric": "D_bri apply GB/s (% HBM peak); overlap applies/s at 1e-10, mixed vs FP64",
        "value": rate if gate_ok else 0.0,
        "unit": "overlap applies/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64+f32" if inner == bri.F32 else "f64+f32/bf16",
        "data": "synthetic",
        "config": {
            "workload": f"32^3x64, 12 spin-colour point sources x Kenney-Laub [16/16] (16 shifts), rho=1, "
            f"multi-shift stopped at the result bound {RESULT_TOL:g} (error of D_ov psi <= rho {RESULT_TOL:g} |psi|), "
            f"links exp(0.7iA) + 3 APE(0.6); mixed-precision batched ov_apply (FP64 multi-shift, "
            f"{args.inner} links and vectors once the residual allows, FP64 final apply); "
            f"step = bri_build_links (FP64) + bri_round_links ({args.inner}) + ov_apply over the 12 sources",
            "lattice": list(L),
            "kl_n": KL_N,
            "nrhs": NSRC,
            "inner": args.inner,
            "stopping": {"rule": "result bound", "tol": RESULT_TOL},
            "cg_iterations": int(last.iters),
            "low_precision_iterations": int(last.refine),
            "stencil_config": bri.get_stencil_cfg(L, bri.F64, 1).as_dict(),
        },
        "gate": {"tol": GATE_TOL, "checked": gate_rows, "pass": gate_ok, "applies_per_s_measured": rate},
        "roofline": {
            "bound": "hbm",
            "kernel": "bri_apply FP64 1-RHS at 32^3x64 (default launch: stencil_xline_kernel<LinkF64, 4, false, EPI_PLAIN>)",
            "achieved": achieved,
            "peak": HBM_PEAK_GBPS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBPS,
            "traffic": None if traffic is None else traffic / (us_launch * 1e-6) / 1e9,
            "traffic_bytes_per_launch": traffic,
            "traffic_ratio": None if traffic is None else traffic / alg_bytes,
            "us_per_launch": us_launch,
            "alg_bytes_per_launch": alg_bytes,
        },
    }

    if not args.no_extra:
        extra = {}
        # FP64 single source (the speedup's denominator) and the FP64 batch, same workload
        op1 = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, max_iter=5000, **stop)
        o1 = torch.empty_like(b12[:1])
        srcs = [b12[r:r + 1].contiguous() for r in (0, 7, 11)]
        op1.apply(srcs[0], out=o1)
        ms1 = timed(lambda: [op1.apply(s, out=o1) for s in srcs], 1) / len(srcs)
        _, st1 = op1.apply(srcs[0], out=o1)
        del op1, o1
        op64 = bri.OverlapOp(L, W, kl_n=KL_N, rho=RHO, max_iter=5000, nrhs=NSRC, **stop)
        o64 = torch.empty_like(b12)
        op64.apply(b12, out=o64)
        ms64 = timed(lambda: op64.apply(b12, out=o64), 2)
        gate64 = gate(torch, bri, synth, o64, cases)
        _, st64 = op64.apply(b12, out=o64)
        diff = float(torch.linalg.vector_norm(o12 - o64) / torch.linalg.vector_norm(o64))
        del op64, o64
        torch.cuda.empty_cache()
        r1 = 1e3 / ms1
        r64 = NSRC * 1e3 / ms64
        extra["fp64_1src"] = {"applies_per_s": r1, "ms_per_apply": ms1, "cg_iterations": st1.iters}
        extra["fp64_12src"] = {"applies_per_s": r64, "ms_per_call": ms64, "cg_iterations": st64.iters,
                               "gate": gate64}
        extra["mixed_12src"] = {"applies_per_s": rate, "ms_per_step": ms_step, "rel_diff_vs_fp64_batch": diff,
                                "shift_rel_resid_max": max(last.rel_resid)}
        extra["speedup_mixed_12src_vs_fp64_1src"] = rate / r1
        extra["speedup_mixed_12src_vs_fp64_12src"] = rate / r64
        extra["speedup_fp64_12src_vs_fp64_1src"] = r64 / r1
        # the FP32 stencil beside the FP64 roofline, and the multi-RHS kernels in flops
        W32 = Wlo if inner == bri.F32 else bri.build_links(L, U, bri.F32)
        x32 = t_in.to(torch.complex64)
        y32 = torch.empty_like(x32)
        bri.apply(L, W32, bri.F32, -RHO, x32, out=y32)
        us32 = timed(lambda: bri.apply(L, W32, bri.F32, -RHO, x32, out=y32), args.stencil_reps) * 1e3
        a32 = stencil_bytes_per_site(4, 4) * V
        extra["stencil_f32_1rhs"] = {"us_per_launch": us32, "achieved_GBps": a32 / (us32 * 1e-6) / 1e9,
                                     "frac": a32 / (us32 * 1e-6) / 1e9 / HBM_PEAK_GBPS,
                                     "config": bri.get_stencil_cfg(L, bri.F32, 1).as_dict()}
        for prec, Wp, name, peak in ((bri.F64, W, "f64", FP64_PEAK_TFLOPS), (bri.F32, W32, "f32", FP32_PEAK_TFLOPS)):
            xm = b12.to(bri.spinor_dtype(prec))
            ym = torch.empty_like(xm)
            bri.apply(L, Wp, prec, -RHO, xm, out=ym)
            us = timed(lambda: bri.apply(L, Wp, prec, -RHO, xm, out=ym), 5) * 1e3
            tf = FLOP_PER_SITE_RHS * V * NSRC / (us * 1e-6) / 1e12
            extra[f"stencil_{name}_12rhs"] = {"us_per_launch": us, "TFLOPs": tf, "peak_TFLOPs": peak,
                                              "frac_of_peak": tf / peak,
                                              "config": bri.get_stencil_cfg(L, prec, NSRC).as_dict()}
            del xm, ym
        del W32, x32, y32
        torch.cuda.empty_cache()
        extra["16x16x16x16"] = small_line(torch, bri, synth, dev, timed)
        if args.extras:
            extra.update(extras_16(torch, bri, synth, dev, timed, args.stencil_reps))
        result["extra"] = extra
        print(f"[bench] extra: {json.dumps(extra)}", file=sys.stderr, flush=True)

    if not args.no_cpu:
        print("[bench] CPU oracle sample ...", file=sys.stderr, flush=True)
        its = [c["shift_iters"] for c in cases if str(c["source_kind"]) == "point"]
        note = "per-shift CG iterations of the oracle's own runs on this field"
        if not its:
            its = [last.shift_iters]
            note = "per-shift iterations of the GPU multi-shift on this field (no stored oracle run)"
        result["cpu_baseline"] = cpu_baseline(its, note, args.cpu_seconds)
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
