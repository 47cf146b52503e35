"""Benchmark of the REXII shifted-solve path on one MI355X.

One step = one complete u = exp(tA) f (all poles: coefficients, every shifted
solve, the weighted FP64 sum, reconstruction) for the 512 x 512 linear
rotating shallow-water workload: centred differences, g = H = 1, f_c = 10,
t rho = 1000, initial height a sum of 16 seeded Gaussian bumps, zero initial
velocity; FP32 inner Krylov iterations with FP64 residuals, refinement,
weights and pole sum (tol 1e-6).  Inputs are resident in HBM before the
timed region, and the timed steps run the library's default path (each
batch of solver kernels replayed from a HIP graph).

Prints one JSON line (see the keys at the bottom).  Also reported:
  * roofline of the dominant kernel (k_pass_f32: one COCG step or FP64
    residual round of every live solve) from one more apply with per-launch
    HIP events on the stream it runs on (the library's private stream),
  * the all-FP64 path on the same workload (timed steps, and k_pass_f64's
    roofline from a profiled apply),
  * the 2048^2 depth field at t rho = 100 (8 states in one batched call,
    mixed precision): k_bcg_u1_f32 and the whole BiCGStab step,
  * the adjoint workload (256^2, t rho = 500, FP64): forward and adjoint
    against the plain FP64 forward, gradients against stored oracle values,
  * for comparison, the shared-Krylov (multi-shift) and Fourier-space paths
    on the 512^2 workload (FP64, tol 1e-10),
  * the CPU oracle's per-mode REXII on a bounded sample of poles, on every
    host core (one process per core), and its exact exponential.
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "grid-pt·pole solves/s + HBM GB/s at rel-L2 ≤1e-6 vs FP64 oracle"
HBM_PEAK_GBS = 8000.0
FP32_PEAK_TFLOPS = 157.3
# COCG inner step, real flops per complex point: (L - zeta) p 20, the updates
# of d, r and p 24, four bilinear sums and |r|^2 36
COCG_FLOPS_PER_POINT = 80
D = 512
TRHO = 1000.0
FC = 10.0
NBUMPS = 16
SEED = 2


def workload():
    from paper_2008_11607_amd import inputs
    from paper_2008_11607_amd import rexii
    f = inputs.gaussian_bumps(D, nbumps=NBUMPS, seed=SEED)
    rho = rexii.rho(D, D, fc=FC)
    return f, rho, TRHO / rho


# HBM bytes per launch from two rocprofv3 counter runs (FETCH_SIZE x 2.0000,
# WRITE_SIZE x 1.0000, scales from a 1 GiB copy): k_pass_f32 and k_pass_f64
# on the 512^2 workload (128 slots), k_bcg_u1_f32 on the 2048^2 depth-field
# workload (one state, 8 slots); valid only for the kernel sources they were
# taken on.
TRAFFIC = {
    "k_pass_f32": {"bytes_per_launch": 1552237728.5, "fetch_kib": 390436.601, "write_kib": 734983.956,
                   "measured_on": "512^2 t rho 1000 mixed, 128 slots",
                   "sources": ["kernels.hip", "kernels.h", "device_util.h"],
                   "sources_sha256": "170d6851ff9acd7b82b98d1b0135ddb85c09c932c9da36aee58af692ed2a2bef"},
    "k_pass_f64": {"bytes_per_launch": 2619046913.6, "fetch_kib": 661923.708, "write_kib": 1233815.586,
                   "measured_on": "512^2 t rho 1000 fp64, 128 slots",
                   "sources": ["kernels.hip", "kernels.h", "device_util.h"],
                   "sources_sha256": "170d6851ff9acd7b82b98d1b0135ddb85c09c932c9da36aee58af692ed2a2bef"},
    # the Fourier path's pole-sum kernel: not measured (it is bound by FP64
    # arithmetic and writes 16 bytes per distinct frequency)
    "k_mode_coef": {"bytes_per_launch": None, "sources": ["kernels_fft.hip", "kernels_fft.h"], "sources_sha256": None},
    "k_bcg_u1_f32": {"bytes_per_launch": 1426113288.6, "fetch_kib": 430385.906, "write_kib": 531916.946,
                     "measured_on": "2048^2 depth field t rho 100 mixed, one state, 8 slots",
                     "sources": ["kernels_vh.hip", "kernels.h", "device_util.h"],
                     "sources_sha256": "d46707395c2f3676effb17af1cba10fed044ea5ba51a41c2337c352943362c56"},
}


def sources_sha256(files):
    import hashlib
    h = hashlib.sha256()
    for f in files:
        with open(os.path.join(ROOT, "paper_2008_11607_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def traffic_if_current(kernel, size=None):
    """The counter-based traffic of a kernel (at one grid size where it was
    taken per size) when its sources are unchanged, else None."""
    t = TRAFFIC.get(kernel)
    if t is None or t["sources_sha256"] is None or sources_sha256(t["sources"]) != t["sources_sha256"]:
        return None
    b = t["bytes_per_launch"]
    return b.get(size) if isinstance(b, dict) else b


def golden(name):
    """Stored oracle values (tests/golden, written by the scripts there)."""
    with open(os.path.join(ROOT, "tests", "golden", name)) as fh:
        return json.load(fh)


def sampled_rel_l2(u, gold):
    """Relative L2 error of a [3, ny, nx] result over the stored sample points."""
    idx = np.asarray(gold["index"])
    ref = np.asarray(gold["value"])
    got = u.cpu().numpy().reshape(-1)[idx]
    return float(np.linalg.norm(got - ref) / np.linalg.norm(ref))


def w_energy(u, H, g=1.0):
    """g |eta|^2 + H (|u|^2 + |v|^2) summed over the grid (conserved by exp(tA))."""
    return float(g * np.sum(u[0] ** 2) + np.sum(H * (u[1] ** 2 + u[2] ** 2)))


def _cpu_worker(args):
    """One host core's share of the CPU baseline: the oracle's per-mode REXII
    on the poles [lo, hi) of the 512^2 workload's pole set, in chunks of 8,
    until the range or the time budget is used up.  Returns (poles, seconds)."""
    lo, hi, t, tol, budget_s = args
    from oracle import coeffs as oc
    from oracle import lrsw
    from oracle import rexii_modes as rm
    from paper_2008_11607_amd import inputs
    op = lrsw.LRSW(D, D, fc=FC)
    f = inputs.gaussian_bumps(D, nbumps=NBUMPS, seed=SEED)
    c = oc.api_coeffs(t, lrsw.rho(op), h=0.5, tol=tol)
    done, k = 0, lo
    t0 = time.perf_counter()
    while k < hi and time.perf_counter() - t0 < budget_s:
        sl = slice(k, min(hi, k + 8))
        rm.rexii_direct(op, f, t, c["z"][sl], c["w"][sl])
        done += sl.stop - sl.start
        k = sl.stop
    return done, time.perf_counter() - t0


def cpu_model():
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(budget_s=12.0, tol=1e-6):
    """The oracle's per-mode REXII (one batched 3x3 solve per pole over all D^2
    Fourier modes, numpy) on the 512^2 workload, one process per host core
    (at most 16), each on its own range of the pole set until the time
    budget is spent; plus one call of the oracle's exact exponential (per-mode
    closed form) of the same state.  Runs before the GPU is touched: the
    worker processes are started fresh (spawn) and use no GPU."""
    import multiprocessing as mp
    from oracle import coeffs as oc
    from oracle import expm_modes as em
    from oracle import lrsw
    from paper_2008_11607_amd import inputs
    op = lrsw.LRSW(D, D, fc=FC)
    rho = lrsw.rho(op)
    t = TRHO / rho
    f = inputs.gaussian_bumps(D, nbumps=NBUMPS, seed=SEED)
    t0 = time.perf_counter()
    em.expm_closed_real(op, f, t)
    t_exact = time.perf_counter() - t0
    P = len(oc.api_coeffs(t, rho, h=0.5, tol=tol)["z"])
    cores = max(1, min(16, len(os.sched_getaffinity(0))))
    bounds = np.linspace(0, P, cores + 1).round().astype(int)
    jobs = [(int(bounds[i]), int(bounds[i + 1]), t, tol, budget_s) for i in range(cores)]
    # one BLAS/OpenMP thread per worker process: the cores are used by the processes
    old_env = {k: os.environ.get(k) for k in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS")}
    for k in old_env:
        os.environ[k] = "1"
    try:
        with mp.get_context("spawn").Pool(cores) as pool:
            res = pool.map(_cpu_worker, jobs)
    finally:
        for k, v in old_env.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v
    done = sum(r[0] for r in res)
    el = max(r[1] for r in res)
    return {"value": done * D * D / el, "unit": "grid-pt·pole solves/s", "cores": cores, "kind": "oracle",
            "cpu_model": cpu_model(), "threads_per_process": 1,
            "sample": f"oracle per-mode REXII (exact 3x3 solve per pole and Fourier mode, numpy) on {done} of "
                      f"{P} poles of the same 512x512 workload, {cores} processes x {el:.1f} s; the oracle's "
                      f"exact exponential (per-mode closed form) of the same state takes {t_exact:.2f} s "
                      f"(one process)",
            "exact_exponential_s": t_exact, "poles_done": done, "of_P": P, "seconds": el}


def copy_calibration(nbytes=1 << 30, reps=8):
    """A copy of known size (nbytes read + nbytes written per launch): the
    per-dispatch FETCH_SIZE / WRITE_SIZE it reports scale the counters of
    the solver kernels to bytes."""
    import torch
    x = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
    y = torch.empty_like(x)
    for _ in range(reps):
        y.copy_(x)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_per_launch": nbytes, "launches": reps}), flush=True)


def run_varh2048(args):
    """2048 x 2048 flux-form variable depth H = 1 + 0.3 sin(2 pi x) cos(2 pi y),
    g = 1, f_c = 20, rho the guaranteed spectral bound.
    (a) full REXII sum at t rho = 100 for 8 seeded states (seeds 50..57, 16
        bumps each) in one batched call, mixed precision; state 50 against
        the oracle's stored Chebyshev-Bessel samples; plus the same state in
        FP64;
    (b) throughput at t rho = 5000 (P ~ 2e4 poles) on a stratified subset of
        the poles (both poles of n = 0, ..., N in even steps), per-pole
        tolerances as in the full sum; the full-sum time is extrapolated
        from it."""
    import torch
    from paper_2008_11607_amd import inputs, rexii
    D, FC = 2048, 20.0
    gold = golden("varh2048_trho100.json")
    Hf = inputs.variable_depth(D)
    Hd = torch.from_numpy(Hf).cuda()
    rho = rexii.rho(D, D, fc=FC, Hfield=Hd)
    seeds = list(range(50, 50 + args.rhs))
    fs = [torch.from_numpy(inputs.gaussian_bumps(D, nbumps=16, seed=sd)).cuda() for sd in seeds]
    t = 100.0 / rho
    opts = dict(fc=FC, Hfield=Hd, precision="mixed", tol=1e-6, profile=1, pole_batch=args.slots if args.slots > 0 else 0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    us, reps = rexii.apply_batched(fs, [t] * len(fs), **opts)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    u0 = us[0].cpu().numpy()
    err = sampled_rel_l2(us[0], gold)
    wE = w_energy(u0, Hf) / gold["w_energy_f"] - 1.0
    P = reps[0]["P"]
    k_l = reps[0]["kernel_launches"]
    k_ms = reps[0]["kernel_ms"]
    k_b = reps[0]["kernel_bytes"]
    step = reps[0]["step_ms"]
    u1_ms, u1_b = step[1], reps[0]["u1_bytes"]
    u1_gbs = (u1_b / k_l) / (u1_ms / k_l * 1e-3) / 1e9
    out = {"metric": METRIC, "value": len(fs) * D * D * P / el, "unit": "grid-pt·pole solves/s", "n_gpus": 1,
           "steps": 1, "warmup": 0, "ms_per_step": 1000 * el, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "f32+f64", "data": "synthetic",
           "config": {"workload": f"varh-fd-2048x2048-fc20-trho100-{len(fs)}rhs-batched", "D": D, "t_rho": 100.0,
                      "f_c": FC, "precision": "mixed (FP32 inner BiCGStab, FP64 residual/refinement/pole sum)",
                      "tol": 1e-6, "P": P, "rhs": len(fs), "slots": reps[0]["slots"]},
           "rel_l2_vs_oracle_samples": err, "w_energy_drift": wE,
           "krylov": {"total_iters": sum(r["total_iters"] for r in reps), "max_iters": max(r["max_iters"] for r in reps),
                      "not_converged": sum(r["not_converged"] for r in reps), "stagnated": sum(r["stagnated"] for r in reps)},
           "roofline": {"bound": "hbm", "kernel": "k_bcg_u1_f32", "achieved": u1_gbs, "peak": HBM_PEAK_GBS,
                        "unit": "GB/s", "frac": u1_gbs / HBM_PEAK_GBS, "traffic": traffic_if_current("k_bcg_u1_f32"),
                        "avg_launch_ms": u1_ms / k_l, "launches": k_l, "alg_bytes_per_launch": u1_b / k_l,
                        "kernel_time_share": u1_ms * 1e-3 / el},
           "iteration": {"kernels": "k_bcg_outer, k_bcg_u1, k_bcg_u2, k_bcg_scalars_u, k_bcg_s, k_bcg_scalars_s",
                         "achieved_gbs": (k_b / k_l) / (k_ms / k_l * 1e-3) / 1e9,
                         "frac": (k_b / k_l) / (k_ms / k_l * 1e-3) / 1e9 / HBM_PEAK_GBS,
                         "alg_bytes_per_step": k_b / k_l, "avg_step_ms": k_ms / k_l, "steps": k_l,
                         "ms_by_kernel": dict(zip(["outer", "u1", "u2", "scalars_u", "s", "scalars_s"],
                                                  [round(x, 1) for x in step])),
                         "time_share": k_ms * 1e-3 / el}}
    if not args.no_fp64:
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        u64, r64 = rexii.apply(fs[0], t, fc=FC, Hfield=Hd, precision="fp64", tol=1e-10)
        torch.cuda.synchronize()
        e64 = time.perf_counter() - t1
        u64n = u64.cpu().numpy()
        out["fp64"] = {"value": D * D * r64["P"] / e64, "ms": 1000 * e64, "P": r64["P"],
                       "rel_l2_vs_oracle_samples": sampled_rel_l2(u64, gold),
                       "mixed_vs_fp64_rel_l2": float(np.linalg.norm(u0 - u64n) / np.linalg.norm(u64n)),
                       "total_iters": r64["total_iters"]}
    if args.subset > 0:
        t5 = 5000.0 / rho
        beta, alpha, kap = rexii.coeffs(t5, rho, h=0.5, tol=1e-6)
        z = beta * t5
        Pf = len(z)
        ns = np.unique(np.linspace(0, Pf // 2 - 1, args.subset).round().astype(int))
        # per-pole tolerances of the full sum: tol / (P a_k), a_k = |w_k| / |h mu|
        # (|h mu| = sum |w| / kappa_sum), capped at 1e-2; the subset runs as
        # two shifted-solve calls (first and second pole of each term), each
        # at the tightest tolerance of its group
        wabs = np.abs(alpha) * t5
        hmu = wabs.sum() / kap
        eps = np.minimum(1e-6 / (Pf * wabs / hmu), 1e-2)
        e5, it5, mx5, nc5, st5, kb5, km5, kl5 = 0.0, 0, 0, 0, 0, 0.0, 0.0, 0
        for first in (0, 1):
            ks = np.array([2 * n + first for n in ns])
            torch.cuda.synchronize()
            t2 = time.perf_counter()
            _, rs = rexii.shifted_solve(fs[0], t5, z[ks], fc=FC, Hfield=Hd, precision="mixed",
                                        tol=float(eps[ks].min()), profile=1, max_iter=400000)
            torch.cuda.synchronize()
            e5 += time.perf_counter() - t2
            it5 += rs["total_iters"]
            mx5 = max(mx5, rs["max_iters"])
            nc5 += rs["not_converged"]
            st5 += rs["stagnated"]
            kb5 += rs["kernel_bytes"]
            km5 += rs["kernel_ms"]
            kl5 += rs["kernel_launches"]
        npol = 2 * len(ns)
        out["trho5000_subset"] = {
            "poles": int(npol), "of_P": Pf, "seconds": e5, "value": D * D * npol / e5,
            "extrapolated_full_sum_s": e5 * Pf / npol, "total_iters": it5,
            "max_iters": mx5, "not_converged": nc5, "stagnated": st5,
            "iteration_gbs": (kb5 / kl5) / (km5 / kl5 * 1e-3) / 1e9}
    print(json.dumps(out), flush=True)


def run_multishift(args):
    """Shared-Krylov (multi-shift) path, FP64 (tol 1e-10), on the 2048 x 2048
    flux-form depth field H = 1 + 0.3 sin(2 pi x) cos(2 pi y), g = 1,
    f_c = 20, rho the guaranteed spectral bound:
    (a) t rho = 100, one state (seed 50) against the oracle's stored
        Chebyshev-Bessel samples;
    (b) t rho = 5000, --rhs states (seeds 50, 51, ...) in one call: the full
        REXII sum of the large configuration; state 50 against stored
        Chebyshev-Bessel samples."""
    import torch
    from paper_2008_11607_amd import inputs, rexii
    D, FC = 2048, 20.0
    Hf = inputs.variable_depth(D)
    Hd = torch.from_numpy(Hf).cuda()
    rho = rexii.rho(D, D, fc=FC, Hfield=Hd)

    def case(trho, nst, gold_name):
        fd = torch.stack([torch.from_numpy(inputs.gaussian_bumps(D, nbumps=16, seed=50 + k)) for k in range(nst)]).cuda()
        t = trho / rho
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        u, rep = rexii.apply_multishift(fd, t, fc=FC, Hfield=Hd, tol=1e-10, profile=1)
        torch.cuda.synchronize()
        el = time.perf_counter() - t0
        gold = golden(gold_name) if os.path.exists(os.path.join(ROOT, "tests", "golden", gold_name)) else None
        if gold is not None:
            assert abs(gold["t"] - t) <= 1e-12 * t, "workload differs from the stored oracle values"
        beta, _, _ = rexii.coeffs(t, rho, h=0.5, tol=1e-10)
        m = rep["solves"]
        k_ms, k_b = rep["kernel_ms"], rep["kernel_bytes"]
        ach = (k_b / m) / (k_ms / m * 1e-3) / 1e9
        return {"t_rho": trho, "states": nst, "seconds": el, "P": rep["P"], "P_rule_rho_bound": len(beta),
                "krylov_dim": m, "pass2_steps": rep["total_iters"], "step_launches": rep["kernel_launches"],
                "alg_bytes": rep["alg_bytes"], "rho_T": rep["rho"], "rho_bound": rho,
                "value": nst * D * D * rep["P"] / el,
                "rel_l2_vs_oracle_samples": sampled_rel_l2(u[0], gold) if gold else None,
                "w_energy_drift": (w_energy(u[0].cpu().numpy(), Hf) / gold["w_energy_f"] - 1.0) if gold else None,
                "ms_pass1": rep["step_ms"][0], "ms_host_small": rep["step_ms"][1], "ms_pass2": rep["step_ms"][2],
                "tail": rep["max_rel_residual"],
                "roofline": {"bound": "hbm", "kernel": "pass 2 (k_lz_gather; k_lz_step for vectors that were not kept)", "achieved": ach, "peak": HBM_PEAK_GBS,
                             "unit": "GB/s", "frac": ach / HBM_PEAK_GBS, "traffic": None,
                             "avg_launch_ms": k_ms / m, "launches": m, "alg_bytes_per_launch": k_b / m,
                             "kernel_time_share": k_ms * 1e-3 / el}}

    cases = {float(x) for x in args.multishift_cases.split(",")}
    small = case(100.0, 1, "varh2048_trho100.json") if 100.0 in cases else None
    big = case(5000.0, args.rhs, "varh2048_trho5000.json") if 5000.0 in cases else small
    out = {"metric": METRIC, "value": big["value"], "unit": "grid-pt·pole solves/s", "n_gpus": 1, "steps": 1,
           "warmup": 0, "ms_per_step": 1000 * big["seconds"], "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "f64", "data": "synthetic",
           "config": {"workload": f"varh-fd-2048x2048-fc20-trho5000-{args.rhs}rhs-multishift", "D": D,
                      "t_rho": 5000.0, "f_c": FC, "method": "shared-Krylov (one W-skew Lanczos per state, two "
                      "passes), REXII sum on the tridiagonal", "tol": 1e-10, "P": big["P"], "rhs": args.rhs},
           "rel_l2_vs_oracle_samples": big["rel_l2_vs_oracle_samples"], "roofline": big["roofline"],
           "trho5000": big, "trho100": small}
    print(json.dumps(out), flush=True)


def _batch_vs_plain(spec, warm=True):
    """One batched call against one plain call per state (mixed precision):
    (states, sizes, work, seconds batched, seconds plain, max rel diff, not converged)."""
    import torch
    from paper_2008_11607_amd import inputs, rexii
    fs, ts, sizes = [], [], []
    for s_ in spec:
        f = inputs.gaussian_bumps(s_["D"], nbumps=16, seed=s_["seed"])
        fs.append(torch.from_numpy(f).cuda())
        ts.append(s_["trho"] / rexii.rho(s_["D"], s_["D"], fc=FC))
        sizes.append(s_["D"])
    opts = dict(fc=FC, precision="mixed", tol=1e-6)
    if warm:
        rexii.apply_batched(fs[:2], ts[:2], **opts)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    us, reps = rexii.apply_batched(fs, ts, **opts)
    torch.cuda.synchronize()
    eb = time.perf_counter() - t0
    t1 = time.perf_counter()
    plain = [rexii.apply(f, t, **opts)[0] for f, t in zip(fs, ts)]
    torch.cuda.synchronize()
    ep = time.perf_counter() - t1
    work = sum(n * n * r["P"] for n, r in zip(sizes, reps))
    diffs = [float(torch.linalg.norm(u - v) / torch.linalg.norm(v)) for u, v in zip(us, plain)]
    return fs, sizes, work, eb, ep, max(diffs), sum(r["not_converged"] for r in reps), reps[0]["slots"]


def run_batched(args):
    """Heterogeneous batch: 16 states (seeds 300..315) on grids drawn from
    {128, 256, 512}^2 and t rho from U[50, 500] (a reduced form of 64 states on
    up to 1024^2 with t rho up to 2000), mixed precision; one batched call
    against one call per state (the oracle parity of batched calls is in the
    tests).  Also 64 small states (128^2, t rho from U[50, 200], seeds
    400..463), where one state alone cannot fill the GPU."""
    from paper_2008_11607_amd import inputs
    spec = inputs.batched_instances(count=args.rhs if args.rhs > 8 else 16, seed0=300, sizes=(128, 256, 512),
                                    trho_range=(50.0, 500.0))
    fs, sizes, work, eb, ep, dmax, nc, slots = _batch_vs_plain(spec)
    small = inputs.batched_instances(count=64, seed0=400, sizes=(128,), trho_range=(50.0, 200.0))
    _, _, work_s, eb_s, ep_s, dmax_s, nc_s, slots_s = _batch_vs_plain(small, warm=False)
    full = _full_batch_other_paths(args)
    print(json.dumps({"metric": METRIC, "value": work / eb, "unit": "grid-pt·pole solves/s", "n_gpus": 1, "steps": 1,
                      "warmup": 1, "ms_per_step": 1000 * eb, "higher_is_better": True, "scaling": "weak",
                      "vs_baseline": None, "dtype": "f32+f64", "data": "synthetic",
                      "config": {"workload": f"lrsw-fd-batched-{len(fs)}-mixed-grids-128-512-trho50-500",
                                 "states": len(fs), "grids": sorted(set(sizes)),
                                 "precision": "mixed", "tol": 1e-6, "slots": slots},
                      "plain_calls_value": work / ep, "speedup_vs_plain_calls": ep / eb,
                      "max_rel_l2_batched_vs_plain": dmax, "not_converged": nc,
                      "small_states": {"workload": "64 states, 128^2, t rho U[50, 200]", "value": work_s / eb_s,
                                       "ms": 1000 * eb_s, "plain_calls_value": work_s / ep_s,
                                       "speedup_vs_plain_calls": ep_s / eb_s, "slots": slots_s,
                                       "max_rel_l2_batched_vs_plain": dmax_s, "not_converged": nc_s},
                      "full_batch_other_paths": full}), flush=True)


def run_fullbatch(args):
    """The full heterogeneous batch (64 states, seeds 500..563, grids from
    {128, 256, 512, 1024}^2, t rho from U[50, 2000]) through the slot engine
    in ONE batched call, mixed precision (tol 1e-6, per-solve iteration caps
    from the solves' Chebyshev estimates); every state compared with the
    Fourier-space path's FP64 result (tol 1e-10, itself held to the oracle's
    per-mode REXII in the tests).  With --plain, also one plain call per state
    (the same solves without batching; progress line after each)."""
    import torch
    from paper_2008_11607_amd import inputs, rexii
    spec = inputs.batched_instances(count=64, seed0=500)
    fs, ts = [], []
    for s_ in spec:
        fs.append(torch.from_numpy(inputs.gaussian_bumps(s_["D"], nbumps=16, seed=s_["seed"])).cuda())
        ts.append(s_["trho"] / rexii.rho(s_["D"], s_["D"], fc=FC))
    opts = dict(fc=FC, precision="mixed", tol=1e-6)
    print("fullbatch: one call, 64 states", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    us, reps = rexii.apply_batched(fs, ts, **opts)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    work = sum(f.shape[-1] * f.shape[-2] * r["P"] for f, r in zip(fs, reps))
    worst, worst_bound = 0.0, 0.0
    for f, t, u, r in zip(fs, ts, us, reps):
        ref, _ = rexii.apply_fourier(f, t, fc=FC, tol=1e-10)
        worst = max(worst, float(torch.linalg.norm(u - ref) / torch.linalg.norm(ref)))
        worst_bound = max(worst_bound, r["err_bound"])
    print(f"fullbatch: one call {el:.1f} s, worst rel-L2 {worst:.2e}", file=sys.stderr, flush=True)
    out = {"metric": METRIC, "value": work / el, "unit": "grid-pt·pole solves/s", "n_gpus": 1,
           "steps": 1, "warmup": 0, "ms_per_step": 1000 * el, "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None, "dtype": "f32+f64", "data": "synthetic",
           "config": {"workload": "lrsw-fd-batched-64-grids-128-1024-trho50-2000-mixed-one-call",
                      "states": len(fs), "calls": 1, "precision": "mixed", "tol": 1e-6,
                      "slots": reps[0]["slots"]},
           "max_rel_l2_vs_fourier_fp64": worst, "max_err_bound": worst_bound,
           "not_converged": sum(r["not_converged"] for r in reps), "retried_fp64": sum(r["retried"] for r in reps),
           "total_iters": sum(r["total_iters"] for r in reps), "max_iters": max(r["max_iters"] for r in reps)}
    if args.plain:
        ep, dmax = 0.0, 0.0
        for i, (f, t, u) in enumerate(zip(fs, ts, us)):
            torch.cuda.synchronize()
            t1 = time.perf_counter()
            v, _ = rexii.apply(f, t, **opts)
            torch.cuda.synchronize()
            ep += time.perf_counter() - t1
            dmax = max(dmax, float(torch.linalg.norm(u - v) / torch.linalg.norm(v)))
            print(f"fullbatch: plain call {i} done, {ep:.1f} s so far", file=sys.stderr, flush=True)
        out["plain_calls"] = {"seconds": ep, "value": work / ep, "speedup_of_one_call": ep / el,
                              "max_rel_l2_batched_vs_plain": dmax}
    print(json.dumps(out), flush=True)


def _full_batch_other_paths(args):
    """The full heterogeneous batch (64 states, seeds 500..563, grids from
    {128, 256, 512, 1024}^2, t rho from U[50, 2000]) through the Fourier-space
    and shared-Krylov paths (FP64, tol 1e-10), one call per state; the two
    paths' results are compared with each other (their oracle parity is in
    the tests)."""
    import torch
    from paper_2008_11607_amd import inputs, rexii
    spec = inputs.batched_instances(count=64, seed0=500)
    fs, ts = [], []
    for s_ in spec:
        fs.append(torch.from_numpy(inputs.gaussian_bumps(s_["D"], nbumps=16, seed=s_["seed"])).cuda())
        ts.append(s_["trho"] / rexii.rho(s_["D"], s_["D"], fc=FC))
    # warm every grid size (rocFFT builds its plans, and compiles kernels for
    # a size the first time it is used) and both code paths
    first = {}
    for f, t in zip(fs, ts):
        first.setdefault(f.shape[-1], (f, t))
    for f, t in first.values():
        rexii.apply_fourier(f, t, fc=FC, tol=1e-10)
    rexii.apply_multishift(fs[0], ts[0], fc=FC, tol=1e-10)
    out = {}
    res = {}
    for name, fn in (("fourier", rexii.apply_fourier), ("multishift", rexii.apply_multishift)):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        us, work = [], 0
        for f, t in zip(fs, ts):
            u, r = fn(f, t, fc=FC, tol=1e-10)
            us.append(u)
            work += f.shape[-1] * f.shape[-2] * r["P"]
        torch.cuda.synchronize()
        el = time.perf_counter() - t0
        res[name] = us
        out[name] = {"seconds": el, "value": work / el}
    out["max_rel_l2_fourier_vs_multishift"] = max(
        float(torch.linalg.norm(a - b) / torch.linalg.norm(b)) for a, b in zip(res["fourier"], res["multishift"]))
    out["workload"] = "64 states, grids from {128, 256, 512, 1024}^2, t rho U[50, 2000], one call per state"
    out["grids"] = sorted({s_["D"] for s_ in spec})
    return out


FP64_PEAK_TFLOPS = 78.6
# algorithmic FP64 flops of the pole-sum kernel k_mode_coef: per (term,
# distinct frequency) s = a + theta^2 (1), d = s^2 + b^2 (2), 1/d (1), the two
# accumulations (A s + B)/d (8)
FLOPS_PER_TERM = 12


def _fourier_case(D, fc, trho, nbumps, seed, gold_name, steps, warmup):
    import torch
    from paper_2008_11607_amd import inputs
    from paper_2008_11607_amd import rexii
    f = inputs.gaussian_bumps(D, nbumps=nbumps, seed=seed)
    rho = rexii.rho(D, D, fc=fc)
    t = trho / rho
    gold = golden(gold_name)
    assert abs(gold["t"] - t) <= 1e-12 * t, "workload differs from the stored oracle values"
    fd = torch.from_numpy(f).cuda()
    u = torch.empty_like(fd)
    opts = dict(fc=fc, tol=1e-10)
    ws = torch.empty(rexii.fourier_workspace_size(D, D, t, fc=fc, tol=1e-10), dtype=torch.uint8, device="cuda")
    for _ in range(warmup):
        rexii.apply_fourier(fd, t, out=u, workspace=ws, **opts)
    torch.cuda.synchronize()
    # timed: the plain calls (no events); then as many profiled calls (HIP
    # events around every stage) for the kernel roofline and the stage split
    t0 = time.perf_counter()
    for _ in range(steps):
        rexii.apply_fourier(fd, t, out=u, workspace=ws, **opts)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    reps = []
    for _ in range(steps):
        _, rep = rexii.apply_fourier(fd, t, out=u, workspace=ws, profile=1, **opts)
        reps.append(rep)
    torch.cuda.synchronize()
    P, nterm, nfreq = reps[0]["P"], reps[0]["solves"], reps[0]["total_iters"]
    nm = (D // 2 + 1) * D
    k_ms = sum(r["kernel_ms"] for r in reps) / steps
    flops = nfreq * nterm * FLOPS_PER_TERM
    achieved = flops / (k_ms * 1e-3) / 1e12
    step_ms = [sum(r["step_ms"][k] for r in reps) / steps for k in range(5)]
    roof = {"bound": "alu", "kernel": "k_mode_coef", "achieved": achieved, "peak": FP64_PEAK_TFLOPS,
            "unit": "TFLOP/s", "frac": achieved / FP64_PEAK_TFLOPS,
            "traffic": traffic_if_current("k_mode_coef", D),
            "avg_launch_ms": k_ms, "launches": steps, "alg_flops_per_launch": flops,
            "waves_per_block": reps[0]["slots"], "term_splits": reps[0]["tile_rows"]}
    if achieved > FP64_PEAK_TFLOPS:
        # the far terms are summed as polynomials here, the direct sums'
        # operations are not done; the largest kernel is the column pass,
        # which moves the spectrum in and out once
        k_ms = step_ms[3]
        cols = reps[0]["kernel_bytes"] / (k_ms * 1e-3) / 1e9
        roof = {"bound": "hbm", "kernel": "k_cols", "achieved": cols, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": cols / HBM_PEAK_GBS, "avg_launch_ms": k_ms, "launches": steps,
                "alg_bytes_per_launch": reps[0]["kernel_bytes"]}
    roof["measured_in"] = "profiled calls after the timed ones (same workload)"
    roof["kernel_time_share"] = k_ms * steps * 1e-3 / el
    return {"D": D, "t_rho": trho, "f_c": fc, "P": P, "terms": nterm, "distinct_frequencies": nfreq,
            "half_spectrum_modes": nm, "el": el, "ms": 1000.0 * el / steps,
            "value": D * D * P / (el / steps), "rel_l2_vs_oracle": sampled_rel_l2(u, gold),
            "roofline": roof,
            "ms_by_stage": {"rows_forward_eta": step_ms[0], "rows_forward_uv": step_ms[1], "pole_sums": step_ms[2],
                            "columns": step_ms[3], "rows_inverse": step_ms[4]},
            "hbm_gbs_alg": sum(r["alg_bytes"] for r in reps) / el / 1e9}


def run_fourier(args):
    """Fourier-space REXII (constant depth, FP64): the 512^2 t rho = 1000
    workload of the headline line, and a 2048^2 t rho = 5000 constant-depth
    workload (f_c = 20)."""
    steps = max(args.steps, 20)
    sizes = {int(x) for x in args.fourier_sizes.split(",")}
    if 512 not in sizes:
        # the 2048^2 case alone (for per-size counter runs): its own line
        big = _fourier_case(2048, 20.0, 5000.0, 16, 5, "lrsw2048_trho5000.json", max(args.steps, 5),
                            max(args.warmup, 1))
        print(json.dumps({"workload": "lrsw-fd-2048x2048-fc20-trho5000-16bumps-fourier", "value": big["value"],
                          "unit": "grid-pt·pole solves/s", "ms_per_step": big["ms"],
                          "rel_l2_vs_oracle": big["rel_l2_vs_oracle"], "roofline": big["roofline"],
                          "ms_by_stage": big["ms_by_stage"]}), flush=True)
        return
    cpu = None if args.no_cpu else cpu_baseline(tol=1e-10)   # before the GPU is touched
    c = _fourier_case(D, FC, TRHO, NBUMPS, SEED, "lrsw512_trho1000.json", steps, max(args.warmup, 3))
    big = None
    if 2048 in sizes:
        big = _fourier_case(2048, 20.0, 5000.0, 16, 5, "lrsw2048_trho5000.json", max(args.steps, 5),
                            max(args.warmup, 1))
    out = {
        "metric": METRIC, "value": c["value"], "unit": "grid-pt·pole solves/s", "n_gpus": 1,
        "steps": steps, "warmup": max(args.warmup, 3), "ms_per_step": c["ms"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "lrsw-fd-512x512-trho1000-16bumps-fourier", "D": D, "t_rho": TRHO, "f_c": FC,
                   "method": "Fourier-space REXII: real transforms, per-mode closed-form pole sum (FP64)",
                   "tol": 1e-10, "P": c["P"], "terms": c["terms"], "h": 0.5,
                   "distinct_frequencies": c["distinct_frequencies"], "half_spectrum_modes": c["half_spectrum_modes"]},
        "rel_l2_vs_oracle": c["rel_l2_vs_oracle"],
        "hbm_gbs_alg": c["hbm_gbs_alg"],
        "roofline": c["roofline"],
        "ms_by_stage": c["ms_by_stage"],
    }
    if big is not None:
        out["large"] = {k: big[k] for k in ("D", "t_rho", "f_c", "P", "terms", "distinct_frequencies", "ms", "value",
                                            "rel_l2_vs_oracle", "roofline", "ms_by_stage")}
        out["large"]["workload"] = "lrsw-fd-2048x2048-fc20-trho5000-16bumps-fourier"
    if cpu is not None:
        out["cpu_baseline"] = cpu
    print(json.dumps(out), flush=True)


# algorithmic FP64 flops per term and mode of k_circ_sums: x - z (2), |x - z|^2
# (3), the reciprocal (1), 1/(x - z) (2), w / (x - z) accumulated (8); REXIE
# accumulates a second weight set (8 more)
CIRC_FLOPS_PER_TERM = {"rexii": 16, "rexi": 16, "rexie": 24}


def _matrix_large(name, scheme, steps, warmup):
    """One large circulant workload (2^20 points, 8 vectors, t rho = 1000):
    timed calls, then profiled ones for the k_circ_sums roofline; the
    result against the oracle's stored samples of the exact exponential."""
    import numpy as np
    import torch
    from paper_2008_11607_amd import inputs, rexii
    g = golden("matrix_cases.json")[name]
    n, nrhs = g["n"], g["nrhs"]
    st = inputs.advection_stencil(n) if name == "advection" else inputs.schroedinger_stencil(n)
    f = torch.from_numpy(inputs.random_vectors(n, nrhs, g["seed"])).cuda()
    u = torch.empty(f.shape, dtype=torch.complex128, device="cuda")
    opts = dict(scheme=scheme, nu=1j * g["nu_im"], tol=1e-10, out=u)
    for _ in range(warmup):
        rexii.apply_circulant(f, g["t"], st, **opts)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        _, rep = rexii.apply_circulant(f, g["t"], st, **opts)
    torch.cuda.synchronize()
    el = (time.perf_counter() - t0) / steps
    assert abs(rep["rho"] - g["rho"]) <= 1e-9 * g["rho"], "workload differs from the stored oracle values"
    got = u.cpu().numpy().reshape(-1)[np.asarray(g["index"])]
    ref = np.asarray(g["re"]) + 1j * np.asarray(g["im"])
    if scheme != "rexie":
        ref = ref.real
    err = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    ks = []
    for _ in range(steps):
        _, r = rexii.apply_circulant(f, g["t"], st, profile=1, **opts)
        ks.append(r["step_ms"])
    stage = [sum(k[i] for k in ks) / steps for i in range(5)]
    flops = n * rep["P"] * CIRC_FLOPS_PER_TERM[scheme]
    ach = flops / (stage[2] * 1e-3) / 1e12
    return {"workload": f"circulant-{name}-n{n}-{nrhs}rhs-trho{int(g['t_rho'])}-{scheme}", "n": n, "nrhs": nrhs,
            "P": rep["P"], "M": rep["M"], "ms": 1000 * el, "value": n * nrhs * rep["P"] / el,
            "rel_l2_vs_oracle_samples": err,
            "roofline": {"bound": "alu", "kernel": "k_circ_sums", "achieved": ach, "peak": FP64_PEAK_TFLOPS,
                         "unit": "TFLOP/s", "frac": ach / FP64_PEAK_TFLOPS, "traffic": None,
                         "avg_launch_ms": stage[2], "alg_flops_per_launch": flops,
                         "waves_per_block": rep["slots"],
                         "measured_in": "profiled calls after the timed ones (same workload)"},
            "ms_by_stage": {"load": stage[0], "fft_forward": stage[1], "pole_sums": stage[2], "apply": stage[3],
                            "fft_inverse": stage[4]}}


def run_matrix(args):
    """The paper's matrix experiments (Sec. 3.2, Fig. matrixRexiExample) on
    the GPU through rexii_apply_circulant: the error of REXII and the
    original REXI on A_1 (70 points) for M from 20 to 400 at h = 0.5, and of
    REXIE on A_2 shifted by -2450 i, against the stored dense expm; then the
    throughput of the same path on 2^20-point circulant matrices (8 vectors,
    t rho = 1000), REXII on the advection matrix and REXIE on the shifted
    Schroedinger matrix."""
    import numpy as np
    import torch
    from paper_2008_11607_amd import inputs, rexii
    gd = golden("matrix_cases.json")
    n = gd["A1"]["n"]
    st1, st2 = inputs.advection_stencil(n), inputs.schroedinger_stencil(n)
    f1 = torch.from_numpy(inputs.matrix_case_vector(n)).cuda()
    f2 = torch.from_numpy(inputs.matrix_case_vector(n, start=-1.0, length=2.0)).cuda()
    e1 = np.asarray(gd["A1"]["re"])
    e2 = np.asarray(gd["A2"]["re"]) + 1j * np.asarray(gd["A2"]["im"])
    rexii.apply_circulant(f1, 1.0, st1, M=20)   # plans and warm-up
    torch.cuda.synchronize()
    sweep = []
    t0 = time.perf_counter()
    for M in list(range(20, 401, 10)):
        ur, _ = rexii.apply_circulant(f1, 1.0, st1, scheme="rexii", M=M, h=0.5)
        ui, _ = rexii.apply_circulant(f1, 1.0, st1, scheme="rexi", M=M, h=0.5)
        sweep.append((M, float(np.linalg.norm(ur.cpu().numpy().real - e1) / np.linalg.norm(e1)),
                      float(np.linalg.norm(ui.cpu().numpy().real - e1) / np.linalg.norm(e1))))
    rexie = []
    for M in list(range(4700, 5101, 50)):
        ue, _ = rexii.apply_circulant(f2, 1.0, st2, scheme="rexie", nu=-2450j, M=M, h=0.5)
        rexie.append((M, float(np.linalg.norm(ue.cpu().numpy() - e2) / np.linalg.norm(e2))))
    sweep_s = time.perf_counter() - t0
    steps, warm = max(args.steps, 10), max(args.warmup, 2)
    adv = _matrix_large("advection", "rexii", steps, warm)
    adv_rexi = _matrix_large("advection", "rexi", steps, warm)
    sch = _matrix_large("schroedinger", "rexie", steps, warm)
    print(json.dumps({
        "metric": METRIC, "value": adv["value"], "unit": "grid-pt·pole solves/s", "n_gpus": 1, "steps": steps,
        "warmup": warm, "ms_per_step": adv["ms"], "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f64", "data": "synthetic",
        "config": {"workload": adv["workload"], "method": "per-mode resolvents of a circulant matrix (rocFFT), FP64",
                   "P": adv["P"], "h": 0.5, "tol": 1e-10},
        "rel_l2_vs_oracle_samples": adv["rel_l2_vs_oracle_samples"], "roofline": adv["roofline"],
        "ms_by_stage": adv["ms_by_stage"], "rexi_same_matrix": adv_rexi, "rexie_schroedinger": sch,
        "figure_matrix_example": {
            "A1_h0.5_M_rexii_rexi": sweep, "A2_rexie_nu-2450i_M": rexie, "seconds": sweep_s,
            "rexii_bound_M": int(np.ceil(70.0 / 0.5)) + 11,
            "note": "relative L2 error against dense expm (stored); REXII drops to round-off once (M - 11) h "
                    "reaches rho(A_1), the original REXI stays far above it"}}), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-fp64", action="store_true", help="skip the all-FP64 and comparison runs")
    ap.add_argument("--no-varh", action="store_true", help="skip the 2048^2 depth-field leg")
    ap.add_argument("--no-adjoint", action="store_true", help="skip the adjoint leg")
    ap.add_argument("--slots", type=int, default=-1,
                    help="concurrent solves; -1 (default) autotunes on the first call and caches the choice")
    ap.add_argument("--workload", default="lrsw512",
                    choices=["lrsw512", "varh2048", "batched", "fourier", "multishift", "fullbatch", "matrix",
                             "precond"],
                    help="lrsw512 (default): the headline line; varh2048: 2048^2 variable depth; "
                         "batched: heterogeneous batch against plain calls; fourier: the Fourier-space "
                         "path (constant depth) on the 512^2 workload and a 2048^2 one; multishift: the "
                         "shared-Krylov path on the 2048^2 depth field at t rho = 100 and 5000; matrix: the "
                         "paper's matrix experiments and 2^20-point circulant matrices (REXII, REXI, REXIE); "
                         "precond: the 2048^2 depth field through the FFT-preconditioned solves")
    ap.add_argument("--rhs", type=int, default=8, help="states of the varh2048 / batched workloads")
    ap.add_argument("--subset", type=int, default=16,
                    help="varh2048: values of n in the t rho = 5000 pole subset (0 = skip)")
    ap.add_argument("--fourier-sizes", default="512,2048",
                    help="fourier workload: grid sizes to run (512: t rho = 1000, the headline line; "
                         "2048: t rho = 5000, f_c = 20)")
    ap.add_argument("--multishift-cases", default="100,5000",
                    help="multishift workload: t rho values to run (100: one state; 5000: --rhs states)")
    ap.add_argument("--plain", action="store_true",
                    help="fullbatch workload: also one plain call per state")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain 1 GiB device-to-device copy 8 times (reference for HBM counters)")
    args = ap.parse_args()
    if args.copy_calibration:
        copy_calibration()
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (got --gpus {args.gpus}); the pole-sharded multi-GPU "
              "form is described in the design notes and not implemented.", file=sys.stderr)
        sys.exit(2)

    if args.workload == "varh2048":
        run_varh2048(args)
        return
    if args.workload == "batched":
        run_batched(args)
        return
    if args.workload == "fourier":
        run_fourier(args)
        return
    if args.workload == "multishift":
        run_multishift(args)
        return
    if args.workload == "matrix":
        run_matrix(args)
        return
    if args.workload == "precond":
        run_precond(args)
        return
    if args.workload == "fullbatch":
        run_fullbatch(args)
        return

    cpu = None if args.no_cpu else cpu_baseline()   # before the GPU is touched
    import torch
    from paper_2008_11607_amd import rexii

    f, rho, t = workload()
    fd = torch.from_numpy(f).cuda()
    gold = golden("lrsw512_trho1000.json")
    assert abs(gold["t"] - t) <= 1e-12 * t, "workload differs from the stored oracle values"
    # pole_batch=-1: slot count autotuned on the first (warm-up) call, cached
    opts = dict(fc=FC, precision="mixed", tol=1e-6, pole_batch=args.slots)
    u = torch.empty_like(fd)
    for _ in range(max(1, args.warmup)):
        rexii.apply(fd, t, out=u, **opts)
    torch.cuda.synchronize()
    reps = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        _, rep = rexii.apply(fd, t, out=u, **opts)
        reps.append(rep)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    ms = 1000.0 * el / args.steps
    P = reps[0]["P"]
    value = D * D * P / (el / args.steps)
    err = sampled_rel_l2(u, gold)
    print(f"headline: {args.steps} steps, {ms:.1f} ms/step, rel-L2 {err:.2e}", file=sys.stderr, flush=True)

    def pass_roofline(precision, tol, peak):
        """One more apply with a HIP event pair around every launch of k_chip
        (on the library's stream), which holds the solves' vectors in
        registers and LDS: algorithmic flops of the inner steps / its time."""
        t1 = time.perf_counter()
        up, rp = rexii.apply(fd, t, fc=FC, precision=precision, tol=tol, pole_batch=args.slots, profile=1)
        torch.cuda.synchronize()
        ep = time.perf_counter() - t1
        k_l, k_ms = rp["kernel_launches"], rp["kernel_ms"]
        flops = rp["total_iters"] * D * D * COCG_FLOPS_PER_POINT
        ach = flops / (k_ms * 1e-3) / 1e12
        return up, rp, {"bound": "alu", "kernel": "k_chip", "achieved": ach, "peak": peak, "unit": "TFLOP/s",
                        "frac": ach / peak, "traffic": None,
                        "avg_launch_ms": k_ms / k_l, "launches": k_l, "alg_flops_per_launch": flops / k_l,
                        "hbm_gbs": rp["kernel_bytes"] / (k_ms * 1e-3) / 1e9,
                        "streaming_equivalent_gbs": rp["alg_bytes"] / (k_ms * 1e-3) / 1e9,
                        "kernel_time_share": k_ms * 1e-3 / ep, "profiled_apply_ms": 1000 * ep,
                        "measured_in": "a separate apply with per-launch HIP events (same workload)"}

    up, rp, roof = pass_roofline("mixed", 1e-6, FP32_PEAK_TFLOPS)
    out = {
        "metric": METRIC, "value": value, "unit": "grid-pt·pole solves/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32+f64", "data": "synthetic",
        "config": {"workload": "lrsw-fd-512x512-trho1000-16bumps", "D": D, "t_rho": TRHO, "f_c": FC,
                   "precision": "mixed (FP32 inner COCG, FP64 residual/refinement/pole sum)", "tol": 1e-6,
                   "P": P, "solves": reps[0]["solves"], "h": 0.5, "slots": reps[0]["slots"],
                   "path": "default (inner steps on the chip)"},
        "rel_l2_vs_oracle": err,
        "err_bound": reps[0]["err_bound"],
        "krylov": {"total_iters": reps[0]["total_iters"], "max_iters": reps[0]["max_iters"],
                   "max_refine": reps[0]["max_refine"], "kappa_sum": reps[0]["kappa_sum"],
                   "pole_tol": reps[0]["pole_tol"], "max_rel_residual": reps[0]["max_rel_residual"],
                   "retried_fp64": reps[0]["retried"], "iter_hist_log2": reps[0]["iter_hist"],
                   "seconds_solve": reps[0]["seconds_solve"], "seconds_total": reps[0]["seconds"]},
        "roofline": roof,
    }
    if not args.no_fp64:
        # the all-FP64 path on the same workload: the precision of the paper
        o64 = dict(fc=FC, precision="fp64", tol=1e-10, pole_batch=args.slots)
        rexii.apply(fd, t, out=u, **o64)   # tunes its own slot count
        torch.cuda.synchronize()
        n64 = max(1, min(3, args.steps))
        r64s = []
        t1 = time.perf_counter()
        for _ in range(n64):
            _, r64 = rexii.apply(fd, t, out=u, **o64)
            r64s.append(r64)
        torch.cuda.synchronize()
        e64 = (time.perf_counter() - t1) / n64
        e64rel = sampled_rel_l2(u, gold)
        _, _, roof64 = pass_roofline("fp64", 1e-10, FP64_PEAK_TFLOPS)
        out["fp64"] = {"value": D * D * r64s[0]["P"] / e64, "ms": 1000 * e64, "steps": n64, "P": r64s[0]["P"],
                       "rel_l2_vs_oracle": e64rel, "err_bound": r64s[0]["err_bound"],
                       "total_iters": r64s[0]["total_iters"], "max_iters": r64s[0]["max_iters"],
                       "roofline": roof64}
        print(f"fp64: {1000 * e64:.1f} ms/step, rel-L2 {e64rel:.2e}", file=sys.stderr, flush=True)
    if not args.no_fp64:
        # the same two Krylov runs with a wider pole spacing h = 1: half the
        # poles, each better separated from the spectrum; the approximation's
        # aliasing floor e^{4 pi h - 4 pi^2} is 2e-12 there, below both bars
        wide = {}
        for name, prec, tol in (("mixed", "mixed", 1e-6), ("fp64", "fp64", 1e-10)):
            ow = dict(fc=FC, precision=prec, tol=tol, pole_batch=args.slots, h=1.0)
            rexii.apply(fd, t, out=u, **ow)
            torch.cuda.synchronize()
            t1 = time.perf_counter()
            _, rw = rexii.apply(fd, t, out=u, **ow)
            torch.cuda.synchronize()
            ew = time.perf_counter() - t1
            wide[name] = {"ms": 1000 * ew, "P": rw["P"], "value": D * D * rw["P"] / ew, "tol": tol,
                          "rel_l2_vs_oracle": sampled_rel_l2(u, gold), "err_bound": rw["err_bound"],
                          "total_iters": rw["total_iters"], "kappa_sum": rw["kappa_sum"]}
        out["h1"] = wide
        print("h = 1 runs done", file=sys.stderr, flush=True)
    if not args.no_fp64:
        # the other two paths on the same workload, for comparison (FP64, tol 1e-10)
        rexii.apply_multishift(fd, t, fc=FC, tol=1e-10)   # warm
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        ums, rms = rexii.apply_multishift(fd, t, fc=FC, tol=1e-10)
        torch.cuda.synchronize()
        ems = time.perf_counter() - t2
        out["multishift"] = {"ms": 1000 * ems, "P": rms["P"], "krylov_dim": rms["solves"],
                             "value": D * D * rms["P"] / ems, "rel_l2_vs_oracle": sampled_rel_l2(ums, gold)}
        ws = torch.empty(rexii.fourier_workspace_size(D, D, t, fc=FC, tol=1e-10), dtype=torch.uint8, device="cuda")
        ufo = torch.empty_like(fd)
        for _ in range(3):
            rexii.apply_fourier(fd, t, fc=FC, tol=1e-10, out=ufo, workspace=ws)
        torch.cuda.synchronize()
        t3 = time.perf_counter()
        for _ in range(20):
            _, rfo = rexii.apply_fourier(fd, t, fc=FC, tol=1e-10, out=ufo, workspace=ws)
        torch.cuda.synchronize()
        efo = (time.perf_counter() - t3) / 20
        out["fourier"] = {"ms": 1000 * efo, "P": rfo["P"], "value": D * D * rfo["P"] / efo,
                          "rel_l2_vs_oracle": sampled_rel_l2(ufo, gold)}
    if not args.no_varh:
        out["depth_field_2048"] = varh2048_leg(rexii, torch)
        print("depth field 2048^2 done", file=sys.stderr, flush=True)
    if not args.no_varh:
        out["depth_field_2048_precond"] = precond_leg(rexii, torch)
        print("depth field 2048^2 (preconditioned) done", file=sys.stderr, flush=True)
    if not args.no_adjoint:
        out["adjoint_256"] = adjoint_leg(rexii, torch)
        print("adjoint 256^2 done", file=sys.stderr, flush=True)
    if cpu is not None:
        out["cpu_baseline"] = cpu
    print(json.dumps(out), flush=True)


def varh2048_leg(rexii, torch, nrhs=8):
    """2048^2 depth field H = 1 + 0.3 sin(2 pi x) cos(2 pi y), f_c = 20,
    t rho = 100, nrhs states (seeds 50..) in one batched call, mixed
    precision (tol 1e-6), per-launch HIP events: the BiCGStab kernels'
    roofline at the 2048^2 shape; state 50 against stored oracle samples."""
    from paper_2008_11607_amd import inputs
    D2, FC2 = 2048, 20.0
    gold = golden("varh2048_trho100.json")
    Hf = inputs.variable_depth(D2)
    Hd = torch.from_numpy(Hf).cuda()
    rho = rexii.rho(D2, D2, fc=FC2, Hfield=Hd)
    t = 100.0 / rho
    assert abs(gold["t"] - t) <= 1e-12 * t, "workload differs from the stored oracle values"
    fs = [torch.from_numpy(inputs.gaussian_bumps(D2, nbumps=16, seed=50 + k)).cuda() for k in range(nrhs)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    us, reps = rexii.apply_batched(fs, [t] * nrhs, fc=FC2, Hfield=Hd, precision="mixed", tol=1e-6, profile=1)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    r0 = reps[0]
    k_l, k_ms, k_b, step = r0["kernel_launches"], r0["kernel_ms"], r0["kernel_bytes"], r0["step_ms"]
    u1_ms, u1_b = step[1], r0["u1_bytes"]
    u1 = (u1_b / k_l) / (u1_ms / k_l * 1e-3) / 1e9
    it = (k_b / k_l) / (k_ms / k_l * 1e-3) / 1e9
    return {"workload": f"varh-fd-2048x2048-fc20-trho100-{nrhs}rhs-batched-mixed", "P": r0["P"], "states": nrhs,
            "seconds": el, "value": nrhs * D2 * D2 * r0["P"] / el,
            "rel_l2_vs_oracle_samples": sampled_rel_l2(us[0], gold),
            "err_bound_max": max(r["err_bound"] for r in reps),
            "total_iters": sum(r["total_iters"] for r in reps), "max_iters": max(r["max_iters"] for r in reps),
            "roofline": {"bound": "hbm", "kernel": "k_bcg_u1_f32", "achieved": u1, "peak": HBM_PEAK_GBS,
                         "unit": "GB/s", "frac": u1 / HBM_PEAK_GBS, "traffic": traffic_if_current("k_bcg_u1_f32"),
                         "avg_launch_ms": u1_ms / k_l, "launches": k_l, "alg_bytes_per_launch": u1_b / k_l,
                         "kernel_time_share": u1_ms * 1e-3 / el},
            "iteration": {"kernels": "k_bcg_outer, k_bcg_u1, k_bcg_u2, k_bcg_scalars_u, k_bcg_s, k_bcg_scalars_s",
                          "achieved_gbs": it, "frac": it / HBM_PEAK_GBS, "alg_bytes_per_step": k_b / k_l,
                          "avg_step_ms": k_ms / k_l, "steps": k_l,
                          "ms_by_kernel": dict(zip(["outer", "u1", "u2", "scalars_u", "s", "scalars_s"],
                                                   [round(x, 1) for x in step])),
                          "time_share": k_ms * 1e-3 / el}}


def precond_leg(rexii, torch, nrhs=8):
    """The 2048^2 depth-field workload (t rho = 100, states 50..) through the
    FFT-preconditioned solves (method 2, FP64, tol 1e-10), one batched call
    after a one-state warm-up (rocFFT builds its plans on first use); state
    50 against the stored oracle samples."""
    from paper_2008_11607_amd import inputs
    D2, FC2 = 2048, 20.0
    gold = golden("varh2048_trho100.json")
    Hd = torch.from_numpy(inputs.variable_depth(D2)).cuda()
    t = 100.0 / rexii.rho(D2, D2, fc=FC2, Hfield=Hd)
    assert abs(gold["t"] - t) <= 1e-12 * t, "workload differs from the stored oracle values"
    fs = [torch.from_numpy(inputs.gaussian_bumps(D2, nbumps=16, seed=50 + k)).cuda() for k in range(nrhs)]
    rexii.apply(fs[0], t, fc=FC2, Hfield=Hd, method="precond")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    us, reps = rexii.apply_batched(fs, [t] * nrhs, fc=FC2, Hfield=Hd, method="precond")
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    r0 = reps[0]
    return {"workload": f"varh-fd-2048x2048-fc20-trho100-{nrhs}rhs-precond-fp64", "P": r0["P"], "states": nrhs,
            "seconds": el, "value": nrhs * D2 * D2 * r0["P"] / el,
            "rel_l2_vs_oracle_samples": sampled_rel_l2(us[0], gold), "err_bound_max": max(r["err_bound"] for r in reps),
            "total_iters": sum(r["total_iters"] for r in reps), "max_iters": max(r["max_iters"] for r in reps),
            "slots": r0["slots"], "hbm_gbs_alg": sum(r["alg_bytes"] for r in reps) / el / 1e9,
            "method": "BiCGStab right-preconditioned by the FFT inverse of the mean-depth operator (FP64)"}


def run_precond(args):
    """The 2048^2 depth-field workload (t rho = 100, --rhs states) through the
    FFT-preconditioned solves (method 2, FP64) in one batched call, beside
    one state through the slot engine's BiCGStab (FP64) for comparison."""
    import torch
    from paper_2008_11607_amd import inputs, rexii
    leg = precond_leg(rexii, torch, nrhs=args.rhs)
    Hd = torch.from_numpy(inputs.variable_depth(2048)).cuda()
    t = 100.0 / rexii.rho(2048, 2048, fc=20.0, Hfield=Hd)
    f = torch.from_numpy(inputs.gaussian_bumps(2048, nbumps=16, seed=50)).cuda()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    _, rb = rexii.apply(f, t, fc=20.0, Hfield=Hd)
    torch.cuda.synchronize()
    eb = time.perf_counter() - t0
    print(json.dumps({"metric": METRIC, "value": leg["value"], "unit": "grid-pt·pole solves/s", "n_gpus": 1,
                      "steps": 1, "warmup": 1, "ms_per_step": 1000 * leg["seconds"], "higher_is_better": True,
                      "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
                      "config": {"workload": leg["workload"], "P": leg["P"], "states": leg["states"], "tol": 1e-10},
                      "precond": leg,
                      "slot_engine_fp64_one_state": {"seconds": eb, "total_iters": rb["total_iters"],
                                                     "value": 2048 * 2048 * rb["P"] / eb}}), flush=True)


def adjoint_leg(rexii, torch):
    """The gradient workload (256^2, t rho = 500, FP64, tol 1e-10): J =
    |P u - y|^2 with 1024 sampled eta points.  Times the plain FP64 forward
    apply and the adjoint call (dJ/df and dJ/dH together) and checks both
    gradients against the oracle's stored values."""
    from paper_2008_11607_amd import inputs
    g = golden("adjoint256_trho500.json")
    D4 = g["D"]
    rho = rexii.rho(D4, D4, fc=g["f_c"])
    t = g["t_rho"] / rho
    assert abs(g["t"] - t) <= 1e-12 * t, "workload differs from the stored oracle values"
    fd = torch.from_numpy(inputs.gaussian_bumps(D4, nbumps=g["nbumps"], seed=g["seed_f"])).cuda()
    idx = torch.tensor(g["sample_index"], dtype=torch.int64, device="cuda")
    y = torch.tensor(g["y"], dtype=torch.float64, device="cuda")
    opts = dict(fc=g["f_c"], precision="fp64", tol=1e-10)

    def forward_and_gbar():
        u, r = rexii.apply(fd, t, **opts)
        gbar = torch.zeros_like(u)
        gbar[0].view(-1)[idx] = 2.0 * (u[0].reshape(-1)[idx] - y)
        return u, r, gbar

    u, _, gbar = forward_and_gbar()   # warm
    rexii.apply_adjoint(fd, gbar, t, **opts)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    u, rf, gbar = forward_and_gbar()
    torch.cuda.synchronize()
    ef = time.perf_counter() - t0
    t1 = time.perf_counter()
    dJdf, dJdH, ra = rexii.apply_adjoint(fd, gbar, t, **opts)
    torch.cuda.synchronize()
    ea = time.perf_counter() - t1
    J = float(((u[0].reshape(-1)[idx] - y) ** 2).sum())
    oi = np.asarray(g["index"])
    got = dJdf.cpu().numpy().reshape(-1)[oi]
    ref = np.asarray(g["dJdf"])
    return {"workload": "lrsw-fd-256x256-trho500-adjoint-fp64", "P": rf["P"],
            "forward_ms": 1000 * ef, "adjoint_ms": 1000 * ea, "adjoint_over_forward": ea / ef,
            "forward_value": D4 * D4 * rf["P"] / ef, "adjoint_value": D4 * D4 * ra["P"] / ea,
            "J_rel_err": abs(J - g["J"]) / g["J"],
            "dJdH_rel_err": abs(dJdH - g["dJdH"]) / abs(g["dJdH"]),
            "dJdf_rel_l2_samples": float(np.linalg.norm(got - ref) / np.linalg.norm(ref)),
            "err_bound_forward": rf["err_bound"], "err_bound_adjoint": ra["err_bound"]}

if __name__ == "__main__":
    main()
