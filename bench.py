"""Benchmark of structured random phase retrieval on one MI355X.

Headline (the JSON line's `value`): gradient-descent iterations per second on
the 2D image workload -- a 256x256 complex image zero-padded to 512x512
(alpha = 4), L = 2 random phase layers, Poisson noise at 1000 photons per
pixel, complex64.  One step = one GD solve of 500 iterations (Eq. (2)) from
the spectral estimate (100 power iterations, Eq. (3)-(4), timed alongside).
Inputs are synthetic, seeded, and resident in HBM before the timed region.

Beside it (skipped with --quick): the 1024^2 -> 2048^2, L = 3 operator and
solver, the dense i.i.d. MFMA baseline (16384 x 4096 complex64 A, 32
signals), 256 uneven problems batched vs the per-problem loop, the
64-problem mask-gradient (autograd) step vs a per-problem loop, the tiny 1D
problem, and the FP64 oracle timed on the host (`cpu_baseline`).

Prints one JSON line.  `python bench.py [--steps K] [--warmup W] [--quick]`.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
if HERE not in sys.path:
    sys.path.insert(0, HERE)

HBM_PEAK_GBS = 8000.0
FP32_MFMA_PEAK_TFLOPS = 157.3
GD_ITERS = 500
PI_ITERS = 100


# --------------------------------------------------------------------------
# Algorithmic byte model of the fused pass schedule (per unit of work)
# --------------------------------------------------------------------------

def schedule_bytes_gd(n_shape, m_shape, L):
    """Algorithmic HBM bytes of one GD iteration under the fused pass schedule
    (2L+1 passes, each one read and one write of its buffer).

    Pass 1 reads x (8n) and the support part of theta_1 (4n), writes the
    compact M1 x N2 buffer; each later pass reads and writes its buffer
    (compact next to the padding, full m-grid elsewhere) plus its phases
    (4 B per grid point) or measurements; the last pass reads the compact
    buffer, theta_1's support part and x, and writes x."""
    N1, N2 = n_shape
    M1, M2 = m_shape
    n, m, mc = N1 * N2, M1 * M2, M1 * N2
    b = 8 * n + 4 * n + 8 * mc                       # [U D1 F0]
    for k in range(2, L + 1):                          # [F D_k F]
        b += 8 * (mc if k == 2 else m) + 4 * m + 8 * m
    b += 8 * (mc if L == 1 else m) + 4 * m + 8 * (mc if L == 1 else m)  # turnaround (+ y)
    for k in range(L, 1, -1):                          # [F^H D_k^* F^H]
        b += 8 * m + 4 * m + 8 * (mc if k == 2 else m)
    b += 8 * mc + 4 * n + 8 * n + 8 * n               # [F0^H D1^* U^H] + x update
    return b


def compulsory_bytes_gd(n_shape, m_shape, L):
    """The floor of one GD iteration's HBM traffic if every intermediate stayed
    on chip: x read and written, y, theta_1 on the signal's support (D_1 only
    meets U x) and theta_2..theta_L on the whole grid."""
    N1, N2 = n_shape
    M1, M2 = m_shape
    n, m = N1 * N2, M1 * M2
    return 8 * n + 8 * n + 4 * m + 4 * n + 4 * m * (L - 1)


_CEILING = [None]  # the copy ceiling the headline measured, for the side workloads' fractions


def copy_ceiling_gbps(torch, dev, mib=512, reps=5):
    """Device-to-device copy rate (bytes read + written per second) of a
    `mib` MiB buffer: the practical HBM ceiling beside the 8 TB/s peak."""
    src = torch.empty(mib * 1024 * 1024 // 4, dtype=torch.float32, device=dev).fill_(1.0)
    dst = torch.empty_like(src)
    s = torch.cuda.current_stream()
    ms = _time_calls(torch, s, lambda: dst.copy_(src), reps)
    gbps = 2 * src.numel() * 4 / (ms * 1e-3) / 1e9
    del src, dst
    return gbps


def schedule_bytes_op(n_shape, m_shape, L):
    """Algorithmic bytes of one A (or A^H) application (x in, z out)."""
    N1, N2 = n_shape
    M1, M2 = m_shape
    n, m, mc = N1 * N2, M1 * M2, M1 * N2
    b = 8 * n + 4 * n + 8 * mc
    for k in range(2, L + 1):
        b += 8 * (mc if k == 2 else m) + 4 * m + 8 * m
    b += 8 * (mc if L == 1 else m) + 8 * m
    return b


# the sources the 2D pass kernels and their schedule are compiled from
PASS_SOURCES = ("fft_core.hpp", "passes.hpp", "launch.hpp", "passes_inst.hip", "dispatch.hip", "schedule.hpp",
                "sr_api.hip", "plan.hpp", "plan.hip")


def source_hash() -> str:
    """Hash of the pass-kernel sources, to tell whether stored counter data
    for the GD iteration is stale."""
    h = hashlib.sha256()
    csrc = os.path.join(HERE, "paper_2409_05734_amd", "csrc")
    for f in PASS_SOURCES:
        with open(os.path.join(csrc, f), "rb") as fh:
            h.update(f.encode() + fh.read())
    return h.hexdigest()[:16]


def stored_traffic():
    """Measured HBM bytes per GD iteration from the committed counter summary,
    if it was taken on the current kernels (else None)."""
    path = os.path.join(HERE, "profiles", "gd_image_512_traffic.txt")
    try:
        d = {}
        with open(path) as f:
            for line in f:
                parts = line.split()
                if len(parts) == 2 and not line.startswith("#"):
                    d[parts[0]] = parts[1]
        if d.get("source_hash") == source_hash():
            return float(d["bytes_per_gd_iteration"])
    except Exception:
        pass
    return None


# --------------------------------------------------------------------------
# helpers
# --------------------------------------------------------------------------

def _events(torch, n):
    return [torch.cuda.Event(enable_timing=True) for _ in range(n)]


def _time_calls(torch, stream, fn, reps, warm=3):
    for _ in range(warm):
        fn()
    a, b = _events(torch, 2)
    a.record(stream)
    for _ in range(reps):
        fn()
    b.record(stream)
    torch.cuda.synchronize()
    return a.elapsed_time(b) / reps  # ms


def cpu_baseline(d, y, x0, eta, budget_s=12.0):
    """Time the FP64 oracle's GD iterations on this host (bounded sample)."""
    import oracle
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        threads = os.cpu_count() or 1
    op = oracle.StructuredOperator(d["theta"], d["n_shape"])
    x = x0.astype(np.complex128)
    oracle.gd_solve(op, y, x, 1, eta)  # warm the DFT-matrix cache
    it, t0 = 0, time.perf_counter()
    while True:
        x = oracle.gd_solve(op, y, x, 1, eta)
        it += 1
        el = time.perf_counter() - t0
        if el >= budget_s or it >= 200:
            break
    return {"value": it / el, "unit": "GD iters/s", "cores": int(threads), "kind": "oracle",
            "sample": f"{it} GD iterations of the FP64 explicit-DFT oracle on the same 256^2 -> 512^2, L=2 "
                      f"problem ({el:.1f} s, {threads} BLAS threads, {os.cpu_count()} host cores visible)"}


def make_measurements(torch, srpr, plan, x_star, noise_rng, photons, dev):
    """Noiseless intensities from the library's forward operator, then Poisson
    photon noise drawn on the host (the noise model is an input, not the method)."""
    import sr_inputs
    m = plan.m_total
    yclean = torch.empty(m, dtype=torch.float32, device=dev)
    srpr.sr_forward(plan, torch.from_numpy(x_star.ravel()).to(dev), None, yclean)
    torch.cuda.synchronize()
    if noise_rng is None:
        return yclean
    return torch.from_numpy(sr_inputs.poisson_counts(noise_rng, yclean.cpu().numpy(), photons)).to(dev)


# --------------------------------------------------------------------------
# workloads
# --------------------------------------------------------------------------

def headline(torch, srpr, sr_inputs, dev, steps, warmup):
    d = sr_inputs.image_2d(1)
    n_shape, m_shape, L = d["n_shape"], d["m_shape"], d["layers"]
    n, m = int(np.prod(n_shape)), int(np.prod(m_shape))
    plan = srpr.Plan([srpr.Problem(n_shape, m_shape, L)], d["theta"])
    stream = plan.stream
    y = make_measurements(torch, srpr, plan, d["x_star"], d["noise_rng"], d["photons"], dev)
    y_h = y.cpu().numpy()
    v0 = torch.from_numpy(d["v0"].ravel()).to(dev)
    x0 = torch.empty(n, dtype=torch.complex64, device=dev)
    eta = float(d["mu"] * m / float(y_h.astype(np.float64).mean()))  # mu / (c mean(y)), c = 1/m

    srpr.sr_spectral_init(plan, y, v0, PI_ITERS, d["lam"], x0)
    pi_ms = _time_calls(torch, stream, lambda: srpr.sr_spectral_init(plan, y, v0, PI_ITERS, d["lam"], x0), 5)

    x = torch.empty_like(x0)
    for _ in range(warmup):
        x.copy_(x0)
        srpr.sr_gd_solve(plan, y, x, GD_ITERS, eta)
    torch.cuda.synchronize()
    ev = [_events(torch, 2) for _ in range(steps)]
    t0 = time.perf_counter()
    for i in range(steps):
        x.copy_(x0)
        ev[i][0].record(stream)
        srpr.sr_gd_solve(plan, y, x, GD_ITERS, eta)
        ev[i][1].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    solve_ms = float(np.mean([a.elapsed_time(b) for a, b in ev]))

    xs = torch.from_numpy(d["x_star"].ravel()).to(dev)
    z = torch.empty(m, dtype=torch.complex64, device=dev)
    r = torch.randn(m, dtype=torch.complex64, device=dev)
    xa = torch.empty(n, dtype=torch.complex64, device=dev)
    fwd_ms = _time_calls(torch, stream, lambda: srpr.sr_forward(plan, xs, z, None), 200)
    adj_ms = _time_calls(torch, stream, lambda: srpr.sr_adjoint(plan, r, xa), 200)
    op_bytes = schedule_bytes_op(n_shape, m_shape, L)
    gd_bytes = schedule_bytes_gd(n_shape, m_shape, L)

    xh = x.cpu().numpy().astype(np.complex128)
    xt = d["x_star"].ravel().astype(np.complex128)
    cos = float(abs(np.vdot(xh, xt)) / (np.linalg.norm(xh) * np.linalg.norm(xt)))
    it_us = solve_ms * 1e3 / GD_ITERS
    achieved = gd_bytes / (it_us * 1e-6) / 1e9
    comp_bytes = compulsory_bytes_gd(n_shape, m_shape, L)
    ceiling = copy_ceiling_gbps(torch, dev)
    _CEILING[0] = ceiling
    traffic = stored_traffic()
    return {
        "value": GD_ITERS * steps / wall,
        "ms_per_step": wall * 1e3 / steps,
        "solve_ms_events": solve_ms,
        "gd_iteration_us": it_us,
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "kernel": "one fused GD iteration (2L = 4 pass kernels in steady state, graph-replayed)",
                     "bytes_per_unit": gd_bytes, "unit_of_work": "GD iteration",
                     "copy_ceiling_GBps": ceiling, "frac_of_copy_ceiling": achieved / ceiling,
                     "compulsory_bytes_per_unit": comp_bytes,
                     "compulsory_GBps": comp_bytes / (it_us * 1e-6) / 1e9},
        "operator": {"A_us": fwd_ms * 1e3, "AH_us": adj_ms * 1e3,
                     "A_GBps": op_bytes / (fwd_ms * 1e-3) / 1e9, "AH_GBps": op_bytes / (adj_ms * 1e-3) / 1e9,
                     "bytes_per_application": op_bytes},
        "spectral_init": {"iters": PI_ITERS, "ms": pi_ms, "iters_per_s": PI_ITERS / (pi_ms * 1e-3)},
        "cosine_similarity": cos,
        "_cpu": (d, y_h.reshape(m_shape), x0.cpu().numpy().reshape(n_shape), eta),
    }


def large_2d(torch, srpr, sr_inputs, dev):
    d = sr_inputs.large_2d(4)
    n_shape, m_shape, L = d["n_shape"], d["m_shape"], d["layers"]
    n, m = int(np.prod(n_shape)), int(np.prod(m_shape))
    plan = srpr.Plan([srpr.Problem(n_shape, m_shape, L)], d["theta"])
    s = plan.stream
    y = make_measurements(torch, srpr, plan, d["x_star"], d["noise_rng"], d["photons"], dev)
    v0 = torch.from_numpy(d["v0"].ravel()).to(dev)
    x = torch.empty(n, dtype=torch.complex64, device=dev)
    pi_ms = _time_calls(torch, s, lambda: srpr.sr_spectral_init(plan, y, v0, d["pi_iters"], d["lam"], x), 2, warm=1)
    eta = float(d["mu"] * m / float(y.double().mean().item()))
    x0 = x.clone()

    def solve():
        x.copy_(x0)
        srpr.sr_gd_solve(plan, y, x, d["gd_iters"], eta)
    gd_ms = _time_calls(torch, s, solve, 3, warm=1)
    xs = torch.from_numpy(d["x_star"].ravel()).to(dev)
    z = torch.empty(m, dtype=torch.complex64, device=dev)
    fwd_ms = _time_calls(torch, s, lambda: srpr.sr_forward(plan, xs, z, None), 20)
    adj_ms = _time_calls(torch, s, lambda: srpr.sr_adjoint(plan, z, x), 20)
    op_bytes = schedule_bytes_op(n_shape, m_shape, L)
    gd_bytes = schedule_bytes_gd(n_shape, m_shape, L)
    it_us = gd_ms * 1e3 / d["gd_iters"]
    return {"workload": "1024^2 -> 2048^2 (alpha=4), L=3, Poisson 1000 photons",
            "gd_iters_per_s": d["gd_iters"] / (gd_ms * 1e-3), "gd_iteration_us": it_us,
            "gd_GBps": gd_bytes / (it_us * 1e-6) / 1e9, "gd_frac_hbm": gd_bytes / (it_us * 1e-6) / 1e9 / HBM_PEAK_GBS,
            "gd_frac_copy_ceiling": gd_bytes / (it_us * 1e-6) / 1e9 / _CEILING[0] if _CEILING[0] else None,
            "bytes_per_gd_iteration": gd_bytes,
            "spectral_iters_per_s": d["pi_iters"] / (pi_ms * 1e-3),
            "A_us": fwd_ms * 1e3, "AH_us": adj_ms * 1e3,
            "A_GBps": op_bytes / (fwd_ms * 1e-3) / 1e9, "AH_GBps": op_bytes / (adj_ms * 1e-3) / 1e9}


def dense(torch, srpr, sr_inputs, dev):
    db = sr_inputs.dense_batch(4)
    A = torch.from_numpy(db["dense_A"]).to(dev)
    X = torch.from_numpy(db["X"].ravel()).to(dev)
    R = torch.from_numpy(db["R"].ravel()).to(dev)
    del db
    m, n, nb = 16384, 4096, 32
    plan = srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(nb)], None, dense_A=A)
    s = plan.stream
    Z = torch.empty(nb * m, dtype=torch.complex64, device=dev)
    V = torch.empty(nb * n, dtype=torch.complex64, device=dev)
    fwd_ms = _time_calls(torch, s, lambda: srpr.sr_forward(plan, X, Z, None), 20)
    adj_ms = _time_calls(torch, s, lambda: srpr.sr_adjoint(plan, R, V), 20)
    flops = 8.0 * m * n * nb
    bytes_ = 8.0 * m * n + 8.0 * nb * (m + n)
    return {"workload": "dense i.i.d. CN(0,1) A 16384 x 4096 complex64 (512 MiB), 32 signals, FP32 MFMA",
            "A_us": fwd_ms * 1e3, "AH_us": adj_ms * 1e3,
            "A_TFLOPs": flops / (fwd_ms * 1e-3) / 1e12, "AH_TFLOPs": flops / (adj_ms * 1e-3) / 1e12,
            "A_frac_mfma": flops / (fwd_ms * 1e-3) / 1e12 / FP32_MFMA_PEAK_TFLOPS,
            "AH_frac_mfma": flops / (adj_ms * 1e-3) / 1e12 / FP32_MFMA_PEAK_TFLOPS,
            "A_GBps": bytes_ / (fwd_ms * 1e-3) / 1e9}


def batched(torch, srpr, sr_inputs, dev, iters=300):
    probs = sr_inputs.batched_mixed(2, 256)
    plan = srpr.Plan([srpr.Problem(p["n_shape"], p["m_shape"], p["layers"]) for p in probs],
                     np.concatenate([p["theta"].ravel() for p in probs]))
    s = plan.stream
    xs = np.concatenate([p["x_star"].ravel() for p in probs])
    y = torch.empty(plan.m_total, dtype=torch.float32, device=dev)
    srpr.sr_forward(plan, torch.from_numpy(xs).to(dev), None, y)
    yh = y.cpu().numpy()
    eta = np.array([p["mu"] * int(np.prod(p["m_shape"])) / float(np.mean(yh[plan.y_off[i]:plan.y_off[i + 1]]))
                    for i, p in enumerate(probs)], dtype=np.float32)
    x0 = torch.from_numpy(np.concatenate([p["x0"].ravel() for p in probs])).to(dev)
    x = torch.empty_like(x0)

    def run():
        x.copy_(x0)
        srpr.sr_gd_solve(plan, y, x, iters, eta)
    v0 = torch.randn_like(x0)
    est = torch.empty_like(x0)

    def run_spec():
        srpr.sr_spectral_init(plan, y, v0, 100, -1.0, est)
    xsd = torch.from_numpy(xs).to(dev)
    yop = torch.empty_like(y)

    def run_fwd():
        srpr.sr_forward(plan, xsd, None, yop)
    def status():
        # the library's own report of NaN / Inf results since the last check
        try:
            srpr.sr_plan_sync(plan)
            return "ok"
        except srpr.SrError as e:
            if e.status != srpr.SR_E_NONFINITE:
                raise
            return "SR_E_NONFINITE"
    srpr.sr_plan_set_schedule(plan, srpr.SR_SCHED_BATCHED)
    bf_ms = _time_calls(torch, s, run_fwd, 20, warm=2)
    status()
    b_ms = _time_calls(torch, s, run, 3, warm=1)
    st_batched = status()
    xb = x.clone()
    bs_ms = _time_calls(torch, s, run_spec, 3, warm=1)
    eb_spec = est.clone()
    srpr.sr_plan_set_schedule(plan, srpr.SR_SCHED_LOOP)
    status()
    l_ms = _time_calls(torch, s, run, 1, warm=1)
    st_loop = status()
    ls_ms = _time_calls(torch, s, run_spec, 1, warm=1)
    lf_ms = _time_calls(torch, s, run_fwd, 5, warm=1)
    spec_rel = float(((eb_spec - est).abs().pow(2).sum() / est.abs().pow(2).sum()).sqrt())
    # accuracy of both schedules per problem: phase-aligned relative error to x*
    xbh, xlh = xb.cpu().numpy().astype(np.complex128), x.cpu().numpy().astype(np.complex128)

    def err(xh, i):
        a, r = xh[plan.x_off[i]:plan.x_off[i + 1]], probs[i]["x_star"].ravel().astype(np.complex128)
        if not np.isfinite(a).all():
            return np.inf
        c = np.vdot(a, r)
        a = a * (c / abs(c) if abs(c) > 0 else 1.0)
        return float(np.linalg.norm(a - r) / np.linalg.norm(r))
    eb = np.array([err(xbh, i) for i in range(len(probs))])
    el = np.array([err(xlh, i) for i in range(len(probs))])
    # problems whose 300 steps from the random start diverge (the step mu = 0.2
    # is fixed for all): listed on their own; they cost the same time per step
    diverged = [{"index": i, "n_side": probs[i]["n_shape"][0], "m_shape": list(probs[i]["m_shape"]),
                 "layers": probs[i]["layers"], "batched": bool(np.isinf(eb[i])), "loop": bool(np.isinf(el[i]))}
                for i in range(len(probs)) if np.isinf(eb[i]) or np.isinf(el[i])]
    both = (eb < 1e-3) & (el < 1e-3)
    byt = sum(schedule_bytes_gd(p["n_shape"], p["m_shape"], p["layers"]) for p in probs)
    return {"workload": "256 problems, N in {32,64,96,128}^2, alpha in {2,4,8}, L in {1,2,3}, 300 GD steps",
            "batched_ms": b_ms, "loop_ms": l_ms, "speedup_vs_loop": l_ms / b_ms,
            "forward_batched_us": bf_ms * 1e3, "forward_loop_us": lf_ms * 1e3,
            "spectral_100_batched_ms": bs_ms, "spectral_100_loop_ms": ls_ms,
            "spectral_speedup_vs_loop": ls_ms / bs_ms, "spectral_rel_diff_vs_loop": spec_rel,
            "batched_gd_iters_per_s": iters / (b_ms * 1e-3),
            "batched_GBps": byt * iters / (b_ms * 1e-3) / 1e9, "bytes_per_batched_iteration": byt,
            "recovered_batched": int((eb < 1e-3).sum()), "recovered_loop": int((el < 1e-3).sum()),
            "nonfinite_batched": int(np.isinf(eb).sum()), "nonfinite_loop": int(np.isinf(el).sum()),
            "library_status_batched": st_batched, "library_status_loop": st_loop, "diverged": diverged,
            "max_err_recovered_batched": float(eb[both].max()) if both.any() else None,
            "max_err_recovered_loop": float(el[both].max()) if both.any() else None,
            "median_err_batched": float(np.median(eb)), "median_err_loop": float(np.median(el)),
            "max_err_gap_finite": float(np.max(np.abs(eb[np.isfinite(eb) & np.isfinite(el)]
                                                     - el[np.isfinite(eb) & np.isfinite(el)])))}


def latency_floor(torch, srpr, sr_inputs, dev, reps=400):
    """What a kernel boundary costs at the headline's size, for comparison
    with its passes (2L = 4 kernels per GD iteration): graph-replayed chains
    of a one-element elementwise kernel (the launch floor) and of a 2 MiB
    elementwise kernel (one 512^2 complex64 grid read and written, as a pass
    does, without the FFTs), per kernel."""
    out = {"workload": f"HIP graph of {reps} dependent elementwise kernels, replayed"}
    s = torch.cuda.Stream()
    for name, numel in (("tiny_kernel_us", 1), ("grid_2MiB_kernel_us", 512 * 512)):
        a = torch.ones(numel, dtype=torch.complex64, device=dev)
        b = torch.empty_like(a)
        with torch.cuda.stream(s):
            torch.add(a, 1.0, out=b)
            torch.add(b, 1.0, out=a)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            for i in range(reps // 2):
                torch.add(a, 1.0, out=b)
                torch.add(b, 1.0, out=a)
        g.replay()
        torch.cuda.synchronize()
        e0, e1 = _events(torch, 2)
        cur = torch.cuda.current_stream()  # replay() launches on the current stream
        e0.record(cur)
        for _ in range(3):
            g.replay()
        e1.record(cur)
        torch.cuda.synchronize()
        out[name] = e0.elapsed_time(e1) * 1e3 / (3 * reps)
        del g, a, b
    return out


def library_loop(torch, srpr, sr_inputs, dev, iters=200):
    """The headline's GD iteration written with PyTorch's FFT (rocFFT) and
    elementwise ops on the same GPU, one library call at a time (pad, L x
    [phase, 2D FFT], residual, L x [inverse FFT, conjugate phase], crop,
    update): the plain loop the fused passes replace.  Same inputs and step;
    reports both times per iteration and the relative difference of the
    iterates after the run."""
    d = sr_inputs.image_2d(1)
    n_shape, m_shape, L = d["n_shape"], d["m_shape"], d["layers"]
    (N1, N2), (M1, M2) = n_shape, m_shape
    n, m = N1 * N2, M1 * M2
    o1, o2 = (M1 - N1) // 2, (M2 - N2) // 2
    plan = srpr.Plan([srpr.Problem(n_shape, m_shape, L)], d["theta"])
    xs = torch.from_numpy(d["x_star"].ravel()).to(dev)
    y = torch.empty(m, dtype=torch.float32, device=dev)
    srpr.sr_forward(plan, xs, None, y)
    th = torch.from_numpy(d["theta"]).to(dev)
    D = torch.polar(torch.ones_like(th), th)
    Dc = D.conj().resolve_conj()
    y2 = y.reshape(m_shape)
    step = float(d["mu"] * m / float(y.double().mean().item())) / m
    x0 = (xs + 0.3 * torch.randn_like(xs)).reshape(n_shape).contiguous()

    def lib_step(x):
        w = torch.zeros(m_shape, dtype=torch.complex64, device=dev)
        w[o1:o1 + N1, o2:o2 + N2] = x
        for l in range(L):
            w = torch.fft.fft2(D[l] * w, norm="ortho")
        r = (w.real * w.real + w.imag * w.imag - y2) * w
        for l in reversed(range(L)):
            r = Dc[l] * torch.fft.ifft2(r, norm="ortho")
        return x - step * r[o1:o1 + N1, o2:o2 + N2]

    xl = x0.clone()

    def run_lib():
        nonlocal xl
        xl = x0.clone()
        for _ in range(iters):
            xl = lib_step(xl)
    s = torch.cuda.current_stream()
    lib_ms = _time_calls(torch, s, run_lib, 2, warm=1)
    xf = torch.empty(n, dtype=torch.complex64, device=dev)
    eta = np.float32(step * m)

    def run_fused():
        xf.copy_(x0.ravel())
        srpr.sr_gd_solve(plan, y, xf, iters, eta)
    fused_ms = _time_calls(torch, plan.stream, run_fused, 3, warm=1)
    rel = float(((xf - xl.ravel()).abs().pow(2).sum() / xl.abs().pow(2).sum()).sqrt())
    return {"workload": f"256^2 -> 512^2, L=2, {iters} GD steps: torch.fft + elementwise ops vs the fused passes",
            "library_iteration_us": lib_ms * 1e3 / iters, "fused_iteration_us": fused_ms * 1e3 / iters,
            "speedup_vs_library_loop": lib_ms / fused_ms, "rel_diff_of_iterates": rel}


def stacked_gd(torch, srpr, sr_inputs, dev, count=16, iters=300):
    """A uniform batch at the headline shape (256^2 -> 512^2, L = 2, each
    problem with its own masks and step): every pass launched once for the
    whole stack against the problem-by-problem loop."""
    rng = np.random.default_rng(17)
    n_shape, m_shape, L = (256, 256), (512, 512), 2
    n, m = 256 * 256, 512 * 512
    theta = rng.uniform(0, 2 * np.pi, (count, L) + m_shape).astype(np.float32)
    plan = srpr.Plan([srpr.Problem(n_shape, m_shape, L, theta_offset=i * L * m) for i in range(count)], theta.ravel())
    xs = torch.from_numpy(np.concatenate([sr_inputs.complex_gaussian(rng, n_shape).ravel()
                                          for _ in range(count)])).to(dev)
    y = torch.empty(plan.m_total, dtype=torch.float32, device=dev)
    srpr.sr_forward(plan, xs, None, y)
    x0 = (xs + 0.5 * torch.randn_like(xs)).contiguous()
    ym = y.reshape(count, m).double().mean(dim=1).cpu().numpy()
    eta = (0.2 * m / ym).astype(np.float32)
    x = torch.empty_like(x0)

    def run():
        x.copy_(x0)
        srpr.sr_gd_solve(plan, y, x, iters, eta)
    v0 = torch.randn_like(xs)
    est = torch.empty_like(xs)

    def run_spec():
        srpr.sr_spectral_init(plan, y, v0, iters, -1.0, est)
    s_ms = _time_calls(torch, plan.stream, run, 3, warm=1)
    xa = x.clone()
    s_spec_ms = _time_calls(torch, plan.stream, run_spec, 3, warm=1)
    ea = est.clone()
    srpr.sr_plan_set_schedule(plan, srpr.SR_SCHED_LOOP)
    l_ms = _time_calls(torch, plan.stream, run, 2, warm=1)
    l_spec_ms = _time_calls(torch, plan.stream, run_spec, 2, warm=1)
    byt = count * schedule_bytes_gd(n_shape, m_shape, L)
    return {"workload": f"{count} problems 256^2 -> 512^2, L=2, own masks and steps, {iters} GD steps; "
                        f"{iters} power iterations",
            "stacked_ms": s_ms, "loop_ms": l_ms, "speedup_vs_loop": l_ms / s_ms,
            "stacked_problem_iters_per_s": count * iters / (s_ms * 1e-3),
            "stacked_GBps": byt * iters / (s_ms * 1e-3) / 1e9,
            "stacked_frac_copy_ceiling": byt * iters / (s_ms * 1e-3) / 1e9 / _CEILING[0] if _CEILING[0] else None,
            "bit_identical_to_loop": bool(torch.equal(xa, x)),
            "spectral_stacked_ms": s_spec_ms, "spectral_loop_ms": l_spec_ms,
            "spectral_speedup_vs_loop": l_spec_ms / s_spec_ms,
            "spectral_bit_identical_to_loop": bool(torch.equal(ea, est))}


def autograd(torch, srpr, sr_inputs, dev):
    from paper_2409_05734_amd.autograd import unrolled_gd_loss
    d = sr_inputs.mask_design(3)
    B, L = d["x_star"].shape[0], d["layers"]
    n_shape, m_shape = d["n_shape"], d["m_shape"]
    th = torch.from_numpy(d["theta"].ravel()).to(dev)
    xs = torch.from_numpy(d["x_star"].reshape(B, -1)).to(dev)
    x0 = torch.from_numpy(d["x0"].reshape(B, -1)).to(dev)
    plan = srpr.Plan([srpr.Problem(n_shape, m_shape, L, theta_offset=0) for _ in range(B)], d["theta"])
    singles = [srpr.Plan([srpr.Problem(n_shape, m_shape, L, theta_offset=0)], d["theta"]) for _ in range(1)]
    s = plan.stream

    def batch_step():
        t = th.clone().requires_grad_(True)
        loss = unrolled_gd_loss(plan, t, xs, x0, d["steps"], d["mu"])
        loss.backward()
        return t.grad

    def loop_step():
        t = th.clone().requires_grad_(True)
        tot = 0.0
        for b in range(B):
            tot = tot + unrolled_gd_loss(singles[0], t, xs[b:b + 1], x0[b:b + 1], d["steps"], d["mu"]) / B
        tot.backward()
        return t.grad

    def peak_bytes(steps):
        # torch-allocated device memory of one objective and its gradient
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats(dev)
        base = torch.cuda.memory_allocated(dev)
        t = th.clone().requires_grad_(True)
        unrolled_gd_loss(plan, t, xs, x0, steps, d["mu"]).backward()
        torch.cuda.synchronize()
        return torch.cuda.max_memory_allocated(dev) - base

    g1 = batch_step()
    g2 = loop_step()
    rel = float(((g1 - g2).norm() / g2.norm()).item())
    b_ms = _time_calls(torch, s, batch_step, 2, warm=1)
    l_ms = _time_calls(torch, s, loop_step, 1, warm=0)
    p20, p10 = peak_bytes(d["steps"]), peak_bytes(d["steps"] // 2)
    n_tot, m_tot = B * int(np.prod(n_shape)), B * int(np.prod(m_shape))
    return {"workload": "64 problems 128^2 -> 256^2, L=2, loss after 20 unrolled GD steps, d loss / d theta",
            "batched_plan_ms": b_ms, "per_problem_loop_ms": l_ms, "speedup_vs_loop": l_ms / b_ms,
            "grad_rel_diff_vs_loop": rel,
            "torch_peak_bytes_20_steps": int(p20), "torch_peak_bytes_10_steps": int(p10),
            "torch_bytes_per_step": (p20 - p10) / (d["steps"] - d["steps"] // 2),
            "signal_bytes_per_step": 8 * n_tot, "measurement_bytes": 8 * m_tot,
            "library_temporaries_bytes": 8 * L * m_tot}


def lds_resident(torch, srpr, sr_inputs, dev, count=512, iters=300):
    """Many small 2D problems (64^2 grids, L = 2): the LDS-resident solver (one
    workgroup per problem for the whole solve) against the level launches."""
    rng = np.random.default_rng(7)
    n_shape, m_shape, L = (32, 32), (64, 64), 2
    probs = [srpr.Problem(n_shape, m_shape, L) for _ in range(count)]
    theta = rng.uniform(0, 2 * np.pi, (count, L) + m_shape).astype(np.float32)
    plan = srpr.Plan(probs, theta.ravel())
    srpr.sr_plan_set_schedule(plan, srpr.SR_SCHED_BATCHED)
    xs = torch.from_numpy(np.concatenate([sr_inputs.complex_gaussian(rng, n_shape).ravel() for _ in range(count)]))
    xs = xs.to(dev)
    y = torch.empty(plan.m_total, dtype=torch.float32, device=dev)
    srpr.sr_forward(plan, xs, None, y)
    x0 = (xs + 0.5 * torch.randn_like(xs)).contiguous()
    eta = np.full(count, 0.2 * int(np.prod(m_shape)) / float(y.double().mean().item()), np.float32)
    x = torch.empty_like(x0)
    out = {"workload": f"{count} problems 32^2 -> 64^2, L=2, {iters} GD steps from x* + CN(0, 1/4)"}
    finals = {}
    for key, env in (("lds_resident_ms", "1"), ("levels_ms", "0"), ("stacked_ms", None)):
        if env is None:  # the default schedule of a uniform plan: each pass once for the whole stack
            os.environ.pop("SR_LDS_RESIDENT", None)
            srpr.sr_plan_set_schedule(plan, srpr.SR_SCHED_AUTO)
        else:
            os.environ["SR_LDS_RESIDENT"] = env

        def run():
            x.copy_(x0)
            srpr.sr_gd_solve(plan, y, x, iters, eta)
        out[key] = _time_calls(torch, plan.stream, run, 3, warm=1)
        finals[key] = x.clone()
    os.environ.pop("SR_LDS_RESIDENT", None)
    a, b = finals["lds_resident_ms"], finals["levels_ms"]
    out["rel_diff_between_schedules"] = float(((a - b).abs().pow(2).sum() / b.abs().pow(2).sum()).sqrt())
    out["speedup_vs_levels"] = out["levels_ms"] / out["lds_resident_ms"]
    out["rel_diff_stacked_vs_levels"] = float(((finals["stacked_ms"] - b).abs().pow(2).sum()
                                               / b.abs().pow(2).sum()).sqrt())
    return out


def forward_time_sweep(torch, srpr, sr_inputs, dev):
    """Forward time per application at oversampling ratio 1 against image size,
    structured (L = 2) and dense i.i.d. (the shape of the paper's forward-time
    comparison; the dense matrix is drawn on the device)."""
    rng = np.random.default_rng(11)
    out = {"workload": "alpha = 1, one image per application; structured L = 2, dense i.i.d. CN(0,1)",
           "structured": [], "dense": []}
    for side in (32, 64, 128, 256, 512, 1024, 2048):
        shape = (side, side)
        theta = rng.uniform(0, 2 * np.pi, (2,) + shape).astype(np.float32)
        plan = srpr.Plan([srpr.Problem(shape, shape, 2)], theta)
        x = torch.from_numpy(sr_inputs.complex_gaussian(rng, shape).ravel()).to(dev)
        z = torch.empty(side * side, dtype=torch.complex64, device=dev)
        ms = _time_calls(torch, plan.stream, lambda: srpr.sr_forward(plan, x, z, None), 50)
        out["structured"].append({"pixels": side * side, "forward_us": ms * 1e3})
        del plan
    g = torch.Generator(device=dev)
    g.manual_seed(12)
    for side in (32, 64, 128, 240):
        n = side * side
        A = torch.randn((n, n), dtype=torch.complex64, device=dev, generator=g)
        plan = srpr.Plan([srpr.Problem((n,), (n,), 1, kind=srpr.SR_DENSE)], None, dense_A=A)
        x = torch.randn(n, dtype=torch.complex64, device=dev, generator=g)
        z = torch.empty(n, dtype=torch.complex64, device=dev)
        ms = _time_calls(torch, plan.stream, lambda: srpr.sr_forward(plan, x, z, None), 5 if side >= 240 else 20)
        out["dense"].append({"pixels": n, "forward_us": ms * 1e3, "matrix_GB": n * n * 8 / 1e9})
        del plan, A
        torch.cuda.empty_cache()
    return out


def layer_study(torch, srpr, sr_inputs, dev, grid=64, sides=(46, 42, 38, 36, 34, 32, 30, 28), reps=100, iters=5000):
    """The paper's layer-count comparison (section IV, number of layers): 2D
    structured models on a 64 x 64 grid with L = 1, 2, 3 layers, one layer
    after an extra FFT (L = 2 with theta_1 = 0, i.e. A = F D_2 F U), and a
    random unitary model (the first n columns of a Haar unitary, scaled so
    that the mean squared entry is 1, one draw per ratio shared by its
    signals); spectral estimates after 5000 power iterations (no early stop)
    on phase-only synthetic images.  Square image sides set the oversampling
    ratios (alpha = 4096 / side^2, about 2 to 5; even sides, since the dense
    model takes even signal lengths).  Reports the median and the
    10% / 90% quantiles of the cosine similarity over `reps` signals.  All
    structured problems of one ratio run in one batched plan."""
    rng = np.random.default_rng(21)
    m_shape = (grid, grid)
    m = grid * grid
    models = (("L1", 1, False), ("L2", 2, False), ("L3", 3, False), ("L1+FFT", 2, True))
    names_all = [nm for nm, _, _ in models] + ["unitary"]
    out = {"workload": f"2D, {grid}x{grid} grid, phase-only images, {reps} signals per point, "
                       f"{iters} power iterations",
           "alpha": [round(m / (n * n), 3) for n in sides]}
    for name in names_all:
        out[name] = {"median": [], "q10": [], "q90": []}

    def cosines(est, xs, count, n):
        xe = est.reshape(count, n).cpu().numpy().astype(np.complex128)
        xt = xs.reshape(count, n).cpu().numpy().astype(np.complex128)
        return np.abs(np.sum(np.conj(xe) * xt, axis=1)) / (np.linalg.norm(xe, axis=1) * np.linalg.norm(xt, axis=1))

    def record(name, cos):
        out[name]["median"].append(round(float(np.median(cos)), 4))
        out[name]["q10"].append(round(float(np.quantile(cos, 0.1)), 4))
        out[name]["q90"].append(round(float(np.quantile(cos, 0.9)), 4))

    t0 = time.perf_counter()
    for side in sides:
        n_shape = (side, side)
        n = side * side
        probs, thetas, xs, names = [], [], [], []
        for name, L, extra_fft in models:
            for _ in range(reps):
                th = rng.uniform(0, 2 * np.pi, (L,) + m_shape).astype(np.float32)
                if extra_fft:
                    th[0] = 0.0
                probs.append(srpr.Problem(n_shape, m_shape, L))
                thetas.append(th.ravel())
                xs.append(sr_inputs.phase_only_image(rng, n_shape).ravel())
                names.append(name)
        plan = srpr.Plan(probs, np.concatenate(thetas))
        x = torch.from_numpy(np.concatenate(xs)).to(dev)
        y = torch.empty(plan.m_total, dtype=torch.float32, device=dev)
        srpr.sr_forward(plan, x, None, y)
        v0 = torch.from_numpy(np.concatenate([sr_inputs.complex_gaussian(rng, (n,)) for _ in probs])).to(dev)
        est = torch.empty_like(v0)
        srpr.sr_spectral_init(plan, y, v0, iters, -1.0, est)
        torch.cuda.synchronize()
        cos = cosines(est, x, len(probs), n)
        for name, _, _ in models:
            record(name, cos[[i for i, nm in enumerate(names) if nm == name]])
        # random unitary baseline: Q of the QR factorisation of a complex Gaussian m x n matrix
        g = torch.from_numpy(sr_inputs.complex_gaussian(rng, (m, n))).to(dev)
        q, r = torch.linalg.qr(g)
        d = torch.diagonal(r)
        q = (q * (d / d.abs()).unsqueeze(0) * float(np.sqrt(m))).contiguous()
        dplan = srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(reps)], None, dense_A=q)
        xu = torch.from_numpy(np.concatenate([sr_inputs.phase_only_image(rng, n_shape).ravel()
                                              for _ in range(reps)])).to(dev)
        yu = torch.empty(reps * m, dtype=torch.float32, device=dev)
        srpr.sr_forward(dplan, xu, None, yu)
        v0u = torch.from_numpy(np.concatenate([sr_inputs.complex_gaussian(rng, (n,)) for _ in range(reps)])).to(dev)
        eu = torch.empty_like(v0u)
        srpr.sr_spectral_init(dplan, yu, v0u, iters, -1.0, eu)
        torch.cuda.synchronize()
        record("unitary", cosines(eu, xu, reps, n))
        del plan, dplan, q, g
        print(f"layer study: alpha {m / n:.2f} done ({time.perf_counter() - t0:.1f} s)", file=sys.stderr, flush=True)
    out["gpu_wall_s"] = round(time.perf_counter() - t0, 2)
    return out


def accuracy_sweep(torch, srpr, sr_inputs, dev, side=32, reps=100, dense_groups=4, gd_iters=10000, pi_iters=5000,
                   mu=0.05):
    """The paper's accuracy comparison (section IV-A): cosine similarity of
    gradient descent from a random start (GD), the spectral estimate alone
    (SM, lambda = -1) and GD from the spectral estimate (GD+SM) against the
    oversampling ratio, for the structured model (L = 2, fresh phases per
    repetition) and the i.i.d. CN(0,1) model (`dense_groups` matrices, each
    shared by reps/dense_groups repetitions), on one 32 x 32 phase-only
    synthetic image; 10000 GD / 5000 power iterations without early
    stopping, step eta = mu / (c mean(y)); median and 10 % / 90 % quantiles
    over `reps` repetitions (random starts differ per repetition)."""
    rng = np.random.default_rng(33)
    n_shape = (side, side)
    n = side * side
    x_star = sr_inputs.phase_only_image(rng, n_shape).ravel()
    grids = {1: (32, 32), 2: (64, 32), 3: (96, 32), 4: (64, 64), 6: (96, 64), 8: (128, 64), 9: (96, 96)}
    out = {"workload": f"{side}x{side} phase-only image, {reps} repetitions, {gd_iters} GD / {pi_iters} power "
                       f"iterations, mu = {mu}, structured L = 2 vs i.i.d. CN(0,1)",
           "alpha": sorted(grids)}
    for model in ("structured", "iid"):
        for meth in ("GD", "SM", "GD+SM"):
            out[f"{model} {meth}"] = {"median": [], "q10": [], "q90": [], "nonfinite": []}

    def record(key, est, count):
        xe = est.reshape(count, n).cpu().numpy().astype(np.complex128)
        xt = x_star.astype(np.complex128)
        with np.errstate(invalid="ignore", over="ignore"):
            cos = np.abs(xe.conj() @ xt) / (np.linalg.norm(xe, axis=1) * np.linalg.norm(xt))
        bad = ~np.isfinite(cos)
        cos = np.where(bad, 0.0, cos)  # a diverged run recovers nothing
        out[key]["median"].append(round(float(np.median(cos)), 4))
        out[key]["q10"].append(round(float(np.quantile(cos, 0.1)), 4))
        out[key]["q90"].append(round(float(np.quantile(cos, 0.9)), 4))
        out[key]["nonfinite"].append(int(bad.sum()))

    def starts(count, ysum_over_mc):
        # random starts CN(0,1) scaled to the norm the measurements imply
        v = np.stack([sr_inputs.complex_gaussian(rng, (n,)) for _ in range(count)])
        v *= np.sqrt(ysum_over_mc[:, None] / np.sum(np.abs(v) ** 2, axis=1, keepdims=True))
        return torch.from_numpy(v.astype(np.complex64).ravel()).to(dev)

    def solve_all(plans, c_of, key_model):
        # plans: list of (plan, count); returns nothing, records the three methods
        for meth in ("GD", "SM", "GD+SM"):
            ests = []
            for plan, count, y, m in plans:
                yh = y.cpu().numpy().astype(np.float64).reshape(count, m)
                c = c_of(m)
                eta = (mu / (c * yh.mean(axis=1))).astype(np.float32)
                if meth == "GD":
                    x = starts(count, yh.sum(axis=1) / (m * c))
                    srpr.sr_gd_solve(plan, y, x, gd_iters, eta)
                else:
                    v0 = torch.from_numpy(np.concatenate([sr_inputs.complex_gaussian(rng, (n,))
                                                          for _ in range(count)])).to(dev)
                    x = torch.empty_like(v0)
                    srpr.sr_spectral_init(plan, y, v0, pi_iters, -1.0, x)
                    if meth == "GD+SM":
                        srpr.sr_gd_solve(plan, y, x, gd_iters, eta)
                ests.append(x)
            torch.cuda.synchronize()
            record(f"{key_model} {meth}", torch.cat(ests), reps)

    t0 = time.perf_counter()
    xs_all = torch.from_numpy(np.tile(x_star, reps)).to(dev)
    for alpha in sorted(grids):
        m_shape = grids[alpha]
        m = m_shape[0] * m_shape[1]
        # structured, L = 2: one plan with a fresh theta per repetition
        th = rng.uniform(0, 2 * np.pi, (reps, 2) + m_shape).astype(np.float32)
        plan = srpr.Plan([srpr.Problem(n_shape, m_shape, 2) for _ in range(reps)], th.ravel())
        y = torch.empty(plan.m_total, dtype=torch.float32, device=dev)
        srpr.sr_forward(plan, xs_all, None, y)
        solve_all([(plan, reps, y, m)], lambda mm: 1.0 / mm, "structured")
        del plan, y
        # i.i.d.: dense_groups matrices, each shared by reps / dense_groups signals
        per = reps // dense_groups
        dplans = []
        for _ in range(dense_groups):
            A = torch.from_numpy(sr_inputs.complex_gaussian(rng, (m, n))).to(dev)
            dp = srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(per)], None, dense_A=A)
            yd = torch.empty(per * m, dtype=torch.float32, device=dev)
            srpr.sr_forward(dp, xs_all[:per * n], None, yd)
            dplans.append((dp, per, yd, m))
        solve_all(dplans, lambda mm: 1.0, "iid")
        del dplans
        torch.cuda.empty_cache()
        print(f"accuracy sweep: alpha {alpha} done ({time.perf_counter() - t0:.1f} s)", file=sys.stderr, flush=True)
    out["gpu_wall_s"] = round(time.perf_counter() - t0, 2)
    return out


def poisson_loss(torch, srpr, sr_inputs, dev, iters=1000, time_iters=500, pi_iters=400):
    """GD on the image workload (256^2 -> 512^2, L = 2, Poisson noise at 1000
    photons) with the l2 intensity loss (mu = 0.05) and with the Poisson
    negative log-likelihood (eta = mu / c, mu = 0.05, eps = 1e-2 mean(y)),
    both from the same spectral start (400 power iterations: the headline's
    100 leave the start unconverged at this size): cosine similarity after
    `iters` steps and time per iteration."""
    d = sr_inputs.image_2d(1)
    n_shape, m_shape, L = d["n_shape"], d["m_shape"], d["layers"]
    n, m = int(np.prod(n_shape)), int(np.prod(m_shape))
    plan = srpr.Plan([srpr.Problem(n_shape, m_shape, L)], d["theta"])
    s = plan.stream
    y = make_measurements(torch, srpr, plan, d["x_star"], d["noise_rng"], d["photons"], dev)
    ybar = float(y.double().mean().item())
    v0 = torch.from_numpy(d["v0"].ravel()).to(dev)
    x0 = torch.empty(n, dtype=torch.complex64, device=dev)
    srpr.sr_spectral_init(plan, y, v0, pi_iters, d["lam"], x0)
    xt = d["x_star"].ravel().astype(np.complex128)
    out = {"workload": f"256^2 -> 512^2, L = 2, Poisson noise (1000 photons), {pi_iters} PI then {iters} GD"}
    xh0 = x0.cpu().numpy().astype(np.complex128)
    out["spectral_start_cosine"] = float(abs(np.vdot(xh0, xt)) / (np.linalg.norm(xh0) * np.linalg.norm(xt)))
    x = torch.empty_like(x0)
    for name, loss, eps, eta in (("l2", srpr.SR_LOSS_L2, 0.0, 0.05 * m / ybar),
                                 ("poisson", srpr.SR_LOSS_POISSON, 1e-2 * ybar, 0.05 * m)):
        srpr.sr_plan_set_loss(plan, loss, eps)

        def solve(k):
            x.copy_(x0)
            srpr.sr_gd_solve(plan, y, x, k, float(eta))
        ms = _time_calls(torch, s, lambda: solve(time_iters), 3, warm=1)
        solve(iters)
        torch.cuda.synchronize()
        xh = x.cpu().numpy().astype(np.complex128)
        with np.errstate(invalid="ignore"):
            cos = float(abs(np.vdot(xh, xt)) / (np.linalg.norm(xh) * np.linalg.norm(xt)))
        out[name] = {"gd_iteration_us": ms * 1e3 / time_iters, "cosine_similarity": cos}
    srpr.sr_plan_set_loss(plan, srpr.SR_LOSS_L2)
    return out


def tiny_1d(torch, srpr, sr_inputs, dev):
    d = sr_inputs.tiny_1d(0)
    plan = srpr.Plan([srpr.Problem(d["n_shape"], d["m_shape"], d["layers"])], d["theta"])
    s = plan.stream
    y = make_measurements(torch, srpr, plan, d["x_star"], None, 0, dev)
    v0 = torch.from_numpy(d["v0"]).to(dev)
    x = torch.empty(64, dtype=torch.complex64, device=dev)
    eta = float(d["mu"] * 256 / float(y.double().mean().item()))

    def solve():
        srpr.sr_spectral_init(plan, y, v0, d["pi_iters"], d["lam"], x)
        srpr.sr_gd_solve(plan, y, x, d["gd_iters"], eta)
    ms = _time_calls(torch, s, solve, 20)
    xh = x.cpu().numpy().astype(np.complex128)
    xt = d["x_star"].astype(np.complex128)
    cos = float(abs(np.vdot(xh, xt)) / (np.linalg.norm(xh) * np.linalg.norm(xt)))
    return {"workload": "1D n=64, m=256, L=2: 50 power iterations + 200 GD (one workgroup, LDS-resident)",
            "solve_us": ms * 1e3, "gd_plus_pi_iters_per_s": 250 / (ms * 1e-3), "cosine_similarity": cos}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--quick", action="store_true", help="headline only (no side workloads, no CPU baseline)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--extras", default="all",
                    help="comma-separated side workloads to run (default: all but accuracy_sweep)")
    ap.add_argument("--calibration-copy", action="store_true",
                    help="first run one 256 MiB device copy (reference for hardware byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "single-GPU build: the benchmark runs on one GPU only; use --gpus 1"}))
        sys.exit(2)

    import torch
    import paper_2409_05734_amd as srpr
    import sr_inputs

    dev = torch.device("cuda:0")
    if args.calibration_copy:
        # one elementwise kernel that reads 256 MiB and writes 256 MiB
        src = torch.ones(64 * 1024 * 1024, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        torch.mul(src, 2.0, out=dst)
        torch.cuda.synchronize()
        del src, dst
    h = headline(torch, srpr, sr_inputs, dev, args.steps, args.warmup)
    cpu_args = h.pop("_cpu")
    out = {
        "metric": "GD iters/s (n=256^2, alpha=4, L=2)",
        "value": h["value"],
        "unit": "GD iters/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": h["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c64",
        "data": "synthetic",
        "config": {"workload": "2D image 256x256 -> 512x512 (alpha=4), L=2, Poisson 1000 photons, "
                               "one GD solve of 500 iterations per step", "n": 65536, "m": 262144, "layers": 2,
                   "gd_iters_per_step": GD_ITERS},
        "roofline": h["roofline"],
        "operator": h["operator"],
        "spectral_init": h["spectral_init"],
        "gd_iteration_us": h["gd_iteration_us"],
        "cosine_similarity": h["cosine_similarity"],
    }
    if not args.quick:
        extras = {}
        side = (("large_2d", large_2d), ("dense_baseline", dense), ("batched", batched),
                ("latency_floor", latency_floor), ("library_loop", library_loop), ("stacked_gd", stacked_gd), ("autograd", autograd), ("lds_resident_2d", lds_resident), ("forward_time_sweep", forward_time_sweep),
                ("layer_study", layer_study), ("poisson_loss", poisson_loss), ("tiny_1d", tiny_1d),
                ("accuracy_sweep", accuracy_sweep))
        on_request = {"accuracy_sweep"}  # about a minute of GPU time: run only when named
        wanted = None if args.extras == "all" else set(args.extras.split(","))
        for name, fn in side:
            if (wanted is None and name in on_request) or (wanted is not None and name not in wanted):
                continue
            t0 = time.perf_counter()
            try:
                extras[name] = fn(torch, srpr, sr_inputs, dev)
            except Exception as e:  # report, do not hide: the headline stays valid
                extras[name] = {"error": f"{type(e).__name__}: {e}"}
            extras[name]["wall_s"] = round(time.perf_counter() - t0, 2)
            torch.cuda.empty_cache()
        out["extras"] = extras
    if not args.quick and not args.no_cpu_baseline:
        d, y_h, x0_h, eta = cpu_args
        out["cpu_baseline"] = cpu_baseline(d, y_h, x0_h, eta)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
