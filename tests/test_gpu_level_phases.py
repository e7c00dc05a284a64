"""Where the level launches take their phase diagonals from: polynomials up to
kPhasePolyMax, the exp(i theta) tables past it (phases of any size stay phases)
and everywhere when the phase source is pinned to the tables."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import aligned, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

SHAPES = [((24, 20), (64, 32), 2), ((40, 90), (96, 192), 3), ((30, 30), (64, 64), 1)]


def _plan(srpr, ths, shapes):
    plan = srpr.Plan([srpr.Problem(n, m, L) for n, m, L in shapes], np.concatenate([t.ravel() for t in ths]))
    srpr.sr_plan_set_schedule(plan, srpr.SR_SCHED_BATCHED)
    return plan


@pytest.mark.parametrize("via", ("create", "set_theta"))
def test_phases_of_any_size(gpu, via):
    """A problem of phases up to 10^9, one on both sides of the line between
    polynomials and tables, one of ordinary phases with a few huge ones."""
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(21)
    ths = [rng.uniform(-span, span, (L,) + m).astype(np.float32)
           for (_, m, L), span in zip(SHAPES, (1e9, 2.0 * 131072, 2 * np.pi))]
    ths[2].ravel()[::97] = 3e7
    plan = _plan(srpr, ths if via == "create" else [np.zeros_like(t) for t in ths], SHAPES)
    if via == "set_theta":
        srpr.sr_plan_set_theta(plan, to_dev(np.concatenate([t.ravel() for t in ths]), gpu))
    ops = [oracle.StructuredOperator(t, n) for t, (n, _, _) in zip(ths, SHAPES)]
    x, gv = ([sr_inputs.complex_gaussian(rng, n) for n, _, _ in SHAPES] for _ in range(2))
    r, gz = ([sr_inputs.complex_gaussian(rng, m) for _, m, _ in SHAPES] for _ in range(2))
    dev = {k: to_dev(np.concatenate([a.ravel() for a in v]), gpu) for k, v in dict(x=x, gv=gv, r=r, gz=gz).items()}
    z, v, gx, gr = (torch.empty_like(dev[k]) for k in ("r", "x", "x", "r"))
    y = torch.empty(plan.m_total, device=gpu)
    g1, g2 = (torch.zeros(plan.theta_len, device=gpu) for _ in range(2))
    srpr.sr_forward(plan, dev["x"], z, y)
    srpr.sr_adjoint(plan, dev["r"], v)
    srpr.sr_forward_vjp(plan, dev["x"], dev["gz"], gx, g1)
    srpr.sr_adjoint_vjp(plan, dev["r"], dev["gv"], gr, g2)
    eta = np.array([oracle.default_step(op, np.abs(op.A(a)) ** 2, 0.05) for op, a in zip(ops, x)], np.float32)
    xg = to_dev(np.concatenate([0.8 * a.ravel() for a in x]).astype(np.complex64), gpu)
    est = torch.empty_like(xg)
    srpr.sr_gd_solve(plan, y, xg, 3, eta)
    srpr.sr_spectral_init(plan, y, dev["gv"], 3, -1.0, est)
    srpr.sr_plan_sync(plan)
    yh, t0 = to_host(y), 0
    for i, (n, m, L) in enumerate(SHAPES):
        xs, ys = slice(plan.x_off[i], plan.x_off[i + 1]), slice(plan.y_off[i], plan.y_off[i + 1])
        th = ths[i].astype(np.float64)
        fgx, fgt = oracle.forward_vjp(x[i], th, gz[i])
        agr, agt = oracle.adjoint_vjp(r[i], th, n, gv[i], m)
        yi = yh[ys].reshape(m)
        for got, want, shape, tol in ((z[ys], ops[i].A(x[i]), m, 2e-5), (v[xs], ops[i].AH(r[i]), n, 2e-5),
                                      (gx[xs], fgx, n, 1e-4), (gr[ys], agr, m, 1e-4),
                                      (g1[t0:t0 + th.size], fgt, th.shape, 1e-4),
                                      (g2[t0:t0 + th.size], agt, th.shape, 1e-4)):
            assert rel_l2(to_host(got).reshape(shape), want) <= tol, i
        xr = oracle.gd_solve(ops[i], yi, (0.8 * x[i]).astype(np.complex64), 3, float(eta[i]))
        assert aligned(to_host(xg)[xs].reshape(n), xr) <= 1e-4, i
        assert rel_l2(to_host(est)[xs].reshape(n), oracle.spectral_init(ops[i], yi, gv[i], 3, -1.0)) <= 1e-4, i
        t0 += th.size


@pytest.mark.parametrize("env,table", [({}, False), ({"SR_PHASE_TABLE": "1"}, True), ({"SR_TUNE_FORCE": "8,1,1"}, True),
                                       ({"SR_PHASE_TABLE": "0"}, False), ({"SR_TUNE_FORCE": "8,1,0"}, False)])
def test_pinned_source(gpu, env, table, monkeypatch):
    """All phases are the one where the polynomials are worst (1.54e-7 off;
    sincosf, which fills the tables, is within half an ulp of 1, 6e-8): A x is
    then that phase times F U x, and their inner product averages the
    transforms' rounding away (1e-7 over the square root of the points)."""
    import torch
    import paper_2409_05734_amd as srpr
    for k in ("SR_TUNE_FORCE", "SR_PHASE_TABLE", "SR_TUNE"):
        monkeypatch.delenv(k, raising=False)
    for k, val in env.items():
        monkeypatch.setenv(k, val)
    t = np.float32(1.57088029)
    shapes = [((30, 30), (64, 64), 1), ((20, 30), (64, 256), 1), ((50, 60), (256, 64), 1)]  # scales 1/sqrt(M) exact
    rng = np.random.default_rng(22)
    plan = _plan(srpr, [np.full((1,) + m, t, np.float32) for _, m, _ in shapes], shapes)
    x = [sr_inputs.complex_gaussian(rng, n) for n, _, _ in shapes]
    z = torch.empty(plan.m_total, dtype=torch.complex64, device=gpu)
    srpr.sr_forward(plan, to_dev(np.concatenate([a.ravel() for a in x]), gpu), z, None)
    srpr.sr_plan_sync(plan)
    for i, (n, m, _) in enumerate(shapes):
        fux = oracle.forward(x[i], np.zeros((1,) + m), m).ravel()
        got = to_host(z)[plan.y_off[i]:plan.y_off[i + 1]].astype(np.complex128)
        off = abs(np.vdot(fux, got) / np.vdot(fux, fux) - np.exp(1j * float(t)))
        assert off <= 8e-8 if table else 1.2e-7 <= off <= 2e-7, (i, off)
