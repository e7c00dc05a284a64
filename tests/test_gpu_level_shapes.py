"""The level launches' solvers on both thread shapes (SR_BATCH_EV pins one),
every length, both losses, traces, and power iteration, against the oracle; and
plans on both sides of the rule that picks the shape: the same bits as the shape
that it says."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import aligned, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

LENS = (16, 32, 64, 96, 128, 192, 256, 384, 512)


def _plan(srpr, shapes, rng):
    ths = [sr_inputs.phase_masks(rng, L, m) for _, m, L in shapes]
    plan = srpr.Plan([srpr.Problem(*s) for s in shapes], np.concatenate([t.ravel() for t in ths]))
    srpr.sr_plan_set_schedule(plan, srpr.SR_SCHED_BATCHED)
    return plan, ths


@pytest.mark.parametrize("ev", ("0", "1"))
def test_lengths(gpu, ev, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    monkeypatch.setenv("SR_BATCH_EV", ev)
    rng = np.random.default_rng(41)
    shapes = [((max(2, a // 3), b // 2 - 1), (a, b), 1 + i % 3) for i, (a, b) in enumerate(zip(LENS, LENS[3:] + LENS[:3]))]
    plan, ths = _plan(srpr, shapes, rng)
    ops = [oracle.StructuredOperator(t, n) for t, (n, _, _) in zip(ths, shapes)]
    xs = [sr_inputs.complex_gaussian(rng, n) for n, _, _ in shapes]
    ys = [(np.abs(op.A(x)) ** 2).astype(np.float32) for op, x in zip(ops, xs)]
    x0 = [(x + 0.2 * sr_inputs.complex_gaussian(rng, x.shape)).astype(np.complex64) for x in xs]
    yd, xd = (to_dev(np.concatenate([a.ravel() for a in v]), gpu) for v in (ys, x0))
    eps = 0.1
    for loss, etas in (("l2", [oracle.default_step(op, y, 0.1) for op, y in zip(ops, ys)]), ("poisson", [0.05 * op.m for op in ops])):
        if loss == "poisson":
            srpr.sr_plan_set_loss(plan, srpr.SR_LOSS_POISSON, eps)
        etas = np.array(etas, np.float32)
        got = []
        for tr in (torch.zeros(4 * len(shapes), device=gpu), None):
            x = xd.clone()
            srpr.sr_gd_solve(plan, yd, x, 4, etas, tr)
            got.append((to_host(x), None if tr is None else to_host(tr).reshape(-1, 4)))
        srpr.sr_plan_sync(plan)
        assert np.array_equal(got[0][0], got[1][0])
        for i, (n, _, _) in enumerate(shapes):
            want, lr = oracle.gd_solve(ops[i], ys[i], x0[i], 4, float(etas[i]), return_loss=True, loss=loss, eps=eps)
            assert aligned(got[0][0][plan.x_off[i]:plan.x_off[i + 1]].reshape(n), want) <= 1e-4, (loss, i)
            assert np.max(np.abs(got[0][1][i] - lr)) <= 1e-4 * np.abs(lr).max(), (loss, i)
    est = torch.empty_like(xd)
    for k in (1, 4):
        srpr.sr_spectral_init(plan, yd, xd, k, -1.0, est)
        srpr.sr_plan_sync(plan)
        for i, (n, _, _) in enumerate(shapes):
            want = oracle.spectral_init(ops[i], ys[i], x0[i], k, -1.0)
            assert rel_l2(to_host(est)[plan.x_off[i]:plan.x_off[i + 1]].reshape(n), want) <= 1e-4, (k, i)


# 18 of 128 x 128 (0.29M points), 19 (0.31M, none above 65536 points), 73 and 74
# (either side of 1.2M), 2 of 512 x 256 (0.26M), 3 (0.39M, above 65536 points each)
@pytest.mark.parametrize("grid,P,narrow", [((128, 128), 18, True), ((128, 128), 19, True), ((128, 128), 73, True),
                                           ((128, 128), 74, False), ((512, 256), 2, True), ((512, 256), 3, False)])
def test_rule(gpu, grid, P, narrow, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    outs = []
    for ev in (None, "1", "0"):
        if ev is None:
            monkeypatch.delenv("SR_BATCH_EV", raising=False)
        else:
            monkeypatch.setenv("SR_BATCH_EV", ev)
        monkeypatch.setenv("SR_STACK", "0")
        rng = np.random.default_rng(P)
        plan, _ = _plan(srpr, [((20, 30), grid, 2)] * P, rng)
        x = to_dev(sr_inputs.complex_gaussian(rng, (P, 20, 30)).ravel(), gpu)
        y = torch.empty(plan.m_total, device=gpu)
        srpr.sr_forward(plan, x, None, y)
        x *= 0.9
        tr = torch.zeros(3 * P, device=gpu)
        srpr.sr_gd_solve(plan, y, x, 3, 0.01, tr)
        est = torch.empty_like(x)
        monkeypatch.setenv("SR_BATCH_EV", "0" if ev == "1" else "1")  # (a plan keeps the shape that it took)
        srpr.sr_spectral_init(plan, y, x, 3, -1.0, est)
        srpr.sr_plan_sync(plan)
        outs.append([torch.view_as_real(x), tr, torch.view_as_real(est)])
    assert all(torch.equal(a, b) for a, b in zip(outs[0], outs[1 if narrow else 2]))
    assert not torch.equal(outs[1][1], outs[2][1])
