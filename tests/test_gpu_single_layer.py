"""L = 1, where the turnaround reads and writes compact rows: whole cache lines
(48 columns, in place) and not (50, from one buffer to the other), by itself, past
a graph chunk, without allocation, traced, and against a stack of the same
problem (in place on either)."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import aligned, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n2", (48, 50))
def test_solves(gpu, n2, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    monkeypatch.setenv("SR_TUNE_FORCE", "2,4,1")
    n, grid = (60, n2), (128, 256)
    rng = np.random.default_rng(n2)
    th = sr_inputs.phase_masks(rng, 1, grid)
    op = oracle.StructuredOperator(th, n)
    xs = sr_inputs.complex_gaussian(rng, n)
    y = (np.abs(op.A(xs)) ** 2).astype(np.float32)
    x0 = (xs + 0.2 * sr_inputs.complex_gaussian(rng, n)).astype(np.complex64)
    eta = float(np.float32(oracle.default_step(op, y, 0.1)))
    one = srpr.Plan([srpr.Problem(n, grid, 1)], th.ravel())
    two = srpr.Plan([srpr.Problem(n, grid, 1, theta_offset=0)] * 2, th.ravel())
    yd, xd = to_dev(y.ravel(), gpu), to_dev(x0.ravel(), gpu)

    def gd(plan, k, f=srpr.sr_gd_solve, trace=None):
        p = plan.nprob
        x = xd.repeat(p)
        f(plan, yd.repeat(p), x, k, eta, *([trace] if trace is not None else []))
        srpr.sr_plan_sync(plan)
        return torch.view_as_real(x).view(p, -1)

    for k in (1, 4, 70):
        got = gd(one, k)
        assert all(torch.equal(got[0], row) for row in gd(two, k)), k
    tr = torch.zeros(4, device=gpu)
    x4 = gd(one, 4, trace=tr)
    assert torch.equal(x4, gd(one, 4)) and torch.equal(x4, gd(one, 4, srpr.sr_gd_solve_noalloc))
    want, loss = oracle.gd_solve(op, y, x0, 4, eta, return_loss=True)
    assert aligned(to_host(torch.view_as_complex(x4.view(-1, 2))).reshape(n), want) <= 1e-4
    assert np.max(np.abs(to_host(tr) - loss)) <= 1e-4 * np.abs(loss).max()
    for k in (1, 5, 60):
        est = torch.empty_like(xd)
        srpr.sr_spectral_init(one, yd, xd, k, -1.0, est)
        srpr.sr_plan_sync(one)
        if k < 60:
            assert rel_l2(to_host(est).reshape(n), oracle.spectral_init(op, y, x0, k, -1.0)) <= 1e-4, k
        both = torch.empty(2 * xd.numel(), dtype=torch.complex64, device=gpu)
        srpr.sr_spectral_init(two, yd.repeat(2), xd.repeat(2), k, -1.0, both)
        srpr.sr_plan_sync(two)
        assert all(torch.equal(torch.view_as_real(est), torch.view_as_real(b)) for b in both.view(2, -1)), k
