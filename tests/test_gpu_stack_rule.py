"""Stacks on both sides of the rule that runs them in two parts by itself (no
override): 62 problems on 256 x 256 grids, 16 iterations and one less, gradient
descent with and without a trace and power iteration, bit for bit as in one
part.  That the rule takes these counts as it is said here is asserted on the
host (csrc/host_check.cpp, stack_rule_checks)."""
import numpy as np
import pytest

import sr_inputs
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

P, GRID, N = 62, (256, 256), (128, 100)


def _setup(gpu, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    monkeypatch.setenv("SR_TUNE_FORCE", "4,1,0")  # tiles that hold whole problems
    rng = np.random.default_rng(12)
    th = sr_inputs.phase_masks(rng, 2, GRID)
    plan = srpr.Plan([srpr.Problem(N, GRID, 2, theta_offset=0) for _ in range(P)], th.ravel())
    x0 = to_dev(sr_inputs.complex_gaussian(rng, (P,) + N).ravel(), gpu)
    y = torch.empty(P * GRID[0] * GRID[1], device=gpu)
    srpr.sr_forward(plan, to_dev(sr_inputs.complex_gaussian(rng, (P,) + N).ravel(), gpu), None, y)
    return plan, x0, y


def _parts(monkeypatch, solve):
    outs = []
    for parts in (None, "1"):
        if parts is None:
            monkeypatch.delenv("SR_STACK_PARTS", raising=False)
        else:
            monkeypatch.setenv("SR_STACK_PARTS", parts)
        outs.append(solve())
    return outs


@pytest.mark.parametrize("trace", (False, True))
@pytest.mark.parametrize("iters", (15, 16))
def test_gd(gpu, iters, trace, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    plan, x0, y = _setup(gpu, monkeypatch)
    eta = np.linspace(0.01, 0.05, P).astype(np.float32)

    def solve():
        x = x0.clone()
        tr = torch.zeros(P * iters, device=gpu)
        srpr.sr_gd_solve(plan, y, x, iters, eta, tr if trace else None)
        srpr.sr_plan_sync(plan)
        return torch.view_as_real(x), tr

    (xa, ta), (xb, tb) = _parts(monkeypatch, solve)
    assert torch.equal(xa, xb) and torch.equal(ta, tb)


@pytest.mark.parametrize("iters", (15, 16))
def test_power_iteration(gpu, iters, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    plan, x0, y = _setup(gpu, monkeypatch)

    def solve():
        x = torch.empty_like(x0)
        srpr.sr_spectral_init(plan, y, x0, iters, -1.0, x)
        srpr.sr_plan_sync(plan)
        return torch.view_as_real(x)

    assert torch.equal(*_parts(monkeypatch, solve))
