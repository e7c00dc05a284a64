"""GD on a stack in two parts on streams of their own: the same arithmetic per
problem as in one part, so the same bits, for even and odd counts, own and shared
phases, both losses, with and without a trace, direct launches, captured chunks
and the caller's own capture; and beside other work on the stream."""
import numpy as np
import pytest

import sr_inputs
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

GRID, N = (64, 128), (30, 64)


def _setup(gpu, P, shared, L=2, stream=None):
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(P)
    th = sr_inputs.phase_masks(rng, L if shared else L * P, GRID)
    k = L * GRID[0] * GRID[1]
    plan = srpr.Plan([srpr.Problem(N, GRID, L, theta_offset=0 if shared else i * k) for i in range(P)], th.ravel(),
                     stream=stream)
    x0 = to_dev(sr_inputs.complex_gaussian(rng, (P,) + N).ravel(), gpu)
    y = torch.empty(P * GRID[0] * GRID[1], device=gpu)
    srpr.sr_forward(plan, to_dev(sr_inputs.complex_gaussian(rng, (P,) + N).ravel(), gpu), None, y)
    return plan, x0, y


@pytest.mark.parametrize("P,shared", [(2, False), (5, False), (5, True), (16, True)])
@pytest.mark.parametrize("iters", (1, 3, 64))
@pytest.mark.parametrize("loss,trace", [("l2", False), ("l2", True), ("poisson", True)])
def test_same_as_one_part(gpu, P, shared, iters, loss, trace, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    plan, x0, y = _setup(gpu, P, shared)
    if loss == "poisson":
        srpr.sr_plan_set_loss(plan, srpr.SR_LOSS_POISSON, 0.1)
    eta = np.linspace(0.01, 0.05, P).astype(np.float32) * (1 if loss == "l2" else GRID[0] * GRID[1])
    outs = []
    for parts in ("1", "2", "2"):  # (the third on the graphs captured by the second)
        monkeypatch.setenv("SR_STACK_PARTS", parts)
        if len(outs) < 2:
            x = torch.empty_like(x0)
        x.copy_(x0)
        tr = torch.zeros(P * iters, device=gpu) if trace else None
        srpr.sr_gd_solve(plan, y, x, iters, eta, tr)
        x.mul_(1)  # the caller's next work on the stream
        outs.append((x.clone(), tr))
    srpr.sr_plan_sync(plan)
    for x, tr in outs[1:]:
        assert torch.equal(torch.view_as_real(x), torch.view_as_real(outs[0][0]))
        assert tr is None or torch.equal(tr, outs[0][1])


@pytest.mark.parametrize("P,shared", [(2, False), (5, False), (16, True)])
@pytest.mark.parametrize("iters", (0, 1, 2, 64))
def test_power_iteration(gpu, P, shared, iters, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    monkeypatch.setenv("SR_TUNE_FORCE", "4,1,0")  # tiles that hold whole problems
    plan, x0, y = _setup(gpu, P, shared)
    outs = []
    for parts in ("1", "2"):
        monkeypatch.setenv("SR_STACK_PARTS", parts)
        x = torch.empty_like(x0)
        srpr.sr_spectral_init(plan, y, x0, iters, -1.0, x)
        outs.append(torch.view_as_real(x))
    srpr.sr_plan_sync(plan)
    assert torch.equal(*outs)


def test_captured(gpu, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    monkeypatch.setenv("SR_STACK_PARTS", "2")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        plan, x0, y = _setup(gpu, 5, False, stream=stream)
        x = x0.clone()
        srpr.sr_gd_solve(plan, y, x, 6, 0.02)
        want = x.clone()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            srpr.sr_gd_solve(plan, y, x, 6, 0.02)
        for _ in range(3):
            x.copy_(x0)
            graph.replay()
            stream.synchronize()
            assert torch.equal(torch.view_as_real(x), torch.view_as_real(want))


def test_rule_takes_two_parts(gpu, monkeypatch):
    """Points enough for two parts by themselves: as in one."""
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(1)
    P, grid, n = 62, (256, 256), (128, 100)
    th = sr_inputs.phase_masks(rng, 1, grid)
    plan = srpr.Plan([srpr.Problem(n, grid, 1, theta_offset=0) for _ in range(P)], th.ravel())
    x0 = to_dev(sr_inputs.complex_gaussian(rng, (P,) + n).ravel(), gpu)
    y = torch.rand(P * grid[0] * grid[1], device=gpu)
    outs = []
    for parts in (None, "1"):
        if parts is None:
            monkeypatch.delenv("SR_STACK_PARTS", raising=False)
        else:
            monkeypatch.setenv("SR_STACK_PARTS", parts)
        x = x0.clone()
        srpr.sr_gd_solve(plan, y, x, 4, 0.02)
        srpr.sr_plan_sync(plan)
        outs.append(torch.view_as_real(x))
    assert torch.equal(*outs)
