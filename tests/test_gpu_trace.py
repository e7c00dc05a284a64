"""Loss traces of long GD solves: iterations write their loss partials to rows
that are summed once per chunk of 50, from replayed graphs where the solve is
long enough.  Lengths around the chunk and its remainder, single problems,
stacks and traces beside an untraced solve, against the schedule that launches
every pass directly (bit for bit) and the FP64 oracle; and a change of loss
between solves on the same buffers and step."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import aligned, to_dev, to_host

pytestmark = pytest.mark.gpu


def _setup(rng, n_shape, m_shape, L, B, dev):
    import paper_2409_05734_amd as srpr
    ths = [sr_inputs.phase_masks(rng, L, m_shape) for _ in range(B)]
    ops = [oracle.StructuredOperator(t, n_shape) for t in ths]
    xs = [sr_inputs.complex_gaussian(rng, n_shape) for _ in range(B)]
    ys = [(np.abs(o.A(x)) ** 2).astype(np.float32) for o, x in zip(ops, xs)]
    x0 = [(x + 0.5 * sr_inputs.complex_gaussian(rng, n_shape)).astype(np.complex64) for x in xs]
    blk = L * int(np.prod(m_shape))
    plan = srpr.Plan([srpr.Problem(n_shape, m_shape, L, theta_offset=b * blk) for b in range(B)],
                     np.concatenate([t.ravel() for t in ths]))
    return plan, ops, ys, x0


@pytest.mark.parametrize("B,iters", [(1, 1), (1, 49), (1, 51), (1, 59), (1, 60), (1, 109), (3, 50), (3, 111)])
def test_trace_chunks(gpu, B, iters):
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(iters + B)
    n_shape, m_shape, L = (20, 24), (96, 64) if B == 1 else (64, 64), 2
    plan, ops, ys, x0 = _setup(rng, n_shape, m_shape, L, B, gpu)
    y = to_dev(np.concatenate([v.ravel() for v in ys]), gpu)
    start = np.concatenate([v.ravel() for v in x0])
    eta = np.array([oracle.default_step(o, v, 0.1) for o, v in zip(ops, ys)], np.float32)
    out = []
    for sched in (srpr.SR_SCHED_AUTO, srpr.SR_SCHED_LOOP, srpr.SR_SCHED_AUTO):
        srpr.sr_plan_set_schedule(plan, sched)
        x = to_dev(start, gpu)
        lt = torch.full((iters * B,), -1.0, dtype=torch.float32, device=gpu)
        srpr.sr_gd_solve(plan, y, x, iters, eta, lt)
        srpr.sr_plan_sync(plan)
        out.append((x.clone(), lt.clone()))
        srpr.sr_gd_solve(plan, y, x, iters, eta)  # an untraced solve between
    for x, lt in out[1:]:
        assert torch.equal(x, out[0][0]) and torch.equal(lt, out[0][1])
    lt = to_host(out[0][1]).reshape(B, iters)
    for b in range(B):
        xr, lr = oracle.gd_solve(ops[b], ys[b], x0[b], iters, float(eta[b]), return_loss=True)
        assert aligned(to_host(out[0][0]).reshape(B, *n_shape)[b], xr) <= 1e-4
        assert np.max(np.abs(lt[b] - lr)) <= 1e-4 * lr[0]


@pytest.mark.parametrize("B", [1, 2, 9])
def test_loss_change_on_the_same_buffers(gpu, B):
    """60 steps on the l2 loss, then 60 on the Poisson loss with the same
    buffers and step: the second solve descends the second loss."""
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(B)
    n_shape, m_shape, L = (16, 20), (32, 64), 2
    plan, ops, ys, x0 = _setup(rng, n_shape, m_shape, L, B, gpu)
    if B == 9:
        srpr.sr_plan_set_schedule(plan, srpr.SR_SCHED_BATCHED)
    y = to_dev(np.concatenate([v.ravel() for v in ys]), gpu)
    eta = np.full(B, 0.05 * ops[0].m, np.float32)
    eps = float(0.1 * np.mean(ys[0]))
    x = to_dev(np.concatenate([v.ravel() for v in x0]), gpu)
    start = x.clone()
    srpr.sr_gd_solve(plan, y, x, 60, eta)
    srpr.sr_plan_set_loss(plan, srpr.SR_LOSS_POISSON, eps)
    x.copy_(start)
    srpr.sr_gd_solve(plan, y, x, 60, eta)
    srpr.sr_plan_sync(plan)
    xh = to_host(x).reshape(B, *n_shape)
    for b in range(B):
        xr = oracle.gd_solve(ops[b], ys[b], x0[b], 60, float(eta[b]), loss="poisson", eps=eps)
        assert aligned(xh[b], xr) <= 1e-4
