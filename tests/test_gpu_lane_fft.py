"""One-dimensional problems on the transforms with an element a lane: every
length that has them, L = 1 to 4, whole, odd and single-entry windows of signal
and measurements, A, A^H, both derivatives, GD under both losses and power
iteration, one problem and several of mixed lengths, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import aligned, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

# a transform is at most ten roundings deep a step of 6e-8, two a layer and
# another for each diagonal: 4e-6 of the norm with all errors of one sign at
# L = 4; solves as elsewhere
TOL_OP, TOL_IT = 4e-6, 1e-4
LENGTHS = (64, 128, 192, 256, 384, 512, 768)


def _dev(a, gpu):
    return to_dev(np.ascontiguousarray(a).ravel(), gpu)


@pytest.mark.parametrize("M", LENGTHS)
@pytest.mark.parametrize("L", (1, 2, 3, 4))
def test_operator_and_derivatives(gpu, M, L):
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(10 * M + L)
    for n, m in ((M, M), (M // 2 - 3, M), (M, M - 5), (1, M), (M, 1)):
        th = sr_inputs.phase_masks(rng, L, (M,))
        op = oracle.StructuredOperator(th, (n,), (m,))
        x, gv = (sr_inputs.complex_gaussian(rng, (n,)) for _ in range(2))
        r, gz = (sr_inputs.complex_gaussian(rng, (m,)) for _ in range(2))
        plan = srpr.Plan([srpr.Problem((n,), (m,), L)], th)
        new = lambda k, t=torch.complex64: torch.empty(k, dtype=t, device=gpu)  # noqa: E731
        z, y, v = new(m), new(m, torch.float32), new(n)
        srpr.sr_forward(plan, _dev(x, gpu), z, y)
        srpr.sr_adjoint(plan, _dev(r, gpu), v)
        zr = op.A(x)
        assert rel_l2(to_host(z), zr) <= TOL_OP
        assert rel_l2(to_host(y), np.abs(zr) ** 2) <= 2 * TOL_OP
        assert rel_l2(to_host(v), op.AH(r)) <= TOL_OP
        gx, gr = new(n), new(m)
        g1, g2 = (torch.zeros(th.size, device=gpu) for _ in range(2))
        srpr.sr_forward_vjp(plan, _dev(x, gpu), _dev(gz, gpu), gx, g1)
        srpr.sr_adjoint_vjp(plan, _dev(r, gpu), _dev(gv, gpu), gr, g2)
        gx_o, g1_o = oracle.forward_vjp(x, th, gz)
        gr_o, g2_o = oracle.adjoint_vjp(r, th, (n,), gv, (m,))
        for got, want in ((gx, gx_o), (gr, gr_o), (g1, g1_o), (g2, g2_o)):
            assert rel_l2(to_host(got).reshape(want.shape), want) <= TOL_IT


@pytest.mark.parametrize("loss", ("l2", "poisson"))
@pytest.mark.parametrize("count", (1, 9))
@pytest.mark.parametrize("first", LENGTHS)
def test_solvers(gpu, loss, count, first):
    """(lengths in turn from `first`, among them two that have no such transforms)"""
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(first + count)
    turn = LENGTHS[LENGTHS.index(first):] + (96, 32) + LENGTHS[:LENGTHS.index(first)]
    shapes = [(turn[i] // (2 + i % 3), turn[i]) for i in range(count)]
    ths = [sr_inputs.phase_masks(rng, 2, (m,)) for _, m in shapes]
    ops = [oracle.StructuredOperator(t, (n,)) for (n, m), t in zip(shapes, ths)]
    xs = [sr_inputs.complex_gaussian(rng, (n,)) for n, _ in shapes]
    ys = [(np.abs(op.A(x)) ** 2).astype(np.float32) for op, x in zip(ops, xs)]
    x0 = [(x + 0.25 * sr_inputs.complex_gaussian(rng, x.shape)).astype(np.complex64) for x in xs]
    plan = srpr.Plan([srpr.Problem((n,), (m,), 2) for n, m in shapes], np.concatenate([t.ravel() for t in ths]))
    eps = 0.1
    if loss == "poisson":
        srpr.sr_plan_set_loss(plan, srpr.SR_LOSS_POISSON, eps)
        eta = np.array([0.05 * op.m for op in ops], np.float32)
    else:
        eta = np.array([oracle.default_step(op, y, 0.1) for op, y in zip(ops, ys)], np.float32)
    y, x = _dev(np.concatenate(ys), gpu), _dev(np.concatenate(x0), gpu)
    sp, tr = torch.empty_like(x), torch.empty(4 * count, device=gpu)
    srpr.sr_spectral_init(plan, y, x, 3, -1.0, sp)
    srpr.sr_gd_solve(plan, y, x, 4, eta, tr)
    srpr.sr_plan_sync(plan)
    for i in range(count):
        sl = slice(plan.x_off[i], plan.x_off[i + 1])
        assert rel_l2(to_host(sp)[sl], oracle.spectral_init(ops[i], ys[i], x0[i], 3, -1.0)) <= TOL_IT
        xr, lr = oracle.gd_solve(ops[i], ys[i], x0[i], 4, float(eta[i]), return_loss=True, loss=loss, eps=eps)
        assert aligned(to_host(x)[sl], xr) <= TOL_IT
        assert np.max(np.abs(to_host(tr)[4 * i:4 * i + 4] - lr)) <= 1e-4 * np.abs(lr).max()
