"""The FFT lengths with a factor of three (96, 192, 384, 768) on their split
thread shape, where some threads of a transform hold no elements: every column
and row tile (and ones past the last transform), padded, trimmed and odd
windows, both loss epilogues with their traces, power iteration and both
derivatives, against the FP64 oracle; and plans of many such problems on the
level launches."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import aligned, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL_OP, TOL_IT = 2e-5, 1e-4

COLS = (2, 4, 8, 16, 258, 260, 264, 272)  # 256: single-buffered
ROWS = {96: (4, 16), 192: (2, 8), 384: (1, 4, 257, 260), 768: (1, 2, 257, 258)}


def _cases():
    out = []
    for M, rows in ROWS.items():
        for i, c in enumerate(COLS):
            out.append((M, c, rows[i % len(rows)], i % 2))
    return out


@pytest.mark.parametrize("M,col,row,table", _cases())
def test_split_tiles(gpu, M, col, row, table, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    monkeypatch.setenv("SR_TUNE_FORCE", f"{col},{row},{table}")
    rng = np.random.default_rng(M + col)
    # the length on the columns with 32-point rows, and on the rows of 16 columns' length
    for n_shape, m_shape, L in (((M // 2 - 3, 13), (M, 32), 2), ((9, M // 2 + 1), (16, M), 3), ((M, 16), (M - 7, 32), 1)):
        grid = tuple(max(a, b) for a, b in zip(n_shape, m_shape))
        th = sr_inputs.phase_masks(rng, L, grid)
        op = oracle.StructuredOperator(th, n_shape, m_shape)
        n, m = op.n, op.m
        x, gv = (sr_inputs.complex_gaussian(rng, n_shape) for _ in range(2))
        r, gz = (sr_inputs.complex_gaussian(rng, m_shape) for _ in range(2))
        plan = srpr.Plan([srpr.Problem(n_shape, m_shape, L)], th)
        dev = lambda a: to_dev(np.ascontiguousarray(a).ravel(), gpu)  # noqa: E731
        new = lambda k, t=torch.complex64: torch.empty(k, dtype=t, device=gpu)  # noqa: E731
        z, y, v = new(m), new(m, torch.float32), new(n)
        srpr.sr_forward(plan, dev(x), z, y)
        srpr.sr_adjoint(plan, dev(r), v)
        zr = op.A(x)
        assert rel_l2(to_host(z).reshape(m_shape), zr) <= TOL_OP
        assert rel_l2(to_host(y).reshape(m_shape), np.abs(zr) ** 2) <= 2 * TOL_OP
        assert rel_l2(to_host(v).reshape(n_shape), op.AH(r)) <= TOL_OP
        gx, gr, g1, g2 = new(n), new(m), torch.zeros(th.size, device=gpu), torch.zeros(th.size, device=gpu)
        srpr.sr_forward_vjp(plan, dev(x), dev(gz), gx, g1)
        srpr.sr_adjoint_vjp(plan, dev(r), dev(gv), gr, g2)
        gx_o, g1_o = oracle.forward_vjp(x, th, gz)
        gr_o, g2_o = oracle.adjoint_vjp(r, th, n_shape, gv, m_shape)
        for got, want in ((gx, gx_o), (gr, gr_o), (g1, g1_o), (g2, g2_o)):
            assert rel_l2(to_host(got).reshape(want.shape), want) <= TOL_IT
        if m < n:
            continue  # no solves on trimmed windows (trajectories there amplify rounding)
        yh = (np.abs(zr) ** 2).astype(np.float32)
        x0 = (x + 0.25 * sr_inputs.complex_gaussian(rng, n_shape)).astype(np.complex64)
        srpr.sr_spectral_init(plan, dev(yh), dev(x0), 3, -1.0, v)
        assert rel_l2(to_host(v).reshape(n_shape), oracle.spectral_init(op, yh, x0, 3, -1.0)) <= TOL_IT
        eps = float(0.1 * yh.mean())
        for loss, eta in (("l2", np.float32(oracle.default_step(op, yh, 0.1))), ("poisson", np.float32(0.05 * op.m))):
            if loss == "poisson":
                srpr.sr_plan_set_loss(plan, srpr.SR_LOSS_POISSON, eps)
            xd, lt = dev(x0), torch.zeros(4, device=gpu)
            srpr.sr_gd_solve(plan, dev(yh), xd, 4, eta, lt)
            xr, lr = oracle.gd_solve(op, yh, x0, 4, float(eta), return_loss=True, loss=loss, eps=eps)
            assert aligned(to_host(xd).reshape(n_shape), xr) <= TOL_IT
            assert np.max(np.abs(to_host(lt) - lr)) <= 1e-4 * np.abs(lr).max()


@pytest.mark.parametrize("count,streams", [(9, None), (120, None), (120, "1")])
def test_split_lengths_on_levels(gpu, count, streams, monkeypatch):
    """Uneven problems with such lengths beside powers of two, one to three
    layers (problems of fewer passes start at later levels; 120 of them have
    points enough for two groups on two streams)."""
    import torch
    import paper_2409_05734_amd as srpr
    if streams is not None:
        monkeypatch.setenv("SR_BATCH_STREAMS", streams)
    rng = np.random.default_rng(count)
    grids = [(96, 64), (192, 96), (64, 384), (384, 192), (128, 128), (32, 96), (384, 384), (16, 192), (256, 96)]
    shapes = [grids[i % len(grids)] for i in range(count)]
    layers = [1 + (i // 2) % 3 for i in range(count)]
    ns = [(g[0] // 2 - i % 3, g[1] // 2 + i % 2) for i, g in enumerate(shapes)]
    ths = [sr_inputs.phase_masks(rng, L, g) for L, g in zip(layers, shapes)]
    ops = [oracle.StructuredOperator(t, n) for t, n in zip(ths, ns)]
    xs = [sr_inputs.complex_gaussian(rng, n) for n in ns]
    ys = [(np.abs(o.A(x)) ** 2).astype(np.float32) for o, x in zip(ops, xs)]
    x0 = [(x + 0.25 * sr_inputs.complex_gaussian(rng, x.shape)).astype(np.complex64) for x in xs]
    eta = np.array([oracle.default_step(o, y, 0.05) for o, y in zip(ops, ys)], np.float32)
    plan = srpr.Plan([srpr.Problem(n, g, L) for n, g, L in zip(ns, shapes, layers)],
                     np.concatenate([t.ravel() for t in ths]))
    cat = lambda a: to_dev(np.concatenate([v.ravel() for v in a]), gpu)  # noqa: E731
    y, xd = cat(ys), cat(x0)
    sp = torch.empty_like(xd)
    srpr.sr_spectral_init(plan, y, xd, 5, -1.0, sp)
    srpr.sr_gd_solve(plan, y, xd, 7, eta)
    srpr.sr_plan_sync(plan)
    xh, sh = to_host(xd), to_host(sp)
    for i in range(count):
        sl = slice(plan.x_off[i], plan.x_off[i + 1])
        assert rel_l2(sh[sl].reshape(ns[i]), oracle.spectral_init(ops[i], ys[i], x0[i], 5, -1.0)) <= TOL_IT
        assert aligned(xh[sl].reshape(ns[i]), oracle.gd_solve(ops[i], ys[i], x0[i], 7, float(eta[i]))) <= TOL_IT
