"""The dense products in bf16 parts: tiles and splits with remainders in every
direction, both epilogue kinds, operands far from 1, infinities and NaN, and the
shapes it leaves to the FP32 products, against FP64 and the FP32 products."""
import numpy as np
import pytest

from gpu_helpers import rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

# the parts hold every bit, and a reduction of K adds 6 K/32 times: errors of
# 6e-8 of random sign leave sqrt(6 K / 32) 6e-8 <= 1.7e-6 of the norm at K = 4200;
# |z|^2 and the solvers' updates carry twice that
TOL = 2e-6


def _plan(srpr, A, nb, force, monkeypatch):
    monkeypatch.setenv("SR_DENSE_GEMM", force)
    m, n = A.shape
    return srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(nb)], None, dense_A=A)


def _cn(rng, *shape):
    return ((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.5 ** 0.5).astype(np.complex64)


def _apply(srpr, torch, plan, X, R, gpu):
    z = torch.full((R.size,), 3.0, dtype=torch.complex64, device=gpu)
    y = torch.full((R.size,), 3.0, device=gpu)
    v = torch.full((X.size,), 3.0, dtype=torch.complex64, device=gpu)
    srpr.sr_forward(plan, to_dev(X.ravel(), gpu), z, y)
    srpr.sr_adjoint(plan, to_dev(R.ravel(), gpu), v)
    return to_host(z).reshape(R.shape), to_host(y).reshape(R.shape), to_host(v).reshape(X.shape)


@pytest.mark.parametrize("m,n,nb", [
    (1, 2, 1), (31, 16, 1), (33, 18, 33), (256, 128, 32), (257, 130, 31), (255, 126, 65), (1025, 34, 5),
    (100, 2100, 7), (2100, 258, 64), (4200, 46, 12), (5000, 1026, 9)])
def test_operator(gpu, m, n, nb, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(m + n + nb)
    A, X, R = _cn(rng, m, n), _cn(rng, nb, n), _cn(rng, nb, m)
    z, y, v = _apply(srpr, torch, _plan(srpr, to_dev(A, gpu), nb, "bf16", monkeypatch), X, R, gpu)
    A6 = A.astype(np.complex128)
    zr, vr = X @ A6.T, R @ A6.conj()
    assert rel_l2(z, zr) <= TOL
    assert rel_l2(y, np.abs(zr) ** 2) <= 2 * TOL
    assert rel_l2(v, vr) <= TOL


@pytest.mark.parametrize("sa,sx", [(1.0, 1e-36), (1e-36, 1.0), (1e-18, 1e-17), (1e20, 1e-20), (1e25, 1e10), (1.0, 1e37)])
def test_scales(gpu, sa, sx, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(3)
    A, X, R = _cn(rng, 300, 66) * np.float32(sa), _cn(rng, 6, 66) * np.float32(sx), _cn(rng, 6, 300) * np.float32(sx)
    z, _, v = _apply(srpr, torch, _plan(srpr, to_dev(A, gpu), 6, "bf16", monkeypatch), X, R, gpu)
    A6 = A.astype(np.complex128)
    for got, want in ((z, X @ A6.T), (v, R @ A6.conj())):
        got, want = got.astype(np.complex128).view(np.float64), want.view(np.float64)
        over = np.abs(want) > np.finfo(np.float32).max  # no FP32 value
        assert np.array_equal(~np.isfinite(got), over)
        assert rel_l2(got[~over] / (sa * sx), want[~over] / (sa * sx)) <= TOL


def test_nonfinite(gpu, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(4)
    A, X, R = _cn(rng, 300, 66), _cn(rng, 6, 66), _cn(rng, 6, 300)
    A[7, 3], A[9, 4] = np.inf, 3.4e38
    X[1, 5], X[2, 6], X[3, 1] = np.inf, 3.4e38, np.nan
    R[1, 5], R[2, 6], R[3, 1] = complex(0, -np.inf), -3.4e38, np.nan
    outs = [_apply(srpr, torch, _plan(srpr, to_dev(A, gpu), 6, f, monkeypatch), X, R, gpu) for f in ("bf16", "own")]
    for a, b in zip(*outs):
        a, b = (np.ascontiguousarray(t).view(np.float32) for t in (a, b))
        assert np.array_equal(np.isfinite(a), np.isfinite(b))
        assert np.array_equal(np.isnan(a), np.isnan(b))
        ok = np.isfinite(b)
        assert np.allclose(a[ok], b[ok], rtol=1e-4, atol=1e-4 * np.median(np.abs(b[ok])))


def test_left_to_fp32(gpu, monkeypatch):
    """A that does not start on sixteen bytes."""
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(5)
    m, n, nb = 300, 66, 6
    A, X, R = _cn(rng, m, n), _cn(rng, nb, n), _cn(rng, nb, m)
    buf = torch.empty(m * n + 1, dtype=torch.complex64, device=gpu)
    Ad = buf[1:].view(m, n)
    Ad.copy_(to_dev(A, gpu))
    got = _apply(srpr, torch, _plan(srpr, Ad, nb, "bf16", monkeypatch), X, R, gpu)
    want = _apply(srpr, torch, _plan(srpr, Ad, nb, "own", monkeypatch), X, R, gpu)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("loss", ("l2", "poisson"))
def test_solvers(gpu, loss, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(6)
    m, n, nb = 700, 130, 11
    A, X = _cn(rng, m, n), _cn(rng, nb, n)
    y = (np.abs(X.astype(np.complex128) @ A.astype(np.complex128).T) ** 2).astype(np.float32)
    x0 = X + 0.1 * _cn(rng, nb, n)
    v0 = _cn(rng, nb, n)
    eta = 0.05 / float(y.mean()) if loss == "l2" else 0.05
    outs = []
    for f in ("bf16", "own"):
        plan = _plan(srpr, to_dev(A, gpu), nb, f, monkeypatch)
        if loss == "poisson":
            srpr.sr_plan_set_loss(plan, srpr.SR_LOSS_POISSON, 1e-3)
        x, tr = to_dev(x0.ravel(), gpu), torch.empty(nb * 4, device=gpu)
        sp = torch.empty_like(x)
        srpr.sr_gd_solve(plan, to_dev(y.ravel(), gpu), x, 4, eta, tr)
        srpr.sr_spectral_init(plan, to_dev(y.ravel(), gpu), to_dev(v0.ravel(), gpu), 4, -1.0, sp)
        srpr.sr_plan_sync(plan)
        outs.append([to_host(t) for t in (x, tr, sp)])
    for a, b in zip(*outs):
        assert rel_l2(a, b) <= 2e-5  # eight products of 2e-6 in turn
