"""The row kernels on tall matrices of short signals, where a plan's workgroups
are more and hold fewer rows: row counts on both sides of the lines (512 to 2048
workgroups of one wave from 5120 to 20480 rows, 512 to 1024 of four from 10240
to 20480), operators and one solve of each kind against 64 bits."""
import numpy as np
import pytest

from gpu_helpers import aligned, rel_l2, to_dev, to_host

import oracle
import sr_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,nb", [(5119, 32, 3), (5131, 130, 1), (20479, 16, 4), (20500, 34, 2), (33333, 66, 1),
                                    (10241, 260, 3), (20483, 300, 1), (10250, 514, 2)])
def test_tall(gpu, m, n, nb, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    monkeypatch.delenv("SR_DENSE_GEMM", raising=False)
    rng = np.random.default_rng(m)
    A, X, R = (sr_inputs.complex_gaussian(rng, s) for s in ((m, n), (nb, n), (nb, m)))
    plan = srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(nb)], None, dense_A=to_dev(A, gpu))
    z, v = (torch.empty(k, dtype=torch.complex64, device=gpu) for k in (nb * m, nb * n))
    y = torch.empty(nb * m, device=gpu)
    srpr.sr_forward(plan, to_dev(X.ravel(), gpu), z, y)
    srpr.sr_adjoint(plan, to_dev(R.ravel(), gpu), v)
    A6 = A.astype(np.complex128)
    zr = X @ A6.T
    assert rel_l2(to_host(z).reshape(nb, m), zr) <= 2e-5
    assert rel_l2(to_host(y).reshape(nb, m), np.abs(zr) ** 2) <= 4e-5
    assert rel_l2(to_host(v).reshape(nb, n), R @ A6.conj()) <= 2e-5
    op = oracle.DenseOperator(A)
    Y = (np.abs(zr) ** 2).astype(np.float32)
    yd = to_dev(Y.ravel(), gpu)
    x0 = (X + 0.2 * sr_inputs.complex_gaussian(rng, (nb, n))).astype(np.complex64)
    x, tr = to_dev(x0.ravel(), gpu), torch.zeros(2 * nb, device=gpu)
    eta = float(np.float32(0.1 / Y.mean()))
    srpr.sr_gd_solve(plan, yd, x, 2, eta, tr)
    srpr.sr_spectral_init(plan, yd, to_dev(x0.ravel(), gpu), 2, -1.0, v)
    srpr.sr_plan_sync(plan)
    for p in range(nb):
        want, loss = oracle.gd_solve(op, Y[p], x0[p], 2, eta, return_loss=True)
        assert aligned(to_host(x).reshape(nb, n)[p], want) <= 1e-4
        assert np.max(np.abs(to_host(tr).reshape(nb, 2)[p] - loss)) <= 1e-4 * np.abs(loss).max()
        assert rel_l2(to_host(v).reshape(nb, n)[p], oracle.spectral_init(op, Y[p], x0[p], 2, -1.0)) <= 1e-4
