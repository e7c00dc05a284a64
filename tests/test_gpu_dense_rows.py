"""GPU parity of the dense model's row kernels (few signals, one read of A per
solver iteration) against the FP64 oracle at the edges of their shapes: each
thread count and column slice filled and just overfilled, row counts that leave
a batch or a workgroup short, padded signal slots, two groups of signals, and
the sizes next to the rule that sends a plan to the matrix cores instead."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import aligned, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL_OP = 2e-5  # the parity bar per application
TOL_IT = 1e-4  # ... and on iterates


@pytest.mark.parametrize("m,n,nb", [
    (1, 2, 1), (9, 2, 4), (513, 128, 1), (390, 130, 2), (1025, 256, 3), (1037, 258, 1), (2053, 512, 4),
    (2057, 514, 2), (4099, 1024, 1), (3001, 1026, 4), (2600, 2048, 1), (2571, 2050, 2), (4101, 4096, 1),
    (2311, 4094, 3), (259, 4096, 4), (300, 64, 5), (1000, 258, 8), (403, 94, 7), (700, 4098, 1), (500, 60, 9)])
def test_dense_rows(gpu, m, n, nb, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    monkeypatch.delenv("SR_DENSE_GEMM", raising=False)
    rng = np.random.default_rng(m + 3 * n + 7 * nb)
    A = sr_inputs.complex_gaussian(rng, (m, n))
    op = oracle.DenseOperator(A)
    X = sr_inputs.complex_gaussian(rng, (nb, n))
    R = sr_inputs.complex_gaussian(rng, (nb, m))
    Ad = to_dev(A, gpu)
    plan = srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(nb)], None, dense_A=Ad)
    z = torch.empty(nb * m, dtype=torch.complex64, device=gpu)
    y = torch.empty(nb * m, dtype=torch.float32, device=gpu)
    v = torch.empty(nb * n, dtype=torch.complex64, device=gpu)
    srpr.sr_forward(plan, to_dev(X.ravel(), gpu), z, y)
    srpr.sr_adjoint(plan, to_dev(R.ravel(), gpu), v)
    Z = np.stack([op.A(X[p]) for p in range(nb)])
    torch.cuda.synchronize()
    for p in range(nb):
        assert rel_l2(to_host(z).reshape(nb, m)[p], Z[p]) <= TOL_OP
        assert rel_l2(to_host(y).reshape(nb, m)[p], np.abs(Z[p]) ** 2) <= 2 * TOL_OP
        assert rel_l2(to_host(v).reshape(nb, n)[p], op.AH(R[p])) <= TOL_OP
    Y = (np.abs(Z) ** 2).astype(np.float32)
    yd = to_dev(Y.ravel(), gpu)
    V0 = sr_inputs.complex_gaussian(rng, (nb, n))
    srpr.sr_spectral_init(plan, yd, to_dev(V0.ravel(), gpu), 3, -1.0, v)
    torch.cuda.synchronize()
    for p in range(nb):
        assert rel_l2(to_host(v).reshape(nb, n)[p], oracle.spectral_init(op, Y[p], V0[p], 3, -1.0)) <= TOL_IT
    X0 = (X + 0.25 * sr_inputs.complex_gaussian(rng, (nb, n))).astype(np.complex64)
    eps = float(0.1 * np.mean(Y))
    for loss, eta in (("l2", np.float32(0.05 / float(np.mean(Y.astype(np.float64))))), ("poisson", np.float32(0.05))):
        if loss == "poisson":
            srpr.sr_plan_set_loss(plan, srpr.SR_LOSS_POISSON, eps)
        x = to_dev(X0.ravel(), gpu)
        lt = torch.zeros(3 * nb, dtype=torch.float32, device=gpu)
        srpr.sr_gd_solve(plan, yd, x, 3, eta, lt)
        torch.cuda.synchronize()
        for p in range(nb):
            kw = {"loss": "poisson", "eps": eps} if loss == "poisson" else {}
            xr, lr = oracle.gd_solve(op, Y[p], X0[p], 3, float(eta), return_loss=True, **kw)
            assert aligned(to_host(x).reshape(nb, n)[p], xr) <= TOL_IT
            scale = np.abs(lr).max()
            assert np.max(np.abs(to_host(lt).reshape(nb, 3)[p] - lr)) <= 1e-4 * scale
