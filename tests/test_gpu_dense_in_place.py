"""Dense plans with A x written over x and A^H r over r: on the row kernels,
whose workgroups read x while others store, in bf16 parts and in FP32."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu


def _over(torch, gpu, x, m):
    """x at the start of a buffer of m entries: (x's view, the whole)."""
    buf = torch.zeros(m, dtype=torch.complex64, device=gpu)
    buf[:x.size] = to_dev(x.ravel(), gpu)
    return buf[:x.size], buf


@pytest.mark.parametrize("force,m,n,nb", [(None, 5000, 512, 1), (None, 512, 512, 3), (None, 3000, 4096, 4),
                                          ("bf16", 700, 130, 9), ("own", 700, 130, 9)])
def test_in_place(gpu, force, m, n, nb, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    if force is None:
        monkeypatch.delenv("SR_DENSE_GEMM", raising=False)
    else:
        monkeypatch.setenv("SR_DENSE_GEMM", force)
    rng = np.random.default_rng(m)
    A, X, R = (sr_inputs.complex_gaussian(rng, s) for s in ((m, n), (nb, n), (nb, m)))
    plan = srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(nb)], None,
                     dense_A=to_dev(A, gpu))
    x, z = _over(torch, gpu, X, max(X.size, R.size))
    srpr.sr_forward(plan, x, z[:R.size], None)
    r, v = _over(torch, gpu, R, max(X.size, R.size))
    srpr.sr_adjoint(plan, r, v[:X.size])
    srpr.sr_plan_sync(plan)
    op = oracle.DenseOperator(A)
    for p in range(nb):
        assert rel_l2(to_host(z)[:R.size].reshape(R.shape)[p], op.A(X[p])) <= 2e-5
        assert rel_l2(to_host(v)[:X.size].reshape(X.shape)[p], op.AH(R[p])) <= 2e-5
