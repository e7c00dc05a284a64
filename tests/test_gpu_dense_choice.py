"""What a dense plan runs without the library: the faster of the FP32 and the
bf16 products, and the same answers as the plan with every candidate."""
import pytest

pytestmark = pytest.mark.gpu


def _apply(gpu, monkeypatch, force, A, X, R):
    import torch
    import paper_2409_05734_amd as srpr
    if force is None:
        monkeypatch.delenv("SR_DENSE_GEMM", raising=False)
    else:
        monkeypatch.setenv("SR_DENSE_GEMM", force)
    m, n = A.shape
    plan = srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(len(X))], None, dense_A=A)
    z, v = torch.empty_like(R), torch.empty_like(X)
    srpr.sr_forward(plan, X, z, None)
    srpr.sr_adjoint(plan, R, v)
    srpr.sr_plan_sync(plan)
    return z, v


def _inputs(gpu, m, n, nb):
    import torch
    g = torch.Generator(device=gpu).manual_seed(m)
    return [torch.randn(s, dtype=torch.complex64, device=gpu, generator=g) for s in ((m, n), (nb, n), (nb, m))]


def test_large_products_without_the_library(gpu, monkeypatch):
    """Where the bf16 products win by far (141 and 127 us against 212 and 230
    in the FP32 kernel), a plan takes them though no library is asked."""
    import torch
    A, X, R = _inputs(gpu, 16384, 4096, 32)
    hand, bf16, own = (_apply(gpu, monkeypatch, f, A, X, R) for f in ("hand", "bf16", "own"))
    for a, b, c in zip(hand, bf16, own):
        assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
        assert not torch.equal(torch.view_as_real(a), torch.view_as_real(c))


# n > m, a product of each length of timing, A off the sixteen bytes
@pytest.mark.parametrize("m,n,nb,shift", [(100, 260, 40, 0), (3070, 682, 19, 0), (9000, 4000, 9, 0), (700, 66, 9, 1)])
@pytest.mark.parametrize("force", (None, "hand", "lib"))
def test_same_answers(gpu, m, n, nb, shift, force, monkeypatch):
    import torch
    A, X, R = _inputs(gpu, m, n, nb)
    if shift:
        buf = torch.empty(m * n + 1, dtype=torch.complex64, device=gpu)
        buf[1:].view(m, n).copy_(A)
        A = buf[1:].view(m, n)
    z, v = _apply(gpu, monkeypatch, force, A, X, R)
    A6 = A.to(torch.complex128)
    for got, want in ((z, X.to(torch.complex128) @ A6.T), (v, R.to(torch.complex128) @ A6.conj())):
        assert float((got - want).norm() / want.norm()) <= 2e-5


def test_workspace_of_what_runs(gpu, monkeypatch):
    """A plan holds the scratch of the kernels that it runs: one signal on the
    row kernels 256 workgroups' partials of A^H r (8.4 MB) and the vectors; the
    packed operand and the splits of the bf16 products only where they may run."""
    import torch
    import paper_2409_05734_amd as srpr

    def size(m, n, nb, force=None):
        if force is None:
            monkeypatch.delenv("SR_DENSE_GEMM", raising=False)
        else:
            monkeypatch.setenv("SR_DENSE_GEMM", force)
        A = torch.zeros(m, n, dtype=torch.complex64, device=gpu)
        plan = srpr.Plan([srpr.Problem((n,), (m,), 1, kind=srpr.SR_DENSE) for _ in range(nb)], None, dense_A=A)
        return srpr.sr_plan_workspace_size(plan)

    assert size(16384, 4096, 1) <= 9_000_000
    own, lib, bf16, free = (size(4096, 1024, 32, f) for f in ("own", "lib", "bf16", None))
    assert own == lib < bf16 == free
    assert size(300, 1024, 32) == size(300, 1024, 32, "own")  # n > m: the bf16 products are not considered
