"""The workspace of a plan of 1D problems moved into caller memory and on again:
lengths of every table kind (an element a lane, narrow, default and twelve
elements), the memory left behind overwritten, the same bits as before."""
import numpy as np
import pytest

import sr_inputs
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


def test_moved(gpu):
    import torch
    import paper_2409_05734_amd as srpr
    rng = np.random.default_rng(105)
    shapes = [((m // 2,), (m,), 1 + i % 2) for i, m in enumerate((16, 64, 96, 192, 256, 768, 1024, 2048))]
    ths = [sr_inputs.phase_masks(rng, L, m) for _, m, L in shapes]
    plan = srpr.Plan([srpr.Problem(*s) for s in shapes], np.concatenate([t.ravel() for t in ths]))
    x = to_dev(np.concatenate([sr_inputs.complex_gaussian(rng, n) for n, _, _ in shapes]), gpu)
    r = to_dev(np.concatenate([sr_inputs.complex_gaussian(rng, m) for _, m, _ in shapes]), gpu)

    def run():
        z, v, est, gx = torch.empty_like(r), torch.empty_like(x), torch.empty_like(x), torch.empty_like(x)
        y, gt, xg = torch.empty(plan.m_total, device=gpu), torch.zeros(plan.theta_len, device=gpu), 0.9 * x
        srpr.sr_forward(plan, x, z, y)
        srpr.sr_adjoint(plan, r, v)
        srpr.sr_gd_solve(plan, y, xg, 3, 0.01)
        srpr.sr_spectral_init(plan, y, x, 3, -1.0, est)
        srpr.sr_forward_vjp(plan, x, r, gx, gt)
        srpr.sr_plan_sync(plan)
        return [torch.view_as_real(t).clone() for t in (z, v, xg, est, gx)] + [y, gt]

    before = run()
    size = srpr.sr_plan_workspace_size(plan)
    ws = [torch.empty(size, dtype=torch.uint8, device=gpu) for _ in range(2)]
    for i in range(2):
        srpr.sr_plan_set_workspace(plan, ws[i])
        if i:
            ws[0].fill_(0xFF)
        assert all(torch.equal(a, b) for a, b in zip(before, run())), i
