"""The tuner's file of decisions (SR_TUNE_CACHE): entries whose tiles this build
does not have (written by a build with other thread shapes, or damaged) are
timed anew, the others are taken as they are."""
import numpy as np
import pytest

import oracle
import sr_inputs
from gpu_helpers import rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu


# row tiles of 8 transforms of 384 points and column tiles of 16 of 768 were
# offered when their threads held twelve elements each; 4 and 2 of 384 are
@pytest.mark.parametrize("grid,entry,taken", [((64, 384), "2 8 0", False), ((768, 64), "16 1 1", False),
                                              ((64, 64), "7 -3 0", False), ((64, 384), "2 4 0", True)])
def test_entry(gpu, grid, entry, taken, tmp_path, monkeypatch):
    import torch
    import paper_2409_05734_amd as srpr
    for k in ("SR_TUNE", "SR_TUNE_FORCE", "SR_PHASE_TABLE"):
        monkeypatch.delenv(k, raising=False)
    path = tmp_path / "tiles"
    line = f"{grid[0]}x{grid[1]}:30x40:L2 {entry}\n"
    path.write_text(line)
    monkeypatch.setenv("SR_TUNE_CACHE", str(path))
    rng = np.random.default_rng(grid[0])
    th = sr_inputs.phase_masks(rng, 2, grid)
    x = sr_inputs.complex_gaussian(rng, (30, 40))
    for _ in range(2):  # the second plan finds what the first stored
        plan = srpr.Plan([srpr.Problem((30, 40), grid, 2)], th.ravel())
        z = torch.empty(plan.m_total, dtype=torch.complex64, device=gpu)
        srpr.sr_forward(plan, to_dev(x.ravel(), gpu), z, None)
        srpr.sr_plan_sync(plan)
        assert rel_l2(to_host(z).reshape(grid), oracle.forward(x, th, grid)) <= 2e-5
    lines = path.read_text().splitlines()
    assert lines[0] + "\n" == line and len(lines) == (1 if taken else 2)
