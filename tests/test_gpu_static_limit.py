"""A solve that fits the fixed scratch of ``helm_solve_static`` only with the
fewest partial sums of its line reductions is taken, not refused."""

import numpy as np
import pytest

from oracle import fem
from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid", [(2048, 1700), (2048, 1600)])  # fewest partial sums; as many as pay
def test_near_the_scratch_limit(grid):
    h = (1.0 / (grid[0] - 1),) * 2
    omega = 2 * np.pi * (grid[0] - 1) / 10
    f = inputs.gaussian_batch(grid, [61])
    # two work arrays, and 2 x 1700 partial sums for every 4 (8) of 2048 lines:
    # 111 + 28 MB do not fit 134 MB, 111 + 14 MB do
    with helm.Plan(grid, h, omega, precision=helm.PREC_FP64, check=False) as plan:
        fd = torch.from_numpy(f).cuda()
        ud = torch.empty_like(fd)
        plan.solve_static(fd, ud)
        torch.cuda.synchronize()
        u = ud.cpu().numpy().reshape(1, -1)
    # a plain solve: residuals of 1e-10 to 1e-8 at these sizes; lost partial sums leave one of order one
    assert np.max(fem.rel_residual(grid, h, omega, ((True, True),) * 2, u, f.reshape(1, -1))) <= 1e-6
