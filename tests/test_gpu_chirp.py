"""Chirp-z lengths at the edges of their ranges: 2^k + 1 nodes, whose
convolution of 2n - 2 points has no padding at all, their neighbours, and the
lengths 72, 144 and 288 that only run as one pass; every form that an axis
has, forced through the tune cache, against banded LU."""

import numpy as np
import pytest

from oracle import fem
from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", [helm.PREC_FP64, helm.PREC_MIXED])
@pytest.mark.parametrize("n", [5, 9, 17, 34, 37, 38, 65, 66, 73, 74, 129, 130, 145, 146, 257, 258, 513, 1025, 2049])
def test_chirp_lengths(n, prec, tmp_path):
    grid = (n, 6)
    h = (1.0 / (n - 1),) * 2
    omega = 2 * np.pi * (n - 1) / 10
    abc = ((True, True),) * 2
    f = inputs.gaussian_batch(grid, [61, 62])
    ref = fem.solve(grid, h, omega, abc, f.reshape(2, -1))
    key = f"dim=2 grid={n}x6x1 prec={prec}"
    for choice in (0, 1):
        cache = tmp_path / f"chirp{choice}.txt"
        cache.write_text(f"helm-tune {key} chirp0={choice}\n")
        with helm.Plan(grid, h, omega, precision=prec, check=prec == helm.PREC_MIXED, tune_cache=str(cache)) as plan:
            fd = torch.from_numpy(f).cuda()
            ud = torch.empty_like(fd)
            plan.solve(fd, ud)
            u = ud.cpu().numpy().reshape(2, -1)
        # the bars of the solver's parity tests
        assert np.max(fem.rel_error(u, ref)) <= (1e-9 if prec == helm.PREC_FP64 else 1e-8)


# Columns past the last full tile in a launch of their own: batches whose full
# tiles fill every compute unit once or more, with one column left (513 points,
# several right-hand sides; 1025 and 2049 points, one), and their neighbours
# that leave none or more than the narrow tile takes.
@pytest.mark.parametrize("prec", [helm.PREC_FP64, helm.PREC_MIXED])
@pytest.mark.parametrize("grid,nrhs", [((513, 1025), 2), ((513, 1025), 4), ((1025, 1025), 1), ((1025, 1024), 1),
                                       ((1025, 2050), 1), ((2049, 1027), 1), ((2049, 513), 1), ((257, 2049), 4)])
def test_last_columns(grid, nrhs, prec):
    h = (1.0 / (grid[0] - 1),) * 2
    omega = 2 * np.pi * (grid[0] - 1) / 10
    f = inputs.gaussian_batch(grid, list(range(61, 61 + nrhs)))
    with helm.Plan(grid, h, omega, precision=prec) as plan:
        fd = torch.from_numpy(f).cuda()
        ud = torch.empty_like(fd)
        plan.solve(fd, ud)
        u = ud.cpu().numpy().reshape(nrhs, -1)
    # the solve's own stopping rule
    assert np.max(fem.rel_residual(grid, h, omega, ((True, True),) * 2, u, f.reshape(nrhs, -1))) <= 1e-10
