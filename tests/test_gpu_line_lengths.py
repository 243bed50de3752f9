"""Line lengths at the edges of the chunk geometry: for every lane count P the
shortest and longest lines of each chunk length (one lane, all lanes, all but
one lane with the long chunk), in both precisions, in 2D and in both forms and
layouts of the 3D reductions, against banded LU."""

import numpy as np
import pytest

from oracle import fem
from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LENGTHS = sorted({3, 4, 5, 6, 7} | {n for P in (2, 4, 8, 16, 32, 64, 128, 256)
                                    for n in (4 * P + 1, 5 * P, 5 * P + 1, 6 * P + 2, 7 * P - 1, 7 * P + 1, 8 * P - 1)}
                 | {2051, 2560, 3000, 3584, 4095})


def _check(grid, prec, **kw):
    h = (1.0 / (max(grid) - 1),) * len(grid)
    omega = 2 * np.pi * (max(grid) - 1) / 10
    abc = ((True, True),) * len(grid)
    f = inputs.gaussian_batch(grid, [41, 42])
    ref = fem.solve(grid, h, omega, abc, f.reshape(2, -1))
    with helm.Plan(grid, h, omega, precision=prec, check=prec == helm.PREC_MIXED, **kw) as plan:
        fd = torch.from_numpy(f).cuda()
        ud = torch.empty_like(fd)
        plan.solve(fd, ud)
        u = ud.cpu().numpy().reshape(2, -1)
    # the bars of the solver's parity tests
    assert np.max(fem.rel_error(u, ref)) <= (1e-9 if prec == helm.PREC_FP64 else 1e-8)


@pytest.mark.parametrize("prec", [helm.PREC_FP64, helm.PREC_MIXED])
@pytest.mark.parametrize("n", LENGTHS)
def test_2d_line_lengths(n, prec):
    _check((8 if n < 700 else 4, n), prec)


@pytest.mark.parametrize("layout", ["2", "3"])
@pytest.mark.parametrize("boundary", [helm.BOUNDARY_LINES, helm.BOUNDARY_TABLES])
@pytest.mark.parametrize("grid,prec", [((5, 9, 6), helm.PREC_FP64), ((9, 5, 13), helm.PREC_MIXED),
                                       ((6, 7, 21), helm.PREC_FP64), ((10, 11, 33), helm.PREC_MIXED),
                                       ((7, 6, 90), helm.PREC_FP64), ((9, 8, 129), helm.PREC_MIXED),
                                       ((33, 40, 24), helm.PREC_FP64), ((4, 5, 257), helm.PREC_FP64),
                                       ((4, 5, 450), helm.PREC_MIXED), ((3, 4, 700), helm.PREC_FP64)])
def test_3d_line_lengths(grid, prec, boundary, layout, monkeypatch):
    monkeypatch.setenv("HELM_RED_L_LAYOUT", layout)
    _check(grid, prec, boundary=boundary)


# Blocks that take several lines one after the other, the last tile ragged: the
# reducing kernels load a line's rows while the one before is solved.
@pytest.mark.parametrize("prec", [helm.PREC_FP64, helm.PREC_MIXED])
@pytest.mark.parametrize("grid", [(75, 320), (83, 513), (37, 1024), (43, 2049), (27, 4096), (75, 600), (41, 1500)])
def test_2d_several_lines_per_block(grid, prec):
    _check(grid, prec)


@pytest.mark.parametrize("layout", ["2", "3"])
@pytest.mark.parametrize("grid,prec", [((67, 29, 100), helm.PREC_MIXED), ((35, 61, 128), helm.PREC_FP64),
                                       ((33, 47, 256), helm.PREC_FP64), ((37, 31, 200), helm.PREC_MIXED)])
def test_3d_several_lines_per_block(grid, prec, layout, monkeypatch):
    monkeypatch.setenv("HELM_RED_L_LAYOUT", layout)
    h = (1.0 / (max(grid) - 1),) * 3
    omega = 2 * np.pi * (max(grid) - 1) / 10
    f = inputs.gaussian_batch(grid, [41, 42])
    with helm.Plan(grid, h, omega, precision=prec) as plan:
        fd = torch.from_numpy(f).cuda()
        ud = torch.empty_like(fd)
        plan.solve(fd, ud)
        u = ud.cpu().numpy().reshape(2, -1)
    # the solve's own stopping rule (banded LU would take minutes at these bandwidths)
    assert np.max(fem.rel_residual(grid, h, omega, ((True, True),) * 3, u, f.reshape(2, -1))) <= 1e-10
