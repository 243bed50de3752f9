"""Rounding of the plan's tables: the residual of the plain FP64 solve of 256^3
at 10 points per wavelength, before any refinement, in both forms of the
boundary steps.

The bars are three times what a numpy model of the method has at this size,
which holds one table at a time as the plan does and everything else exactly."""

import pytest

from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRID = (256, 256, 256)


def _first_residuals(boundary, seeds):
    out = []
    with helm.Plan(GRID, inputs.spacing(GRID), inputs.omega_for_ppw(256, 10.0), tol=1.0, boundary=boundary) as plan:
        for seed in seeds:
            g = torch.Generator(device="cuda")
            g.manual_seed(seed)
            f = torch.view_as_complex(torch.randn((1,) + GRID + (2,), generator=g, device="cuda", dtype=torch.float64))
            u = torch.empty_like(f)
            plan.solve(f, u)
            rep = plan.report()
            assert rep["boundary"] == boundary and rep["iterations"] == 0
            out.append(rep["rel_residual_first"])
    return out


@pytest.mark.parametrize("boundary", [helm.BOUNDARY_LINES, helm.BOUNDARY_TABLES])
def test_entering_pivots(boundary):
    """Pivots that enter a lane's rows as the rows before leave them: 5.8e-12 to
    6.9e-12 in the model (composed in a scan over the lanes 2.7e-11 to 3.8e-11)."""
    assert max(_first_residuals(boundary, (1, 2, 3))) <= 2e-11


def test_periodic_spectra():
    """Periodic eigenvalues right to extended precision, not shifted alike in all
    modes: 8.8e-14 to 1.2e-13 in the model with the boundary steps in the
    eigenbasis (with pi rounded to double 3.7e-13 to 4.7e-13)."""
    assert max(_first_residuals(helm.BOUNDARY_TABLES, (1, 2, 3))) <= 3.5e-13


# Refinement to 1e-10 would hide a pass that loses digits: the first residuals of
# the shapes whose last columns run in a launch of their own and of lines that
# blocks take one after the other.  FP64: the error bar of the parity tests;
# mixed: complex64 has 6e-8, which the first solve amplifies up to 150 times at
# 2049 nodes and 10 points per wavelength.
@pytest.mark.parametrize("prec", [helm.PREC_FP64, helm.PREC_MIXED])
@pytest.mark.parametrize("grid,nrhs", [((513, 1025), 4), ((1025, 1025), 1), ((1025, 2050), 1), ((2049, 1027), 1),
                                       ((2049, 513), 1), ((257, 2049), 4), ((67, 29, 100), 2), ((35, 61, 128), 2),
                                       ((33, 47, 256), 2), ((37, 31, 200), 2)])
def test_no_digits_lost_before_refinement(grid, nrhs, prec):
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    f = torch.view_as_complex(torch.randn((nrhs,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))
    h = (1.0 / (max(grid) - 1),) * len(grid)
    with helm.Plan(grid, h, inputs.omega_for_ppw(max(grid), 10.0), precision=prec) as plan:
        plan.solve(f, torch.empty_like(f))
        rep = plan.report()
    mixed = prec == helm.PREC_MIXED
    assert rep["rel_residual_first"] <= (1e-5 if mixed else 1e-9) and rep["iterations"] <= 1
