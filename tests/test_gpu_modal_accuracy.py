"""Plain FP64 solves with the boundary steps in the eigenbasis of the last axis
against line sweeps, from well resolved axes to nearly defective ones (the
eigenbasis may amplify rounding errors there up to the factor that the plan
accepts): neither form is several times further off than the other."""

import math

import pytest

from paper_1809_03808_amd import helm

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _solve(grid, h, omega, f, **kw):
    with helm.Plan(grid, h, omega, **kw) as plan:
        u = torch.empty_like(f)
        plan.solve(f, u, raise_on_error=False)
        return u, plan.report()


# points per wavelength along the last axis; 63 nodes at 3.5 and 256 at 3.7 have
# factors of 36 and 56, those at 4 and 5 of 9 to 32
@pytest.mark.parametrize("n,ppw", [(63, 3.5), (63, 4), (63, 5), (63, 8), (129, 4), (129, 5), (129, 6), (256, 3.7),
                                   (256, 4), (256, 5), (256, 8), (256, 20)])
def test_error_of_plain_solves(n, ppw):
    grid, h, omega = (40, 36, n), (1.0 / (n - 1),) * 3, 2 * math.pi * (n - 1) / ppw
    err = {helm.BOUNDARY_LINES: 0.0, helm.BOUNDARY_TABLES: 0.0}
    for seed in range(4):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        f = torch.view_as_complex(torch.randn((1,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))
        ref, rep = _solve(grid, h, omega, f, boundary=helm.BOUNDARY_LINES, tol=0.0, max_iter=6)
        assert rep["rel_residual_max"] <= 1e-14
        for form in err:
            u, rep = _solve(grid, h, omega, f, boundary=form, check=False)
            assert rep["boundary"] == form
            err[form] += (torch.linalg.vector_norm(u - ref) / torch.linalg.vector_norm(ref)).item() / 4
    # four times, and the reference's own error
    assert err[helm.BOUNDARY_TABLES] <= 4 * err[helm.BOUNDARY_LINES] + 5e-14, err
    assert err[helm.BOUNDARY_LINES] <= 1e-10


def test_host_eigenpairs():
    """Eigenpairs from the host setup serve the eigenbasis as the device's do."""
    grid, h, omega = (40, 36, 63), (1.0 / 62,) * 3, 2 * math.pi * 62 / 10
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    f = torch.view_as_complex(torch.randn((2,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))
    out = []
    for eigen in (helm.EIGEN_HOST, helm.EIGEN_DEVICE):
        u, rep = _solve(grid, h, omega, f, boundary=helm.BOUNDARY_TABLES, eigen=eigen, check=False)
        assert rep["boundary"] == helm.BOUNDARY_TABLES
        out.append(u)
    # each within the bar of the parity tests of the solution
    assert (torch.linalg.vector_norm(out[0] - out[1]) / torch.linalg.vector_norm(out[1])).item() <= 2e-9


@pytest.mark.parametrize("check", [False, True])
@pytest.mark.parametrize("bad", [0, 1, 2])
def test_nan_stays_in_its_right_hand_side(bad, check):
    """One of three right-hand sides holds a NaN: the others' plain solutions are
    what they are without it, and a checked solve reports it."""
    grid, h, omega = (20, 37, 63), (1.0 / 62,) * 3, 2 * math.pi * 62 / 10
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    f = torch.view_as_complex(torch.randn((3,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))
    clean, _ = _solve(grid, h, omega, f, boundary=helm.BOUNDARY_TABLES, check=False)
    f[bad, 3, 5, 7] = float("nan")
    u, rep = _solve(grid, h, omega, f, boundary=helm.BOUNDARY_TABLES, check=check)
    if check:
        assert rep["status"] == helm.HELM_ENONFINITE
    else:
        for b in range(3):
            if b != bad:
                assert torch.equal(u[b], clean[b])
        assert not torch.isfinite(torch.view_as_real(u[bad])).all()


@pytest.mark.parametrize("grid", [(5, 9, 6), (9, 5, 13), (6, 7, 21), (10, 11, 33), (7, 6, 90), (9, 8, 129),
                                  (33, 40, 24), (4, 5, 257), (4, 5, 450), (3, 4, 700)])
def test_tables_run_at_the_edges_of_the_line_lengths(grid):
    """The grids of the line-length tests at 10 points per wavelength."""
    h, omega = (1.0 / (max(grid) - 1),) * 3, 2 * math.pi * (max(grid) - 1) / 10
    f = torch.ones((1,) + grid, dtype=torch.complex128, device="cuda")
    _, rep = _solve(grid, h, omega, f, boundary=helm.BOUNDARY_TABLES)
    assert rep["boundary"] == helm.BOUNDARY_TABLES and rep["status"] == helm.HELM_OK
