"""Mixed precision on short chirp-z axes: first and refined residuals no larger
than with convolutions of at least 2n - 1 rows, whose figures the bars are (the
means over the same law of right-hand sides at 10 points per wavelength)."""

import pytest

from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid,first,refined", [
    ((129, 129), 1.53e-6, 3.8e-13),       # 256 rows for 512
    ((65, 65, 65), 6.8e-7, 2.8e-13),      # 128 for 256
    ((129, 129, 129), 9.6e-7, 3.7e-13),
    ((145, 145, 145), 1.07e-6, 4.1e-13),  # 288 for 512
])
def test_residuals(grid, first, refined):
    omega = inputs.omega_for_ppw(max(grid), 10.0)
    with helm.Plan(grid, inputs.spacing(grid), omega, precision=helm.PREC_MIXED) as plan:
        for seed in (1, 2):
            g = torch.Generator(device="cuda")
            g.manual_seed(seed)
            f = torch.view_as_complex(torch.randn((2,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))
            u = torch.empty_like(f)
            plan.solve(f, u)
            rep = plan.report()
            assert rep["iterations"] == 1
            assert rep["rel_residual_first"] <= first and rep["rel_residual_max"] <= refined
