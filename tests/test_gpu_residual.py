"""Residual launches at the edges of their geometry: strips of 4 to 64 rows
(planes), ragged last strips and tiles, norms finished in the last block or by
the separate kernels, called again on the same plan (the arrival counter has
to be zero again)."""

import numpy as np
import pytest

from oracle import fem
from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

OMEGA = 9.0


@pytest.mark.parametrize("grid,nrhs", [
    ((5, 4), 1),            # one ragged strip
    ((127, 256), 1),        # strips of 4, ragged last one
    ((130, 257), 3),        # a second column tile of one column
    ((1025, 513), 5),       # strips of 16 or 32
    ((4097, 300), 17),      # 2D: more blocks than finish their norms in the last one
    ((6, 9, 65), 1),        # 3D: strips of 4, a second column tile of one column
    ((61, 75, 90), 2),
    ((65, 40, 70), 19),     # longer strips
    ((70, 250, 260), 12),   # 3D, separate finish, strips of 64 planes
])
def test_residual_and_norms(grid, nrhs):
    h = inputs.spacing(grid)
    abc = ((True, True),) * len(grid)
    g = torch.Generator(device="cuda")
    g.manual_seed(len(grid) * 100 + nrhs)
    u = torch.view_as_complex(torch.randn((nrhs,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))
    f = torch.view_as_complex(torch.randn((nrhs,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))
    r = torch.empty_like(f)
    with helm.Plan(grid, h, OMEGA, boundary=helm.BOUNDARY_LINES) as plan:
        rel = plan.residual(u, f, r)
        again = plan.residual(u, f)
    # A has at most 27 entries a row, each a sum of 4 products of 1D entries:
    # under 200 roundings of terms bounded by |A| |u|, whose rms is within 4 of
    # that of A u for independent u
    tol = 1000 * 2.0 ** -53
    picks = sorted({0, nrhs // 2, nrhs - 1})
    for b in picks:
        ref = fem.residual(grid, h, OMEGA, abc, u[b].cpu().numpy().reshape(1, -1),
                           f[b].cpu().numpy().reshape(1, -1)).reshape(-1)
        got = r[b].cpu().numpy().reshape(-1)
        scale = np.sqrt(np.mean(np.abs(ref) ** 2))
        assert np.max(np.abs(got - ref)) <= 10 * tol * scale  # 10: the largest of the |u|
        want = np.linalg.norm(ref) / np.linalg.norm(f[b].cpu().numpy())
        assert abs(rel[b] - want) <= tol * want
    assert np.array_equal(rel, again)
