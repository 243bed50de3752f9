"""Power-of-two axes of 1024 to 4096 points: two passes and both tiles of the
single pass, forced through the tune cache, with ragged column tiles, against
banded LU; the choice is timed once and cached."""

import numpy as np
import pytest

from oracle import fem
from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", [helm.PREC_FP64, helm.PREC_MIXED])
@pytest.mark.parametrize("grid", [(1024, 11), (2048, 7), (4096, 5), (1024, 3, 5), (3, 2048, 4)])
def test_pow2_forms(grid, prec, tmp_path):
    dim = len(grid)
    h = (1.0 / (max(grid) - 1),) * dim
    omega = 2 * np.pi * (max(grid) - 1) / 10
    abc = ((True, True),) * dim
    f = inputs.gaussian_batch(grid, [51, 52])
    ref = fem.solve(grid, h, omega, abc, f.reshape(2, -1))
    key = f"dim={dim} grid={grid[0]}x{grid[1]}x{grid[2] if dim == 3 else 1} prec={prec}"
    axis = int(np.argmax(grid))
    cache = tmp_path / "tune.txt"
    with helm.Plan(grid, h, omega, precision=prec, tune_cache=str(cache)):
        pass
    assert len([ln for ln in cache.read_text().splitlines() if f" pow2{axis}=" in ln]) == 1
    for choice in (0, 1, 2):
        forced = tmp_path / f"forced{choice}.txt"
        forced.write_text(f"helm-tune {key} pow2{axis}={choice}\n")
        # tol 0: refinement steps too, whose last transforms accumulate into u
        with helm.Plan(grid, h, omega, precision=prec, tol=0.0, max_iter=2, tune_cache=str(forced)) as plan:
            fd = torch.from_numpy(f).cuda()
            ud = torch.empty_like(fd)
            rc = plan.solve(fd, ud, raise_on_error=False)
            u = ud.cpu().numpy().reshape(2, -1)
        assert rc in (helm.HELM_OK, helm.HELM_ENOCONV)
        assert len([ln for ln in forced.read_text().splitlines() if " pow2" in ln]) == 1
        assert np.max(fem.rel_error(u, ref)) <= 1e-9
