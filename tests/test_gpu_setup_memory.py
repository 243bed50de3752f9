"""A plan whose shape has more forms than there is memory to time keeps the
default forms: setup needs no more memory than its own tables and the timing of
the line sweeps."""

import gc

import pytest

from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MB = 1 << 20


def test_forms_that_cannot_be_timed(tmp_path):
    # 33.5 M nodes: 270 MB of tables, 540 MB to time the sweeps, 1610 MB to time the
    # passes of the 1024-point axis
    grid = (1024, 64, 512)
    cache = tmp_path / "tune.txt"
    gc.collect()
    torch.cuda.empty_cache()  # (torch would give cached blocks back in need)
    held = []
    for _ in range(4):  # (the runtime gives back memory of its own on a large allocation)
        free, _ = torch.cuda.mem_get_info()
        if free > 1410 * MB:
            held.append(torch.empty(free - 1400 * MB, dtype=torch.uint8, device="cuda"))
    assert torch.cuda.mem_get_info()[0] <= 1450 * MB
    try:
        plan = helm.Plan(grid, (1.0 / 1023,) * 3, inputs.omega_for_ppw(1024, 10.0), boundary=helm.BOUNDARY_LINES,
                         tune_cache=str(cache))
    finally:
        del held
        torch.cuda.empty_cache()
    text = cache.read_text()
    assert " layout=" in text and " pow20=" not in text
    with plan:
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        f = torch.view_as_complex(torch.randn((1,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))
        plan.solve(f, torch.empty_like(f))
        assert plan.report()["rel_residual_max"] <= 1e-10
