"""Captured graphs given up while their last launch may still run: unchecked
solves and batches that move on to other buffers, sizes and streams without a
wait in between.  Every result is that of an eager solve, bit for bit."""

import pytest

from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _rhs(grid, seed, nrhs=1):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.view_as_complex(torch.randn((nrhs,) + grid + (2,), generator=g, device="cuda", dtype=torch.float64))


def _plan(grid, **kw):
    return helm.Plan(grid, inputs.spacing(grid), inputs.omega_for_ppw(max(grid), 10.0), **kw)


@pytest.mark.parametrize("streams", [1, 2])
def test_unchecked_solves_move_on(streams):
    grid = (1024, 700)
    fs = [_rhs(grid, s, 1 + s % 2) for s in range(6)]
    us = [torch.empty_like(f) for f in fs]
    with _plan(grid, check=False) as plan:
        want = []
        for f in fs:
            u = torch.empty_like(f)
            plan.solve(f, u)
            want.append(u)
        torch.cuda.synchronize()
        st = [torch.cuda.Stream() for _ in range(streams)]
        for k in range(2):
            for i, (f, u) in enumerate(zip(fs, us)):
                s = st[i % streams]
                if streams > 1:  # a plan works on one stream at a time
                    s.wait_stream(st[(i - 1) % streams])
                for _ in range(3):  # eager, captured, replayed
                    plan.solve(f, u, stream=s)
        torch.cuda.synchronize()
        for u, w in zip(us, want):
            assert torch.equal(u, w)
        u = us[0].zero_()
        plan.solve(fs[0], u)
        plan.solve(fs[0], u)
    torch.cuda.synchronize()  # the plan is gone with its last launch just made
    assert torch.equal(u, want[0])


def test_batch_moves_on():
    grids = [(512, 300), (257, 129)]
    plans = [_plan(g, precision=helm.PREC_MIXED) for g in grids]
    sets = [([_rhs(g, 10 * k + i, 2) for i, g in enumerate(grids)]) for k in range(3)]
    outs = [[torch.empty_like(f) for f in fs] for fs in sets]
    with helm.Batch(plans, max_nrhs=2) as batch:
        for _ in range(2):
            for fs, us in zip(sets, outs):
                batch.solve(fs, us)  # captures and launches; the next set follows at once
        torch.cuda.synchronize()
    for fs, us in zip(sets, outs):
        for p, f, u in zip(plans, fs, us):
            assert p.residual(u, f).max() <= 1e-10
    for p in plans:
        p.close()
