"""Tune-cache lines whose times are of something that the plan does not run are
not taken: the decision is measured again, and the new line is."""

import pytest

from paper_1809_03808_amd import helm, inputs

pytestmark = pytest.mark.gpu


def _lines(cache, what):
    return [ln for ln in cache.read_text().splitlines() if what in ln]


def _setup(grid, cache, **kw):
    with helm.Plan(grid, inputs.spacing(grid), inputs.omega_for_ppw(max(grid), 10.0), tune_cache=str(cache), **kw):
        pass


@pytest.mark.parametrize("old", [0, 16])
def test_times_of_operator_tables(old, tmp_path):
    """`tables_ms` were the times of n3 x n3 operator tables, not of the eigenbasis."""
    grid = (24, 20, 22)
    key = "helm-tune dim=3 grid=24x20x22 prec=0"
    cache = tmp_path / "tune.txt"
    cache.write_text(f"{key} boundary cap_min_nb={old} lines_ms_1=1 lines_ms_16=9 tables_ms_1=2 tables_ms_16=8\n")
    for _ in range(2):  # measured once, then read
        _setup(grid, cache)
        lines = _lines(cache, " boundary ")
        assert len(lines) == 2 and " eigenbasis_ms_1=" in lines[1]


def test_times_of_another_convolution(tmp_path):
    """129 nodes: a line without a length is of the 512-point convolution that
    2n - 1 rows took, one of another length of another."""
    grid = (129, 33)
    key = "helm-tune dim=2 grid=129x33x1 prec=0"
    cache = tmp_path / "tune.txt"
    cache.write_text(f"{key} chirp0=0 multipass_ms=1 onepass_ms=2\n{key} chirp0=1 M=512 multipass_ms=2 onepass_ms=1\n")
    for _ in range(2):
        _setup(grid, cache)
        lines = _lines(cache, " chirp0=")
        assert len(lines) == 3 and " M=256 " in lines[2]


def test_decisions_without_times_are_taken(tmp_path):
    grid = (24, 20, 22)
    key = "helm-tune dim=3 grid=24x20x22 prec=0"
    cache = tmp_path / "tune.txt"
    cache.write_text(f"{key} boundary cap_min_nb=3\n{key} chirp0=1\n{key} chirp1=0\n")
    _setup(grid, cache)
    assert len(_lines(cache, " boundary ")) == 1 and len(_lines(cache, " chirp")) == 2


@pytest.mark.parametrize("boundary,launch", [(helm.BOUNDARY_TABLES, "plain"), (helm.BOUNDARY_LINES, "rank2")])
def test_layout_timed_on_the_launch_of_the_solves(boundary, launch, tmp_path):
    cache = tmp_path / "tune.txt"
    _setup((24, 20, 22), cache, boundary=boundary)
    lines = _lines(cache, " layout=")
    assert len(lines) == 1 and f" launch={launch} " in lines[0]
