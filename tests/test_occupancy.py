"""Rules on how particles fill cells (occupancy.hpp), on the host: evenly filled
boxes go cell by cell, sparse ones and ones with a crowded cell row by row,
whatever the mean says.  No GPU."""
import pytest

from paper_2206_14780_amd import workloads as W

from occupancy import rules, rules_of


@pytest.mark.parametrize("gauss,mean", [(False, 17), (True, 58)])
@pytest.mark.parametrize("cells", [343, 4096, 60000])
def test_even_boxes_go_by_cells(gauss, mean, cells):
    r = rules(mean * cells, cells, gauss, 2 * mean)
    assert r.sums_by_cells and not r.delta and not r.scan_by_rows


@pytest.mark.parametrize("gauss,mean", [(False, 17), (True, 58)])
@pytest.mark.parametrize("cells", [343, 4096, 60000])
def test_one_crowded_cell_sends_the_work_to_the_rows(gauss, mean, cells):
    # the matrix keeps its windows: they do not depend on who scans
    for fullest in (512, 700, 5000):
        r = rules(mean * cells, cells, gauss, fullest)
        assert not r.sums_by_cells and r.scan_by_rows and not r.delta, fullest


def test_crowding_counts_against_the_mean():
    # 303 particles in every cell are not a crowd
    assert rules(65536, 216, False, 352).sums_by_cells
    assert not rules(65536, 216, False, 1300).sums_by_cells


@pytest.mark.parametrize("gauss", [False, True])
def test_sparse_boxes_go_by_rows(gauss):
    r = rules(1000, 30_000_000, gauss, 20)
    assert not r.sums_by_cells and r.delta and r.scan_by_rows


@pytest.mark.parametrize("gauss,most", [(False, 1088), (True, 1920)])
def test_staged_candidates_are_bounded_whole_waves(gauss, most):
    for mean in (0.001, 1, 17, 35, 36, 66, 67, 1000, 1e6):
        cap = rules(int(mean * 1000) or 1, 1000, gauss).cap
        assert cap % 64 == 0 and 64 <= cap <= most
        assert cap >= min(27 * mean, most - 64)


def test_the_workloads_are_on_the_side_of_the_cells():
    for w in (W.open_box(30, seed=1), W.poiseuille(16), W.incline_papanastasiou(n=20, seed=1), W.lava_channel(19, seed=1)):
        r = rules_of(w)
        assert r.sums_by_cells and not r.scan_by_rows, w.name
