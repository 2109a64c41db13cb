"""Systems that are certain to take the kernels they are meant for (each is
checked against the rules that choose them): sums over neighbours by cells for
particles outside a periodic box, for cells with more candidates than a block
stages at once and for rows with more neighbours than a wave lists before it
sums them; and a Gaussian matrix scanned by cells whose windows do not fit."""
import dataclasses

import numpy as np
import pytest

import test_gpu_cell_rows as rows
from occupancy import cells_of, rules_of
from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import GpuCase
from test_gpu_windows import _cloud

pytestmark = pytest.mark.gpu

LIST = 192  # neighbours that a wave lists per row (kCellList), summed when fewer than 64 places are left


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


def _systems(kernel):
    k = 1.0 if kernel == W.KERNEL_WENDLAND else 1.5  # cells 2h or 3h wide
    n = 1600 if kernel == W.KERNEL_WENDLAND else 3400
    outside = _cloud(n, 6.0 * k, 0.5, 201, (1, 1, 0))
    outside.pos[::7, 0] += 6.0 * k  # the same points, one period further on
    outside.pos[3::11, 1] -= 12.0 * k
    m = 60 if kernel == W.KERNEL_WENDLAND else 80
    crowds = [_cloud(64 * m, 4.05 * k, 0.5, 202), _cloud(64 * m + 1, 4.05 * k, 0.5, 203, (1, 0, 1))]
    out = [dataclasses.replace(w, kernel=kernel) for w in [outside] + crowds]
    for w in out:
        assert rules_of(w).sums_by_cells, w.name
    for w in out[1:]:
        count, _ = cells_of(w)
        assert 27 * w.n / count.size > rules_of(w).cap  # (the inner cells' candidates)
        assert w.n / count.size * 4.19 > LIST
    return out


@pytest.mark.parametrize("kernel", [W.KERNEL_WENDLAND, W.KERNEL_GAUSSIAN])
@pytest.mark.parametrize("prec", [S.SPH_F64, S.SPH_F32])
def test_on_the_fly_operator(ctx, monkeypatch, kernel, prec):
    monkeypatch.setattr(rows, "_systems", lambda: _systems(kernel))
    rows.test_on_the_fly_operator(ctx, kernel, prec)


@pytest.mark.parametrize("kernel", [W.KERNEL_WENDLAND, W.KERNEL_GAUSSIAN])
def test_viscosity_update(ctx, monkeypatch, kernel):
    monkeypatch.setattr(rows, "_systems", lambda: _systems(kernel))
    rows.test_viscosity_update(ctx, kernel)


@pytest.mark.parametrize("variant", [S.SPH_ROBUST, S.SPH_STANDARD])
def test_solves_with_the_on_the_fly_operator(ctx, monkeypatch, variant):
    monkeypatch.setattr(rows, "_systems", lambda: [None] + _systems(W.KERNEL_WENDLAND))
    rows.test_solves_with_the_on_the_fly_operator(ctx, variant)


@pytest.mark.parametrize("prec", [S.SPH_F64, S.SPH_F32, S.SPH_MIXED])
def test_windows_that_do_not_fit(ctx, monkeypatch, prec):
    # slices of this lattice that straddle two rows of cells see 3391 particles
    # of at most 3340
    w = dataclasses.replace(W.incline_papanastasiou(n=20, seed=204), kernel=W.KERNEL_GAUSSIAN)
    r = rules_of(w)
    assert not r.delta and not r.scan_by_rows
    g = GpuCase(ctx, w)
    kw = dict(X0=0.5 * w.rhs, tol=1e-9, max_iter=12, true_res_period=5, restart_drop=0.1)
    print(f"[sides] {w.name} n={w.n} prec={prec}", flush=True)
    X, a = g.solve(w.rhs, prec, **kw)
    monkeypatch.setenv("SPH_BUILD_LEGACY", "1")
    Xd, b = g.solve(w.rhs, prec, **kw)
    monkeypatch.delenv("SPH_BUILD_LEGACY")
    assert a["history"] == b["history"] and a["mat_slots"] == b["mat_slots"] and np.array_equal(X, Xd)


@pytest.mark.parametrize("n,early", [(59, True), (60, False)])
def test_solution_of_several_rounds(ctx, n, early):
    # up to 2^18 particles the solution is written before the host has read the
    # check of a round, and again after the next; beyond, after the last
    w = W.open_box(n, seed=132)
    assert (w.n <= 1 << 18) == early and abs(w.n - (1 << 18)) < 13000
    g = GpuCase(ctx, w)
    print(f"[sides] n={w.n}", flush=True)
    X, r = g.solve(w.rhs, S.SPH_MIXED, tol=3e-9, true_res_period=0)
    assert r["status"] == S.SPH_OK and r["n_true_checks"] >= 2, r["n_true_checks"]
    res = g.apply(X, S.SPH_F64)
    D = g.apply(np.ones_like(X), S.SPH_F64)  # row sums: 1 / A_rr on fluid rows
    b = np.where((w.ptype == W.FLUID)[:, None], w.rhs * D, 0.0)
    got = ((b - res) ** 2).sum(axis=0)
    # FP64 residuals of one x: their difference is rounding of the rows' sums
    assert np.allclose(np.sqrt(got), np.sqrt(r["true_rr"]), rtol=1e-5), (got, r["true_rr"])
