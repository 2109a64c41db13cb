"""The cell-at-a-time sums over neighbours (on-the-fly operator, viscosity
update) where their staging can go wrong: clouds whose cells hold more
candidates than one batch stages and whose rows have more neighbours than one
list, single particles, sparse clouds with mostly empty cells, periodic axes
of one to three cells, four rows of a wave ragged in every way, particles
outside the box on a periodic axis.  Against the oracle within the rounding
of sums of the longest row's length (operator) and 1e-9 (shear rate), and the
operator's dot products through a short solve."""
import dataclasses

import numpy as np
import pytest

import oracle as O
from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import F32_U, F64_U, GpuCase, apply_bound, oracle_op, rel_l2, small_tank
from test_gpu_viscosity import _compare, _gpu
from test_gpu_windows import _cloud

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


def _systems():
    outside = _cloud(300, 6.0, 0.6, 105, (1, 1, 0))
    outside.pos[::7, 0] += 6.0  # the same points, one period further on
    outside.pos[3::11, 1] -= 12.0
    return [_cloud(4096, 2.05, 0.5, 101), _cloud(257, 4.0, 0.5, 102, (1, 1, 1)), _cloud(1, 2.0, 0.5, 103),
            _cloud(65, 30.0, 1.0, 104), outside, _cloud(500, 2.2, 0.5, 106, (1, 0, 1)),
            _cloud(700, 3.2, 0.5, 107, (1, 1, 1)), small_tank(seed=108, n=(9, 7, 5)), W.open_box(13, seed=109)]


@pytest.mark.parametrize("kernel", [W.KERNEL_WENDLAND, W.KERNEL_GAUSSIAN])
@pytest.mark.parametrize("prec", [S.SPH_F64, S.SPH_F32])
def test_on_the_fly_operator(ctx, kernel, prec):
    u = F64_U if prec == S.SPH_F64 else F32_U
    for w in _systems():
        w = dataclasses.replace(w, kernel=kernel)
        print(f"[cells, operator] {w.name} n={w.n} kernel={kernel} prec={prec}", flush=True)
        g = GpuCase(ctx, w)
        X = np.random.default_rng(1).normal(size=(w.n, 3))
        X = X if prec == S.SPH_F64 else X.astype(np.float32).astype(np.float64)
        op = oracle_op(w, jacobi=True)
        Y = g.apply(X, prec, jacobi=True, op_mode=S.SPH_OP_ONTHEFLY)
        D = oracle_op(w, jacobi=False, nbr=(op.row_ptr, op.cols)).diag()
        longest = int(np.diff(op.row_ptr).max())
        bound = apply_bound(D, X, u, True, k=2 * longest + 50)
        assert np.all(np.abs(Y - op.apply(X)).max(axis=1) <= bound), w.name


@pytest.mark.parametrize("kernel", [W.KERNEL_WENDLAND, W.KERNEL_GAUSSIAN])
def test_viscosity_update(ctx, kernel):
    for w in _systems():
        w = dataclasses.replace(w, kernel=kernel)
        print(f"[cells, viscosity] {w.name} n={w.n} kernel={kernel}", flush=True)
        g = GpuCase(ctx, w)
        U = 1e-3 * np.random.default_rng(2).normal(size=(w.n, 3))
        mu, D = _gpu(ctx, g, U, S.SPH_F64)
        muo, Do = O.papanastasiou(oracle_op(w), U, 100.0, 1000.0, 1.0)
        _compare(w, mu, D, muo, Do)


@pytest.mark.parametrize("kernel", [W.KERNEL_WENDLAND, W.KERNEL_GAUSSIAN])
def test_lists(ctx, kernel):
    # rows within, at and beyond the entries that the export lists per row
    for w in _systems() + [dataclasses.replace(small_tank(seed=110, n=(10, 10, 6)), h=1.5)]:
        w = dataclasses.replace(w, kernel=kernel)
        print(f"[cells, lists] {w.name} n={w.n} kernel={kernel}", flush=True)
        g = GpuCase(ctx, w)
        rp, cols = g.export()
        orp, ocols = O.neighbors(w.pos, w.period, w.h, method="brute",
                                 support=3.0 if kernel == W.KERNEL_GAUSSIAN else 2.0)
        assert np.array_equal(rp, orp) and np.array_equal(cols, ocols)


@pytest.mark.parametrize("variant", [S.SPH_ROBUST, S.SPH_STANDARD])
def test_solves_with_the_on_the_fly_operator(ctx, variant):
    for w in _systems()[1:]:
        print(f"[cells, solve] {w.name} n={w.n} variant={variant}", flush=True)
        g = GpuCase(ctx, w)
        X, rep = g.solve(w.rhs, S.SPH_F64, tol=1e-12, op_mode=S.SPH_OP_ONTHEFLY, variant=variant)
        Xo, ro, _ = O.solve(oracle_op(w), w.rhs, tol=1e-12)
        assert rep["status"] == S.SPH_OK and rel_l2(X, Xo) < 1e-10
