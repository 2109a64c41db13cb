"""Sums over neighbours and lists on either side of the rule that takes them a
cell or a row at a time: boxes that are mostly empty (hundreds of cells per
particle, particles in one corner), one or a few crowded cells, and cells with
more candidates than a block stages at once.  Matrix, on-the-fly operator and
viscosity update against the oracle within the rounding of sums of the longest
row's length (shear rate: 1e-9), lists exactly."""
import dataclasses

import numpy as np
import pytest

import oracle as O
from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import F64_U, GpuCase, apply_bound, oracle_op, small_tank
from test_gpu_viscosity import _compare, _gpu
from test_gpu_windows import _cloud

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


def _corner(w, k):
    """The same particles in a box k times as long on its non-periodic axes."""
    hi = np.where(w.periodic, w.hi, w.lo + k * (w.hi - w.lo))
    return dataclasses.replace(w, hi=hi)


def _systems():
    return [_cloud(700, 60.0, 0.5, 141), _cloud(700, 45.0, 0.5, 142, (1, 1, 1)), _corner(W.open_box(13, seed=143), 5),
            _corner(small_tank(seed=144, n=(9, 7, 5)), 20), _cloud(900, 0.9, 0.5, 145), _cloud(4000, 3.05, 0.5, 146, (1, 1, 1)),
            _cloud(6000, 4.05, 0.5, 147, (1, 0, 1)), _cloud(5000, 6.05, 0.5, 148), _cloud(2, 50.0, 0.5, 149)]


@pytest.mark.parametrize("kernel", [W.KERNEL_WENDLAND, W.KERNEL_GAUSSIAN])
@pytest.mark.parametrize("k", range(9))
def test_sums_over_neighbours(ctx, kernel, k):
    w = dataclasses.replace(_systems()[k], kernel=kernel)
    print(f"[sparse] {w.name} n={w.n} kernel={kernel}", flush=True)
    g = GpuCase(ctx, w)
    rp, cols = g.export()
    orp, ocols = O.neighbors(w.pos, w.period, w.h, method="brute", support=3.0 if kernel == W.KERNEL_GAUSSIAN else 2.0)
    assert np.array_equal(rp, orp) and np.array_equal(cols, ocols)
    X = np.random.default_rng(1).normal(size=(w.n, 3))
    op = oracle_op(w, jacobi=True)
    D = oracle_op(w, jacobi=False, nbr=(op.row_ptr, op.cols)).diag()
    bound = apply_bound(D, X, F64_U, True, k=2 * int(np.diff(op.row_ptr).max()) + 50)
    for mode in (S.SPH_OP_CACHED, S.SPH_OP_ONTHEFLY):
        Y = g.apply(X, S.SPH_F64, jacobi=True, op_mode=mode)
        assert np.all(np.abs(Y - op.apply(X)).max(axis=1) <= bound), (w.name, mode)
    U = 1e-3 * X
    mu, sh = _gpu(ctx, g, U, S.SPH_F64)
    muo, Do = O.papanastasiou(oracle_op(w), U, 100.0, 1000.0, 1.0)
    _compare(w, mu, sh, muo, Do)
    # inner products of the operator by rows and by cells
    A, ra = g.solve(w.rhs, S.SPH_F64, tol=1e-10, op_mode=S.SPH_OP_ONTHEFLY)
    B, rb = g.solve(w.rhs, S.SPH_F64, tol=1e-10)
    assert ra["status"] == rb["status"] == 0
    # both solutions have residuals below 1e-10 |b| of a system whose inverse
    # (rows scaled to 1, diagonally dominant) is at most as large as its D
    assert np.linalg.norm(A - B) <= 2e-10 * max(D.max(), 1.0) * np.linalg.norm(B)
