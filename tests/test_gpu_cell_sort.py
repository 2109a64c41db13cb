"""The order of the particles within a cell: by their original index, for
cells of every length class of the sort (one wave's registers, several, by
insertion).  Two listings of the same particles that keep the relative order
within each cell have the same rows and row sums in the same order, so the
operator agrees bit for bit, whatever order the scatter's atomics arrive in;
and each against the oracle within the rounding of the longest row."""
import dataclasses

import numpy as np
import pytest

from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import F32_U, GpuCase, apply_bound, oracle_op

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


@pytest.mark.parametrize("counts", [(1, 0, 2, 63, 64, 65), (127, 128, 129, 1), (255, 256, 257), (600, 0, 3)])
def test_cells_are_in_original_order(ctx, counts):
    rng = np.random.default_rng(sum(counts))
    m, h = len(counts), 0.5
    side = np.array([1.0001 * m, 1.0, 1.0])
    cell = np.repeat(np.arange(m), counts)
    n = cell.size
    pos = rng.uniform(0.01, 0.99, (n, 3))
    pos[:, 0] = (cell + pos[:, 0]) * side[0] / m
    rho = rng.uniform(0.95, 1.05, n)
    w = W.Workload(f"row{counts}", pos, rho * np.prod(side) / n, rho, 10.0 ** rng.uniform(0.0, 2.0, n),
                   np.zeros(n, np.uint8), np.zeros(3), side, np.zeros(3, int), h, 1e-3, W.WALL_DUMMY,
                   W.AVG_HARMONIC, rng.normal(size=(n, 3)), None, 1e-6)
    X = rng.normal(size=(n, 3)).astype(np.float32).astype(np.float64)
    a = rng.permutation(n)                         # cells interleaved
    b = a[np.argsort(cell[a], kind="stable")]      # cell after cell, the same order within each
    out = np.empty((2, n, 3))
    for k, p in enumerate((a, b)):
        wp = dataclasses.replace(w, pos=w.pos[p], mass=w.mass[p], rho=w.rho[p], mu=w.mu[p], rhs=w.rhs[p])
        print(f"[cell order] {counts} listing {k}", flush=True)
        Y = GpuCase(ctx, wp).apply(X[p], S.SPH_F32)
        op = oracle_op(wp, jacobi=True)
        D = oracle_op(wp, jacobi=False, nbr=(op.row_ptr, op.cols)).diag()
        bound = apply_bound(D, X, F32_U, True, k=2 * int(np.diff(op.row_ptr).max()) + 50)
        assert np.all(np.abs(Y - op.apply(X[p])).max(axis=1) <= bound)
        out[k][p] = Y
    assert np.array_equal(out[0], out[1])
