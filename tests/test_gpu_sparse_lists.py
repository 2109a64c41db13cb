"""Neighbour lists of sparse boxes by each of their routes: with lists, without,
counted in the caller's order or in cell order.  The same particles in a larger
box have the same lists, by another route; small ones against the oracle."""
import dataclasses

import numpy as np
import pytest

import oracle as O
from occupancy import rules_of
from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import GpuCase
from test_gpu_windows import _cloud

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


@pytest.mark.parametrize("kernel", [W.KERNEL_WENDLAND, W.KERNEL_GAUSSIAN])
@pytest.mark.parametrize("n", [1, 2, 63, 700, (1 << 17) - 1, 1 << 17])
def test_routes_give_the_same_lists(ctx, kernel, n):
    cell = 1.0 if kernel == W.KERNEL_WENDLAND else 1.5
    w = dataclasses.replace(_cloud(n, cell * max(n, 8) ** (1 / 3), 0.5, 191), kernel=kernel)
    wide = dataclasses.replace(w, hi=w.lo + 1.5 * (w.hi - w.lo))
    assert rules_of(wide).no_lists and rules_of(wide).caller_order == (n < 1 << 17)
    if n >= 63:
        assert not rules_of(w).no_lists
    out = []
    for v in (w, wide):
        print(f"[sparse lists] n={n} kernel={kernel}", flush=True)
        g = GpuCase(ctx, v)
        total = ctx.sph_neighbors_info(g.nb)[1]
        out.append(g.export())
        assert total == out[-1][1].size == out[-1][0][-1]
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    if n < 1000:
        orp, ocols = O.neighbors(w.pos, w.period, w.h, method="brute",
                                 support=3.0 if kernel == W.KERNEL_GAUSSIAN else 2.0)
        assert np.array_equal(out[0][0], orp) and np.array_equal(out[0][1], ocols)
    else:
        assert out[0][1].size > n
