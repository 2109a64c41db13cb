"""Entries of the matrix that are exactly 0 (pairs without viscosity) keep an
Inf or NaN of x out of the rows that do not see it, in both column codes alike
and in every kernel that writes a row's slots: short rows (one block per
slice), rows longer than their list, the paper's single precision."""
import dataclasses

import numpy as np
import pytest

import oracle as O
from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import GpuCase, small_tank
from test_gpu_windows import _cloud

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


def _systems():
    return [W.open_box(13, seed=151), dataclasses.replace(W.open_box(14, seed=152), kernel=W.KERNEL_GAUSSIAN),
            small_tank(seed=153, n=(9, 7, 5)), _cloud(5000, 6.05, 0.5, 154)]


@pytest.mark.parametrize("avg", [W.AVG_ARITH, W.AVG_HARMONIC])
@pytest.mark.parametrize("prec,mode", [(S.SPH_F64, S.SPH_OP_CACHED), (S.SPH_F32, S.SPH_OP_CACHED),
                                       (S.SPH_F32, S.SPH_OP_PAPER32)])
def test_values_behind_zero_coefficients(ctx, avg, prec, mode, monkeypatch):
    for w in _systems():
        if mode == S.SPH_OP_PAPER32 and w.kernel == W.KERNEL_GAUSSIAN:
            continue
        rng = np.random.default_rng(w.n)
        mu = np.where(rng.random(w.n) < 0.6, 0.0, w.mu)
        w = dataclasses.replace(w, mu=mu, avg=avg)
        dead = np.flatnonzero(mu == 0.0)
        bad = rng.choice(dead, 40, replace=False)
        X = rng.normal(size=(w.n, 3)).astype(np.float32).astype(np.float64)
        X[bad] = np.array([np.inf, -np.inf, np.nan])
        print(f"[zeros] {w.name} n={w.n} kernel={w.kernel} avg={avg} prec={prec} mode={mode}", flush=True)
        g = GpuCase(ctx, w)
        Y = g.apply(X, prec, op_mode=mode)
        # the rows that see none of them: neither themselves, nor a neighbour
        # through a coefficient (dummy-wall rows see every fluid neighbour)
        rp, cols = O.neighbors(w.pos, w.period, w.h, method="brute",
                               support=3.0 if w.kernel == W.KERNEL_GAUSSIAN else 2.0)
        rows = np.repeat(np.arange(w.n), np.diff(rp))
        fluid = w.ptype == W.FLUID
        ma, mb = mu[cols], mu[rows]
        some = (ma + mb if avg == W.AVG_ARITH else ma * mb) > 0.0
        sees = np.where(fluid[rows], some, fluid[cols] & (w.wall == W.WALL_DUMMY))
        hit = np.zeros(w.n, bool)
        hit[bad] = True
        hit[rows[sees & hit[cols]]] = True
        assert 0 < hit.sum() < w.n
        assert np.all(np.isfinite(Y[~hit])), (w.name, np.flatnonzero(~hit & ~np.isfinite(Y).all(axis=1))[:5])
        if mode != S.SPH_OP_PAPER32:
            monkeypatch.setenv("SPH_BUILD_LEGACY", "1")
            Yd = g.apply(X, prec, op_mode=mode)
            monkeypatch.delenv("SPH_BUILD_LEGACY")
            assert np.array_equal(Y, Yd, equal_nan=True)
