"""The operator's two column codes give the same bits: a solve on the windowed
matrix (x staged in LDS by ranges of particles) against one on the delta-coded
matrix of the scan-order build, which takes the same terms in the same order.

The systems put every kind of window at its edge: one window per block and
two (Wendland boxes, whose cells of 2 or 3 lattice sites per axis make the
windows of 256 rows straddle the limit), two and four (the truncated
Gaussian), windows that wrap around periodic axes of few cells, ragged last
slices, a single row, and a cloud so dense that no window fits, which keeps
the delta code."""
import dataclasses

import numpy as np
import pytest

from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import warmstart as WS
from paper_2206_14780_amd import workloads as W

from gpu_util import GpuCase, small_tank

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


def _cloud(n, side, h, seed, periodic=(0, 0, 0)):
    """n uniform random fluid particles in a box of the given side."""
    rng = np.random.default_rng(seed)
    mu = 10.0 ** rng.uniform(0.0, 2.0, n)
    rho = rng.uniform(0.95, 1.05, n)
    return W.Workload(f"cloud{n}", rng.uniform(0.0, side, (n, 3)), rho * side ** 3 / n, rho, mu,
                      np.zeros(n, np.uint8), np.zeros(3), np.full(3, side), np.array(periodic), h, 1e-3,
                      W.WALL_DUMMY, W.AVG_HARMONIC, rng.normal(size=(n, 3)), None, 1e-6)


def _systems():
    box = W.open_box(30, seed=81)
    return [box, dataclasses.replace(W.open_box(24, seed=82), kernel=W.KERNEL_GAUSSIAN),
            dataclasses.replace(W.poiseuille(16, shuffle_seed=83), kernel=W.KERNEL_GAUSSIAN),
            W.poiseuille(8, wall=W.WALL_DUMMY, shuffle_seed=84), W.poiseuille(14, shuffle_seed=85),
            W.incline_papanastasiou(n=20, seed=86), W.lava_channel(19, seed=87), small_tank(seed=88),
            _cloud(4096, 2.05, 0.5, 89), _cloud(257, 4.0, 0.5, 90, (1, 1, 1)), _cloud(1, 2.0, 0.5, 91, (1, 0, 0)),
            _cloud(65, 30.0, 1.0, 92)]


@pytest.mark.parametrize("prec", [S.SPH_F64, S.SPH_F32, S.SPH_MIXED])
@pytest.mark.parametrize("variant", [S.SPH_ROBUST, S.SPH_STANDARD, S.SPH_CG])
def test_windowed_solves_equal_delta_coded_ones(ctx, prec, variant, monkeypatch):
    for w in _systems():
        if variant == S.SPH_CG:
            w = dataclasses.replace(w, wall=W.WALL_DYNAMIC)
        print(f"[windows] {w.name} n={w.n} kernel={w.kernel} prec={prec} variant={variant}", flush=True)
        g = GpuCase(ctx, w)
        kw = dict(X0=0.5 * w.rhs, tol=1e-9, max_iter=12, variant=variant, true_res_period=5, restart_drop=0.1)
        Xw, rw = g.solve(w.rhs, prec, **kw)
        monkeypatch.setenv("SPH_BUILD_LEGACY", "1")
        Xd, rd = g.solve(w.rhs, prec, **kw)
        monkeypatch.delenv("SPH_BUILD_LEGACY")
        assert rw["history"] == rd["history"] and rw["true_rr"] == rd["true_rr"]
        assert rw["mat_nnz"] == rd["mat_nnz"]
        assert np.array_equal(Xw, Xd)


@pytest.mark.parametrize("prec", [S.SPH_F64, S.SPH_F32, S.SPH_MIXED])
def test_learned_start_on_windows_equals_delta_code(ctx, prec, monkeypatch):
    import torch
    warm = torch.as_tensor(WS.load()).cuda()
    for w in _systems()[:7]:
        print(f"[windows, learned] {w.name} n={w.n} kernel={w.kernel} prec={prec}", flush=True)
        g = GpuCase(ctx, w)
        kw = dict(X0=0.5 * w.rhs, tol=1e-9, max_iter=6, warm_params=warm)
        Xw, rw = g.solve(w.rhs, prec, **kw)
        monkeypatch.setenv("SPH_BUILD_LEGACY", "1")
        Xd, rd = g.solve(w.rhs, prec, **kw)
        monkeypatch.delenv("SPH_BUILD_LEGACY")
        assert rw["plain_rr"] == rd["plain_rr"] and rw["warm_rr"] == rd["warm_rr"]
        assert rw["history"] == rd["history"] and np.array_equal(Xw, Xd)
