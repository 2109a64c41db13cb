"""How a solve's host side follows the device: iteration limits at and beyond
the per-iteration flags that the pinned copy holds, several rounds, and
solutions written before and after the host knows that a round was the last.
Nothing of it may change the result: bit for bit against one iteration queued
at a time, and the solution handed back against the reported residual."""
import numpy as np
import pytest

from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import GpuCase, small_tank

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


@pytest.mark.parametrize("max_iter", [0, 1, 2, 7, 4094, 4095, 4096, 4300])
def test_iteration_limits(ctx, max_iter):
    # restarts from the true residual every other iteration keep FP32 vectors
    # from ever reaching the tolerance
    w = small_tank(seed=131, n=(4, 4, 3))
    g = GpuCase(ctx, w)
    kw = dict(tol=1e-18, floor=0.0, max_iter=max_iter, true_res_period=2, restart_drop=1e30)
    stall = max(max_iter - 3, 1)
    for kw in (kw, dict(kw, force_stall=(stall, 1))):
        print(f"[rounds] max_iter={max_iter} {kw}", flush=True)
        a, ra = g.solve(w.rhs, S.SPH_F32, **kw)
        b, rb = g.solve(w.rhs, S.SPH_F32, poll_every=1, **kw)
        assert np.array_equal(a, b) and ra["history"] == rb["history"] and ra["true_rr"] == rb["true_rr"]
        assert ra["stall_count"] == rb["stall_count"] and ra["iters"] == rb["iters"] == max_iter
        assert len(ra["history"]) == max_iter + 1
        assert ra["stall_count"][1] >= (1 if "force_stall" in kw and max_iter > stall else 0)


@pytest.mark.parametrize("n", [64, 65])
def test_solution_of_the_last_round(ctx, n):
    # up to 2^18 particles the solution is written before the host's check of
    # the last round is read; tol below what FP32 reaches in one round
    w = W.open_box(n, seed=132)
    g = GpuCase(ctx, w)
    print(f"[rounds] n={w.n}", flush=True)
    X, r = g.solve(w.rhs, S.SPH_MIXED, tol=1e-8, true_res_period=0)
    assert r["status"] == S.SPH_OK and r["n_true_checks"] >= 1
    res = g.apply(X, S.SPH_F64)
    D = g.apply(np.ones_like(X), S.SPH_F64)  # row sums: 1 / A_rr on fluid rows
    b = np.where((w.ptype == W.FLUID)[:, None], w.rhs * D, 0.0)
    got = ((b - res) ** 2).sum(axis=0)
    # FP64 residuals of one x: their difference is rounding of the rows' sums
    assert np.allclose(np.sqrt(got), np.sqrt(r["true_rr"]), rtol=1e-5), (got, r["true_rr"])
