"""Iterations issued past a halt, for any setting of the run-ahead and however
the residual history misleads the forecast: the halting iteration of each round
of host-side residual checks, and at most one more."""
import pytest

from paper_2206_14780_amd import sph as S

from gpu_util import GpuCase, small_tank

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("poll_every", [0, 1, 2, 16, 1000])
@pytest.mark.parametrize("tol", [1e-2, 1e-5, 1e-7])
def test_issued_past_the_halt(poll_every, tol):
    ctx = S.Context(0)
    w = small_tank(seed=72, n=(16, 12, 10), dt_nu=80.0)
    g = GpuCase(ctx, w)
    for _ in range(10):
        _, r = g.solve(w.rhs, S.SPH_F32, tol=tol, poll_every=poll_every, true_res_period=0)
        assert r["iters"] <= r["issued_iters"] <= r["iters"] + r["n_true_checks"] + 1, r
