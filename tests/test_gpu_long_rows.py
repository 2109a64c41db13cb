"""Delta-coded matrices whose rows are longer than their list and that were not
scanned by rows (windows too large to stage): the slots that k_slice_size
reserves for such rows hold the row and its escapes, also where z wraps around.
Bit for bit against the build that counts inside the scan."""
import numpy as np
import pytest

from occupancy import rules_of
from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import GpuCase
from test_gpu_crowded_cells import _crowded

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


@pytest.mark.parametrize("cells", [8, 13])
@pytest.mark.parametrize("prec", [S.SPH_F64, S.SPH_F32])
def test_slots_of_rows_beyond_their_list(ctx, monkeypatch, cells, prec):
    # 13: 140k particles, whose rows at the ends of z reach over 100k indices
    w = _crowded(64 * cells ** 3, cells, 0, W.KERNEL_GAUSSIAN, 171)
    r = rules_of(w)
    assert not r.delta and not r.scan_by_rows
    g = GpuCase(ctx, w)
    kw = dict(X0=0.5 * w.rhs, tol=1e-9, max_iter=2)
    print(f"[long rows] n={w.n} prec={prec}", flush=True)
    X, a = g.solve(w.rhs, prec, **kw)
    monkeypatch.setenv("SPH_BUILD_LEGACY", "1")
    Xd, b = g.solve(w.rhs, prec, **kw)
    monkeypatch.delenv("SPH_BUILD_LEGACY")
    assert a["mat_nnz"] == b["mat_nnz"] and b["mat_slots"] <= a["mat_slots"] <= 1.1 * b["mat_slots"]
    assert a["history"] == b["history"] and np.array_equal(X, Xd)
