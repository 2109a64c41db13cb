"""What an export of the neighbour lists leaves allocated: bounded, whatever the
number of particles, and nothing of what another call keeps is taken away."""
import numpy as np
import pytest

from paper_2206_14780_amd import sph as S
from paper_2206_14780_amd import workloads as W

from gpu_util import GpuCase

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def test_an_export_gives_its_lists_back():
    w = W.open_box(112, seed=181)  # 1.6M particles, 700 MB of lists
    ctx = S.Context(0)
    g = GpuCase(ctx, w)
    before = _free()
    rp, cols = ctx.sph_neighbors_export(g.nb)
    first = cols.clone()
    nnz = int(rp[-1])
    del rp, cols
    rp, cols = ctx.sph_neighbors_export(g.nb)
    assert bool((cols == first).all()) and int(rp[-1]) == nnz
    del rp, cols, first
    print(f"[export memory] n={w.n} kept {(before - _free()) / 2**20:.0f} MiB", flush=True)
    assert before - _free() <= (256 << 20) + 40 * w.n
    # a matrix keeps its lists through an export
    small = W.open_box(30, seed=182)
    h = GpuCase(ctx, small)
    X = np.random.default_rng(1).normal(size=(small.n, 3))
    a = h.apply(X, S.SPH_F64)
    h.export()
    assert np.array_equal(a, h.apply(X, S.SPH_F64))
    ctx.close()
