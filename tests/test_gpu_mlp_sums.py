"""Where the training gradient's sums over the samples are taken in FP32: within
four tiles (64 samples) of a wave and nowhere else, whatever the batch.

Powers of two scale every value of the backward pass exactly, so the gradient
of a batch can be put together from gradients of its parts: with two tiles a
wave, from those of the batches of 32 samples that the waves take, added in
FP64 and rounded once; and a batch that repeats one sample has the same
gradient, bit for bit, at every size whose waves take whole groups of four
tiles."""
import numpy as np
import pytest

from oracle import mlp as M
from paper_2206_14780_amd import sph as S

from test_gpu_mlp import _cuda, _params, _samples

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


def test_sum_over_waves_and_blocks_is_rounded_once(ctx):
    import torch
    batch, part = 32768, 32
    pool = _cuda(_samples(3000, seed=21))
    idx = _cuda(np.random.default_rng(22).integers(0, pool.shape[0], size=batch).astype(np.int32))
    p = _cuda(_params(23))
    grad = torch.empty(M.NPARAM, dtype=torch.float32, device="cuda")
    ctx.sph_mlp_grad(pool, idx, batch, p, grad)
    one = torch.empty_like(grad)
    ref, mag = (torch.zeros(M.NPARAM, dtype=torch.float64, device="cuda") for _ in range(2))
    for k in range(0, batch, part):
        ctx.sph_mlp_grad(pool, idx[k:k + part].contiguous(), part, p, one)
        d = one.double() * (part / batch)
        ref += d
        mag += d.abs()
    # one rounding to FP32, and the roundings of two FP64 sums of 1024 terms
    u, n = 2.0 ** -24, batch // part
    bound = u * ref.abs() * (1 + 2.0 ** -20) + 2 * n * 2.0 ** -53 * mag
    # outside the 64x64 layers a part's gradient is itself a rounded sum over lanes
    square = torch.zeros(M.NPARAM, dtype=torch.bool, device="cuda")
    ow2 = 5 * 64
    ow3 = ow2 + 64 * 64 + 64
    square[ow2:ow2 + 64 * 64] = square[ow3:ow3 + 64 * 64] = True
    bound = torch.where(square, bound, bound + u * mag)
    err = (grad.double() - ref).abs()
    print(f"[mlp sums] {int((err > bound).sum())} beyond, largest err/bound {float((err / (bound + 1e-300)).max()):.3f}",
          flush=True)
    assert bool((err <= bound).all())


@pytest.mark.parametrize("batch", [131072, 262144, 524288, 1048576])
def test_chains_do_not_grow_with_the_batch(ctx, batch):
    import torch
    pool = _cuda(_samples(64, seed=24))
    p = _cuda(_params(25))
    g = [torch.empty(M.NPARAM, dtype=torch.float32, device="cuda") for _ in range(2)]
    for s in range(4):
        print(f"[mlp sums] batch={batch} sample={s}", flush=True)
        loss = [ctx.sph_mlp_grad(pool, torch.full((b,), s, dtype=torch.int32, device="cuda"), b, p, o)
                for b, o in zip((65536, batch), g)]
        assert torch.equal(g[0], g[1]) and loss[0] == loss[1]
