"""Training gradient at the edges of its batches: tiles of 16 samples, pairs of
tiles, groups of four, blocks of four waves, the largest number of blocks; and
samples that do not lie on 16-byte boundaries.  Against the oracle, which
rounds the same values to BF16 and sums in FP64, at the gradient test's
tolerances."""
import numpy as np
import pytest

from oracle import mlp as M
from paper_2206_14780_amd import sph as S

from gpu_util import rel_l2
from test_gpu_mlp import GRAD_REL, _cuda, _params, _samples

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return S.Context(0)


@pytest.mark.parametrize("offset", [0, 1, 3])
@pytest.mark.parametrize("batch", [15, 16, 17, 32, 33, 64, 65, 127, 128, 129, 32768, 32769, 65537, 150001])
def test_gradient_at_batch_edges(ctx, batch, offset):
    import torch
    if offset and batch > 40000:
        pytest.skip("alignment does not depend on the batch")
    pool = _samples(3000, seed=8)
    idx = np.random.default_rng(batch).integers(0, pool.shape[0], size=batch).astype(np.int32)
    p = _params(5)
    buf = torch.zeros(pool.size + 4, dtype=torch.float32, device="cuda")
    buf[offset:offset + pool.size] = _cuda(pool).reshape(-1)
    grad = torch.empty(M.NPARAM, dtype=torch.float32, device="cuda")
    print(f"grad batch={batch} offset={offset}", flush=True)
    loss = ctx.sph_mlp_grad(buf[offset:offset + pool.size], _cuda(idx), batch, _cuda(p), grad)
    torch.cuda.synchronize()
    lo, go = M.loss_grad(p.astype(np.float64), pool[idx].astype(np.float64), bf=True)
    assert abs(loss - lo) <= 1e-4 * lo
    assert rel_l2(grad.cpu().double().numpy(), go) < GRAD_REL
