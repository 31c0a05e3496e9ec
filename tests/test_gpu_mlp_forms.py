"""Loss and bias gradients of batches whose products take the 128 x 128 and 128 x 32
GEMM tiles, at odd ranks and hidden sizes (element-wise operand loads) and even ones:
the sums that the products' epilogues leave per tile cover every row of the batch."""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp
from paper_1904_07935_amd.api import Mlp
from tests.gpu_util import bf16_round, rel_fro
from tests.test_gpu_foldin_mlp import _bf16_params, _net, _np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,H", [(2112, 77, 512), (3000, 201, 512), (3000, 200, 512), (4096, 201, 512),
                                   (4608, 77, 256), (10000, 77, 128), (2050, 20, 33), (32768, 20, 33),
                                   (32768, 21, 32), (9000, 31, 31)])
def test_tile_sums(cuda, N, K, H):
    rng = np.random.default_rng(N + K + H)
    p = _net(rng, K, H)
    net = Mlp(K, H, device=cuda, seed=None)
    net.set_masters(p)
    X = rng.random((N, K)).astype(np.float32)
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    Y = (0.2 * rng.random((N, K))).astype(np.float32)
    loss, grads, _ = net.loss_grad(torch.tensor(X, device=cuda), torch.tensor(Y, device=cuda))
    q = _bf16_params(p)
    lo, go = omlp.loss_and_grads(q, bf16_round(X), Y.astype(np.float64))
    # the hidden activations and the two deltas are rounded to BF16 (2^-9 each)
    assert abs(loss - lo) <= 1e-2 * lo
    for k in ("W1", "b1", "W2", "b2"):
        assert rel_fro(_np(grads[k]), go[k]) <= 2e-2, k
    # element by element, against the size of what is added up: a tile of rows left
    # out of a column is a share of it
    y, (_, z1, _, z2) = omlp.forward(q, bf16_round(X))
    dz2 = 2.0 / y.size * (y - Y) * omlp.softplus_grad(z2)
    dz1 = (dz2 @ q["W2"]) * omlp.gelu_grad(z1)
    for k, d in (("b1", dz1), ("b2", dz2)):
        assert np.all(np.abs(_np(grads[k]) - go[k]) <= 2e-2 * np.abs(d).sum(axis=0)), k
