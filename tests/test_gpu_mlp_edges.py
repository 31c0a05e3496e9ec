"""Loss and gradients of one batch at the edges of the GEMM tiles (64 rows, odd
ranks and hidden sizes, one row), where the loss and the bias gradients are
summed in the products' epilogues, against the FP64 oracle at the same BF16-rounded
weights and inputs; and Adam's BF16 copies of the weights."""
import numpy as np
import pytest
import torch

from tests.gpu_util import bf16_round, rel_fro
from oracle import mlp as omlp
from paper_1904_07935_amd.api import Mlp
from tests.test_gpu_foldin_mlp import _bf16_params, _net, _np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,H", [(64, 32, 64), (65, 33, 40), (130, 7, 31), (257, 129, 65), (1, 5, 3),
                                   (700, 200, 512)])
def test_batch_gradients(cuda, N, K, H):
    rng = np.random.default_rng(N + K + H)
    p = _net(rng, K, H)
    net = Mlp(K, H, device=cuda, seed=None)
    net.set_masters(p)
    X = rng.random((N, K)).astype(np.float32)
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    Y = (0.2 * rng.random((N, K))).astype(np.float32)
    loss, grads, flat = net.loss_grad(torch.tensor(X, device=cuda), torch.tensor(Y, device=cuda))
    lo, go = omlp.loss_and_grads(_bf16_params(p), bf16_round(X), Y.astype(np.float64))
    # the hidden activations and the two deltas are rounded to BF16 (2^-9 each)
    assert abs(loss - lo) <= 1e-2 * lo
    for k in ("W1", "b1", "W2", "b2"):
        assert rel_fro(_np(grads[k]), go[k]) <= 2e-2, k
    net.adam_step(flat)
    w1, w2 = net.working_bf16()
    m = net.masters()
    assert torch.equal(w1, m["W1"].bfloat16()) and torch.equal(w2, m["W2"].bfloat16())
