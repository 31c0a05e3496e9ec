"""The fold-in product R' = A_new^T W on documents of every length around the wave's
list of 128 nonzeros (empty, one term, 127 .. 129, several segments, all terms),
at ranks on both sides of each kernel form, against the 64-bit product: the WTA
start with no sweeps returns max(eps, R')."""
import numpy as np
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu

V = 1500
LENGTHS = {
    "mixed": [0, 1, 127, 128, 129, 256, 257, 1000, V, 0, 3, 64, 64, 64, 5],
    "short": [i % 7 for i in range(997)],
    "empty": [0] * 70,
    "one": [V],
}


@pytest.mark.parametrize("K", [3, 77, 100, 200, 300])
@pytest.mark.parametrize("kind", sorted(LENGTHS))
def test_foldin_product(cuda, kind, K):
    r = np.random.default_rng(K)
    n = LENGTHS[kind]
    col = [np.sort(r.choice(V, size=k, replace=False)) for k in n]
    ptr = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    col = np.concatenate(col).astype(np.int32)
    val = (r.random(col.size) + 0.1).astype(np.float32)
    A = torch.tensor(r.random((V, 2 * K)).astype(np.float32) + 0.1, device=cuda)
    W = torch.tensor(r.random((V, K)).astype(np.float32) + 0.1, device=cuda)
    Ht = torch.tensor(r.random((2 * K, K)).astype(np.float32), device=cuda)
    plan = Plan(Matrix(V, 2 * K, dense=A), W, Ht)
    t = lambda x: torch.tensor(x, device=cuda)
    new = Matrix(len(n), V, rowptr=t(ptr), col=t(col), val=t(val))
    H = torch.full((len(n), K), -1.0, device=cuda)
    plan.foldin(new, H, init="wta", n_sweeps=0, trace=col.size > 0)
    D = torch.zeros(len(n), V, dtype=torch.float64)
    D[np.repeat(np.arange(len(n)), n), torch.tensor(col).long()] = torch.tensor(val).double()
    ref = (D.to(cuda) @ plan.W.double()).clamp(min=1e-16)
    # positive terms: at most 128 + 16 + 16 roundings of 2^-24 on a sum's path
    assert float(((H.double() - ref).abs() / ref).max()) < 160 * 2.0 ** -24
    plan.close()
