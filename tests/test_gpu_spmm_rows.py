"""The planned sparse products R = A^T W and P = A H^T on rows of every length around
a wave's steps and the list of 128 nonzeros, at ranks on both sides of each kernel
form and of a multiple of four, element by element against the 64-bit products."""
import numpy as np
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu

N = 1500
LENGTHS = [0, 1, 2, 15, 16, 17, 31, 33, 63, 65, 127, 128, 129, 256, 257, 1000, N, 0, 3, 64, 64, 0] + [
    i % 9 for i in range(400)]


@pytest.mark.parametrize("K", [1, 3, 4, 5, 31, 77, 128, 129, 130, 255, 301, 402])
@pytest.mark.parametrize("side", ["R", "P"])
def test_products(cuda, side, K):
    r = np.random.default_rng(K)
    m = len(LENGTHS)
    M = np.zeros((m, N), np.float32)
    for i, n in enumerate(LENGTHS):
        M[i, r.choice(N, size=n, replace=False)] = r.random(n).astype(np.float32) + 0.1
    A = M.T if side == "R" else M  # the long rows in A^T, or in A
    rows, col = np.nonzero(A)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=A.shape[0]))]).astype(np.int32)
    t = lambda x: torch.tensor(x, device=cuda)
    V, D = A.shape
    W, Ht = t(r.random((V, K)).astype(np.float32) + 0.1), t(r.random((D, K)).astype(np.float32) + 0.1)
    plan = Plan(Matrix(V, D, rowptr=t(ptr), col=t(col.astype(np.int32)), val=t(A[rows, col])), W, Ht)
    A64 = t(A.astype(np.float64))
    ref = A64.T @ plan.W.double() if side == "R" else A64 @ plan.Ht.double()
    plan.half("H" if side == "R" else "W")
    got = plan.intermediates()[side].double()
    # positive terms: at most 128 + 16 + 16 roundings of 2^-24 on a sum's path
    assert bool(((got - ref).abs() <= 160 * 2.0 ** -24 * ref).all())
    plan.close()
