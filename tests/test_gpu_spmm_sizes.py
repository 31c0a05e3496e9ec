"""Sparse products below and above the number of nonzeros from which fewer gathers are
in flight per step: the sums of a row do not depend on it, nor on how many segments
the other rows have."""
import numpy as np
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu

D = 2000


def _rows(lengths, r):
    """CSR of rows of the given lengths."""
    col = [np.sort(r.choice(D, n, replace=False)) for n in lengths]
    ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return ptr, np.concatenate(col).astype(np.int32), r.random(int(ptr[-1]), dtype=np.float32)


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("K", [1, 3, 4, 16, 33, 50, 64, 77, 96, 100, 128, 200, 257])
def test_rows_in_small_and_large_matrices(cuda, K, precision):
    r = np.random.default_rng(K)
    n = 3000
    lengths = r.integers(0, 300, n)
    lengths[[5, 77, n - 1]] = (D, 129, 128)
    lengths[[6, 78]] = 0
    ptr, col, val = _rows(np.concatenate([lengths, r.integers(100, 200, 1500)]), r)
    small = int(ptr[n])
    assert small < 524288 < int(ptr[-1])
    t = lambda x: torch.tensor(x, device=cuda)
    W, Ht = t(r.random((n + 1500, K), dtype=np.float32)) + 1e-3, t(r.random((D, K), dtype=np.float32))
    out = []
    for rows, nnz in ((n, small), (n + 1500, int(ptr[-1]))):
        A = Matrix(rows, D, rowptr=t(ptr[:rows + 1]), col=t(col[:nnz]), val=t(val[:nnz]))
        plan = Plan(A, W[:rows].clone(), Ht.clone(), precision=precision)
        plan.half("W")
        out.append(plan.intermediates()["P"][:n].clone())
        plan.close()
    assert torch.equal(out[0], out[1])
    cut = (lambda x: x.bfloat16().double()) if precision == "bf16" else (lambda x: x.double())
    dense = torch.zeros(n, D, dtype=torch.float64, device=cuda)
    row = torch.repeat_interleave(torch.arange(n, device=cuda), t(lengths))
    dense[row, t(col[:small]).long()] = cut(t(val[:small]))
    ref = dense @ cut(Ht)
    m = ref > 0
    # positive terms: a segment is at most 128 additions, 16 segments are added
    assert float(((out[0].double() - ref)[m] / ref[m]).abs().max()) <= 2.0 ** -24 * (128 + 16)
    assert bool((out[0][~m] == 0).all())
