"""H updates of documents with an infinite entry: every R' is infinite, the first
column takes it, and all others are clipped (infinity less infinity counts as less
than eps).  Other documents are as without."""
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu

EPS = 1e-16


def _run(cuda, n, K, sweeps):
    V = K + 30
    g = torch.Generator(device=cuda).manual_seed(n + K)
    W = torch.rand(V, K, generator=g, device=cuda) + 1e-3
    plan = Plan(Matrix(V, K + 2, dense=torch.rand(V, K + 2, generator=g, device=cuda)), W,
                torch.rand(K + 2, K, generator=g, device=cuda), eps=EPS)
    A = torch.rand(n, V, generator=g, device=cuda)
    H0 = torch.rand(n, K, generator=g, device=cuda)
    out = []
    for bad in (False, True):
        if bad:
            A[5, 7] = A[n - 1, 0] = float("inf")
        H = H0.clone()
        plan.foldin(Matrix(n, V, dense=A), H, init="given", n_sweeps=sweeps, trace=False)
        out.append(H)
    plan.close()
    same = torch.ones(n, dtype=torch.bool, device=cuda)
    same[5] = same[n - 1] = False
    return out[0][same], out[1][same], out[1][~same]


@pytest.mark.parametrize("K", [1, 5, 33, 100, 200])
def test_few_documents(cuda, K):
    clean, rest, bad = _run(cuda, 300, K, 1)
    assert torch.equal(clean, rest)
    assert bool(torch.isinf(bad[:, 0]).all())
    assert bool((bad[:, 1:] == torch.tensor(EPS, device=cuda)).all())


@pytest.mark.parametrize("K", [1, 33, 100, 400, 512])
def test_many_documents(cuda, K):
    """From 65,536 documents on the infinity turns to NaN in its own column."""
    clean, rest, bad = _run(cuda, 65600, K, 1)
    assert torch.equal(clean, rest)
    assert bool(torch.isnan(bad[:, 0]).all())
    assert bool((bad[:, 1:] == torch.tensor(EPS, device=cuda)).all())


@pytest.mark.parametrize("K", [40, 200])
def test_infinite_start(cuda, K, monkeypatch):
    """Infinities in H before the update: the split kernel against the rows kernel."""
    n, V = 65600, K + 30
    g = torch.Generator(device=cuda).manual_seed(K)
    W = torch.rand(V, K, generator=g, device=cuda) + 1e-3
    plan = Plan(Matrix(V, K + 2, dense=torch.rand(V, K + 2, generator=g, device=cuda)), W,
                torch.rand(K + 2, K, generator=g, device=cuda), eps=EPS)
    A = torch.rand(n, V, generator=g, device=cuda)
    H0 = torch.rand(n, K, generator=g, device=cuda)
    H0[torch.arange(K, device=cuda) * 7, torch.arange(K, device=cuda)] = float("inf")
    H0[n - 1, 1] = float("nan")
    out = []
    for kernel in (None, "rows"):
        if kernel:
            monkeypatch.setenv("NMF_H_KERNEL", kernel)
        H = H0.clone()
        plan.foldin(Matrix(n, V, dense=A), H, init="given", n_sweeps=1, trace=False)
        out.append(H)
    plan.close()
    assert torch.equal(torch.isnan(out[0]), torch.isnan(out[1]))
    assert torch.equal(torch.isinf(out[0]), torch.isinf(out[1]))
    m = torch.isfinite(out[1]).all(dim=1)
    a, b = out[0][m].double(), out[1][m].double()
    assert float((a - b).norm() / b.norm()) < 1e-5
