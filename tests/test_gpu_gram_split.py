"""Grams of 65,536 rows and more (BF16 parts) at the edges of the kernel's forms -- one
unit with eight row shares up to 64 columns, two shares up to 256, two units per wave
above -- and of its stages and chunks, against 64-bit Grams of the same factors."""
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu

SHAPES = [(65536, 1), (65537, 31), (65663, 40), (65600, 64), (65537, 65), (65663, 129), (100000, 200),
          (65600, 256), (65537, 257), (65551, 400), (300000, 400), (65537, 509), (65536, 512)]


def _gram(cuda, D, K, Ht):
    """Q = H H^T of the W half, and its 64-bit value."""
    g = torch.Generator(device=cuda).manual_seed(7 * D + K)
    V = K + 40
    A = torch.rand(V, D, generator=g, device=cuda)
    W = torch.rand(V, K, generator=g, device=cuda) + 1e-3
    plan = Plan(Matrix(V, D, dense=A), W, Ht)
    H0 = plan.Ht.double()
    ref = H0.T @ H0
    plan.half("W")
    q = plan.intermediates()["Q"].double()
    plan.close()
    assert torch.equal(q, q.T)
    return q, ref


@pytest.mark.parametrize("D,K", SHAPES)
def test_gram(cuda, D, K):
    """Positive terms.  A chunk's sum (3,600 rows at most) is rounded three times per 16
    rows, at sizes that grow to its own: by chance 2^-24 sqrt(3 * 3600 / 16 / 3) = 2^-20.1
    of it, and over the chunks (64 or more, independent) 2^-23.1; some ten additions of
    chunks near the full size add 2^-23.4 at most.  2^-22 RMS, eight times that at most."""
    g = torch.Generator(device=cuda).manual_seed(D + K)
    q, ref = _gram(cuda, D, K, torch.rand(D, K, generator=g, device=cuda).pow(3))
    e = (q - ref) / ref
    assert float((e * e).mean().sqrt()) <= 2.0 ** -22
    assert float(e.abs().max()) <= 2.0 ** -19


@pytest.mark.parametrize("D,K", [(65600, 64), (100000, 200), (65551, 400)])
def test_single_products(cuda, D, K):
    """One row of H is not zero: 2^-24 for what the parts' products leave out, 2^-24 for
    the result's rounding, and the small products' own roundings."""
    g = torch.Generator(device=cuda).manual_seed(D + K)
    Ht = torch.zeros(D, K, device=cuda)
    Ht[D // 2 + 1] = 0.1 + torch.rand(K, generator=g, device=cuda)
    q, ref = _gram(cuda, D, K, Ht)
    assert float(((q - ref) / ref).abs().max()) <= 2.0 ** -23 * (1 + 2.0 ** -4)


@pytest.mark.parametrize("V,K", [(65600, 64), (65600, 200), (65663, 400)])
def test_not_finite(cuda, V, K):
    """S of a W with an infinity and a value above the largest BF16: as the values' own
    products give it, and bit for bit as before in the other columns."""
    g = torch.Generator(device=cuda).manual_seed(V + K)
    A = torch.rand(V, K + 3, generator=g, device=cuda)
    plan = Plan(Matrix(V, K + 3, dense=A), torch.rand(V, K, generator=g, device=cuda) + 1e-3,
                torch.rand(K + 3, K, generator=g, device=cuda))
    plan.half("H")
    clean = plan.intermediates()["S"].clone()
    plan.W[5, 3], plan.W[V - 1, K - 2] = float("inf"), 3.4e38
    ref = plan.W.double().T @ plan.W.double()
    plan.half("H")
    S = plan.intermediates()["S"].double()
    plan.close()
    assert torch.equal(torch.isinf(S), torch.isinf(ref.float()))
    m = torch.isfinite(ref.float())
    assert float(((S - ref)[m] / ref[m]).abs().max()) <= 2.0 ** -19
    keep = torch.ones(K, dtype=torch.bool, device=cuda)
    keep[3] = keep[K - 2] = False
    assert torch.equal(S[keep][:, keep], clean[keep][:, keep].double())
