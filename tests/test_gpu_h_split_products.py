"""The H update of 65,536 rows or more (BF16 parts) where an error of one product
shows: a row of H with one entry that is not zero, in the last column, takes from its
first column one product, S[0, K-1] h, and from the same product in R."""
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [33, 100, 200, 400, 509])
def test_single_products(cuda, K):
    D, V = 65536, K + 40
    g = torch.Generator(device=cuda).manual_seed(K)
    W = torch.rand(V, K, generator=g, device=cuda) + 1e-3
    h = 0.1 + torch.rand(D, generator=g, device=cuda)
    H0 = torch.zeros(D, K, device=cuda)
    H0[:, K - 1] = h
    Wn = W.double() / W.double().norm(dim=0)
    A = (Wn[:, K - 1:] * 1.01 * h.double()).float()  # R[:, 0] = 1.01 S[0, K-1] h
    plan = Plan(Matrix(V, D, dense=A), W, H0)
    plan.half("H")
    x = plan.intermediates()
    sh = x["S"][0, K - 1].double() * h.double()
    ref = x["R"][:, 0].double() - sh
    assert float(ref.min()) > 0
    # 2^-24 for what the parts' products leave out and 2^-24 for the product's rounding,
    # the small products' own roundings, and 2^-24 of the difference
    err = (plan.Ht[:, 0].double() - ref).abs()
    assert bool((err <= 2.0 ** -23 * (1 + 2.0 ** -4) * sh + 2.0 ** -24 * ref).all()), float((err / sh).max())
    plan.close()
