"""Accuracy of the FP32 products that run as products of three BF16 parts, where an
error of a part is not hidden by a long sum's roundings, against 64 bits."""
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=g.device)


def _products(A, W, Ht):
    """R and P of a plan and their relative errors."""
    plan = Plan(Matrix(*A.shape, dense=A), W, Ht)
    W0, H0 = plan.W.double().clone(), plan.Ht.clone()
    plan.half("H")
    R = plan.intermediates()["R"].double()
    plan.Ht.copy_(H0)
    plan.half("W")
    P = plan.intermediates()["P"].double()
    plan.close()
    for x, ref in ((R, A.double().T @ W0), (P, A.double() @ H0.double())):
        m = ref != 0
        yield (x - ref)[m] / ref[m]


@pytest.mark.parametrize("V,D,K", [(3000, 3000, 64), (1000, 800, 16), (301, 5003, 240), (8, 1000, 4)])
def test_single_products(cuda, V, D, K):
    """At most one nonzero in a row and a column of A: every entry of R and P is one
    product.  2^-24 for what the parts' products leave out, 2^-24 for the rounding of
    the result, and the small products' own roundings (2^-8 of that each)."""
    g = torch.Generator(device=cuda).manual_seed(V + D + K)
    n = min(V, D)
    A = torch.zeros(V, D, device=cuda)
    A[torch.randperm(V, generator=g, device=cuda)[:n], torch.randperm(D, generator=g, device=cuda)[:n]] = \
        0.1 + _rand(g, n)
    for e in _products(A, _rand(g, V, K) + 1e-3, _rand(g, D, K) + 1e-3):
        assert float(e.abs().max()) <= 2.0 ** -23 * (1 + 2.0 ** -4)


@pytest.mark.parametrize("V,D,K", [(3000, 3000, 64), (2801, 3003, 50)])
def test_split_sums(cuda, V, D, K):
    """Contractions in eight splits or more: a split's sum of a few steps is off by
    about a rounding of its own, the splits' errors are independent (2^-25 together, RMS)
    and adding the partials rounds once (2^-25.3): in all below 2^-24."""
    g = torch.Generator(device=cuda).manual_seed(V + D + K)
    A = _rand(g, V, D).pow(4)
    for e in _products(A, _rand(g, V, K).pow(3) + 1e-3, _rand(g, D, K).pow(3) + 1e-3):
        assert float((e * e).mean().sqrt()) <= 2.0 ** -24
