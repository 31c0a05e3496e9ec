"""Grams S = W^T W and Q = H H^T at the edges of the kernel's forms (one unit with
eight row shares up to 64 columns, two shares up to 256, two units per wave above)
and of its stages and chunks, against 64-bit Grams of the same factors."""
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu

SHAPES = [(64, 64, 1), (130, 70, 31), (129, 65, 64), (40000, 130, 40), (1000, 300, 65), (257, 300, 128),
          (5000, 513, 129), (3001, 400, 200), (2000, 300, 256), (700, 300, 257), (5003, 600, 400),
          (600, 520, 512)]


@pytest.mark.parametrize("V,D,K", SHAPES)
def test_grams(cuda, V, D, K):
    g = torch.Generator(device=cuda).manual_seed(V + 7 * D + 31 * K)
    A = torch.rand(V, D, generator=g, device=cuda)
    W = torch.rand(V, K, generator=g, device=cuda).pow(3) + 1e-3
    Ht = torch.rand(D, K, generator=g, device=cuda).pow(3)
    plan = Plan(Matrix(V, D, dense=A), W, Ht)
    # positive terms: each addition costs at most 2^-23 of the sum; at most about
    # 60 of a chunk's and 32 of the chunks' additions happen near its full size
    tol = 2.0 ** -23 * 100
    for which, name, X in (("H", "S", plan.W), ("W", "Q", plan.Ht)):
        X0 = X.double()
        if which == "W":
            X0 = plan.Ht.double()
        plan.half(which)
        got, ref = plan.intermediates()[name].double(), X0.T @ X0
        assert float(((got - ref).abs() / ref).max()) < tol
        assert torch.equal(got, got.T)
    plan.close()
