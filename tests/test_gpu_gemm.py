"""Dense products R = A^T W and P = A H^T at the edges of the matrix-core GEMM's
tile forms (128 x 128, 64 x 64, 128 x 32), ragged contractions, odd leading
dimensions, and leading dimensions past the 32-bit tile offsets, against 64-bit
products of the same inputs."""
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu

SHAPES = [(1000, 800, 16), (257, 3001, 33), (4096, 301, 129), (5003, 1999, 240), (70, 65, 5),
          (640, 384, 64), (33, 31, 31), (2000, 130, 127)]


def _problem(cuda, V, D, K):
    g = torch.Generator(device=cuda).manual_seed(V + 7 * D + 31 * K)
    A = torch.rand(V, D, generator=g, device=cuda).pow(4)
    W = torch.rand(V, K, generator=g, device=cuda).pow(3) + 1e-3
    Ht = torch.rand(D, K, generator=g, device=cuda).pow(3)
    return A, W, Ht


def _rel(x, ref):
    return float(((x.double() - ref).abs() / ref).max())


def _check(cuda, V, D, K, precision):
    A, W, Ht = _problem(cuda, V, D, K)
    plan = Plan(Matrix(V, D, dense=A), W, Ht, precision=precision)
    cut = (lambda t: t.bfloat16().double()) if precision == "bf16" else (lambda t: t.double())
    # every term is positive, so each addition costs at most one rounding of the
    # sum (2^-23: the matrix cores may cut instead of round): a step of 32 (FP32)
    # or 16 (BF16) terms is one, and 32 cover a step's inside, the split sums and
    # the dropped products
    tol = lambda n: 2.0 ** -23 * (n / (16 if precision == "bf16" else 32) + 32)
    W0 = plan.W.clone()
    plan.half("H")
    assert _rel(plan.intermediates()["R"], cut(A).T @ cut(W0)) < tol(V)
    H1 = plan.Ht.clone()
    plan.half("W")
    ref = cut(A) @ cut(H1)
    assert _rel(plan.intermediates()["P"], ref) < tol(D)
    plan.close()


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("V,D,K", SHAPES)
def test_dense_products(cuda, V, D, K, precision):
    _check(cuda, V, D, K, precision)


def test_dense_products_far(cuda):
    """Rows of A 2^22 or more floats apart."""
    _check(cuda, 8, (1 << 22) + 3, 2, "fp32")


def test_dense_objective_edges(cuda):
    V, D, K = 300, 257, 33
    A, W, Ht = _problem(cuda, V, D, K)
    plan = Plan(Matrix(V, D, dense=A), W, Ht)
    half, rel = plan.objective()
    e2 = float(((A.double() - plan.W.double() @ plan.Ht.double().T) ** 2).sum())
    assert abs(half - 0.5 * e2) <= 1e-6 * e2
    assert abs(rel - (e2 / float((A.double() ** 2).sum())) ** 0.5) <= 1e-6 * rel
    plan.close()
