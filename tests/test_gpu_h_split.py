"""The H update of 65,536 rows or more (split BF16 products, rows in registers) at
ranks around its 32-column tiles and row counts around its workgroups, against the
H loop in 64 bits from the same R and S: no further off than the FP32
rows-in-registers kernel on the same inputs."""
import pytest
import torch

from paper_1904_07935_amd.api import Matrix, Plan

pytestmark = pytest.mark.gpu


def _loop(H, R, S, eps):
    H = H.clone()
    for k in range(H.shape[1]):
        H[:, k] = torch.clamp(H[:, k] + R[:, k] - H @ S[:, k], min=eps)
    return H


@pytest.mark.parametrize("D,K", [(65536, 1), (65537, 5), (65663, 31), (65536, 32), (65600, 33), (66000, 100),
                                 (65551, 200), (65537, 400), (65536, 509), (65536, 512)])
def test_h_update_many_rows(cuda, D, K, monkeypatch):
    g = torch.Generator(device=cuda).manual_seed(K)
    V = K + 40
    W0 = torch.rand(V, K, generator=g, device=cuda).pow(6)
    W0[:K] += torch.eye(K, device=cuda)
    H0 = torch.rand(D, K, generator=g, device=cuda).pow(4)
    A = W0 @ (H0 * (torch.rand(D, K, generator=g, device=cuda) < 0.5)).T
    out = {}
    for name in ("split", "rows"):
        if name == "rows":
            monkeypatch.setenv("NMF_H_KERNEL", "rows")
        else:
            monkeypatch.delenv("NMF_H_KERNEL", raising=False)
        plan = Plan(Matrix(V, D, dense=A), W0.clone(), H0.clone(), eps=1e-16)
        plan.half("H")
        x = plan.intermediates()
        ref = _loop(H0.double(), x["R"].double(), x["S"].double(), 1e-16)
        out[name] = float((plan.Ht.double() - ref).norm() / ref.norm())
        assert float(plan.Ht.min()) > 0.0
        assert float((plan.Ht.double() - ref).abs().max() / ref.norm() * D ** 0.5) < 1e-3
        plan.close()
    assert out["split"] <= 1.5 * out["rows"] + 2.0 ** -24, out
