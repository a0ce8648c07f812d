"""The implicit basis step on both sides of the number of row chunks up to which one workgroup adds the partial inner
products itself (256 chunks: 65536 to 2097152 rows), with and without the explicit pass: the new basis vector is a unit
vector orthogonal to the basis (FP64, 1e-12 of the direction's norm), and the explicit pass runs only where it is due."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inside", [False, True])
@pytest.mark.parametrize("n", [129, 65536, 65537, 2097152, 2097153, 2200001])
def test_basis_extend_chunks(n, inside):
    import torch
    from paper_2501_12497_amd import binding as B
    K = 3
    g = torch.Generator(device="cuda").manual_seed(n)
    Q, _ = torch.linalg.qr(torch.randn(n, K, dtype=torch.float64, device="cuda", generator=g))
    Vs = Q.T.contiguous()
    w = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    for _ in range(2):
        w -= Q @ (Q.T @ w)
    w /= w.norm()
    x0 = Q @ torch.tensor([2.0, -1.0, 0.5], dtype=torch.float64, device="cuda") + (1e-6 if inside else 8.0) * w
    x = x0.clone()
    T = torch.zeros(256, 256, dtype=torch.float64, device="cuda")
    T[:K, :K] = torch.eye(K, dtype=torch.float64, device="cuda")
    rho2 = B.basis_extend(Vs, x, T)
    assert bool(torch.equal(x, x0)) != inside
    v = x / rho2 ** 0.5 + Q @ T[K, :K]
    tol = 1e-12 * (float(x0.norm()) / 1e-6 if inside else 1.0)   # of the direction's norm, as far as w is determined
    assert abs(float(v.norm()) - 1.0) <= tol
    assert float((Q.T @ v).abs().max()) <= 1e-12
    assert float((v - w).abs().max()) <= tol
    assert np.isfinite(rho2)
