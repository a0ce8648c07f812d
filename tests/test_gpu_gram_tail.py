"""Weighted Gram matrices whose last row group ends within the rows a wave takes together, for a smoothing so small that
its square underflows: the rows beyond the last have no weight that could become infinite.  FP64 sums of positive terms
on the diagonal: 1e-12 of it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("eps", [1e-3, 1e-170])
@pytest.mark.parametrize("n,K", [(1, 1), (37, 3), (63, 4), (1003, 39), (70001, 40), (501, 41), (333, 70)])
def test_rows_past_the_last(n, K, eps, which):
    import torch
    from paper_2501_12497_amd import binding as B
    dt = torch.float64 if which == "f64" else torch.float32
    r = np.random.default_rng(n)
    X = r.standard_normal((K, n)).astype(np.float32).astype(np.float64)
    nu = (np.sign(r.standard_normal(n)) * r.uniform(0.1, 2.0, n)).astype(np.float32).astype(np.float64)
    G = B.weighted_gram(torch.as_tensor(X, dtype=dt, device="cuda"), torch.as_tensor(nu, dtype=dt, device="cuda"),
                        eps).cpu().numpy()
    exp = (X / np.sqrt(nu * nu + eps * eps)) @ X.T
    d = np.sqrt(np.diag(exp))
    assert np.abs(G - exp).max() <= 1e-12 * (d[:, None] * d[None]).max()
