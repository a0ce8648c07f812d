"""GPU parity of the weighted Gram on columns of few rows, where waves have one step or none: one row to a few thousand,
at the edges of a step (16, 32 and 64 rows) and of a workgroup's steps, for the 4 x 4, the 16 x 16 and the tiled forms (the
last tile of 1 to 4 blocks);
and the form without allocation, which has its own limit of workgroups.  1e-12 of the largest entry."""
import numpy as np
import pytest

from oracle import mmgks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("K", [1, 4, 39, 40, 41, 64, 65, 80, 81, 97, 113, 130])
def test_few_rows(which, K):
    import torch
    from paper_2501_12497_amd import binding as B
    dt = torch.float64 if which == "f64" else torch.float32
    r = np.random.default_rng(K)
    for n in (1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1023, 4096, 5001):
        X, nu = r.standard_normal((K, n)), r.standard_normal(n)
        if which == "f32":
            X, nu = X.astype(np.float32).astype(np.float64), nu.astype(np.float32).astype(np.float64)
        Xd, nud = torch.as_tensor(X, dtype=dt, device="cuda"), torch.as_tensor(nu, dtype=dt, device="cuda")
        for w, args in ((np.ones(n), (Xd,)), (mmgks.mm_weights_sq(nu, 1e-3), (Xd, nud, 1e-3))):
            G = B.weighted_gram(*args).cpu().numpy()
            exp = X @ (w[:, None] * X.T)
            assert np.abs(G - exp).max() <= 1e-12 * np.abs(exp).max(), (n, len(args))


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("n", [64, 4096, 70000])
def test_without_allocation(which, n):
    import torch
    from paper_2501_12497_amd import _lib
    from paper_2501_12497_amd import binding as B
    from paper_2501_12497_amd._lib import check
    dt = torch.float64 if which == "f64" else torch.float32
    K = 39
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn(K, n, dtype=dt, device="cuda", generator=g)
    nu = torch.randn(n, dtype=dt, device="cuda", generator=g)
    G = torch.empty(K, K, dtype=torch.float64, device="cuda")
    ctx = B.context()
    ctx.bind()
    check(ctx.lib.mmof_weighted_gram_noalloc(ctx.h, _lib.MMOF_F64 if which == "f64" else _lib.MMOF_F32, n, K, X.data_ptr(),
                                             n, nu.data_ptr(), 1e-3, G.data_ptr(), K))
    Xh = X.cpu().numpy().astype(np.float64)
    exp = Xh @ (mmgks.mm_weights_sq(nu.cpu().numpy().astype(np.float64), 1e-3)[:, None] * Xh.T)
    assert np.abs(G.cpu().numpy() - exp).max() <= 1e-12 * np.abs(exp).max()
