"""GPU parity of the projected solve beyond 64 columns at the edges of its 16-column blocks and of its waves' 64 rows, up
to the largest basis: a fixed lambda against the dense solve and the discrepancy root, at a condition number of about
1e8; tolerances as for the small ones (the solution to the condition number times 1e-14, the root to 1e-9)."""
import numpy as np
import pytest

from oracle import mmgks
from test_gpu_projected_blocks import _system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [65, 79, 80, 81, 112, 127, 128, 129, 144, 191, 192, 193, 240, 255, 256])
def test_big_block_edges(K):
    import torch
    from paper_2501_12497_amd import binding as B
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    RA, RT, b = _system(K, 500 + K)
    GA, GT, d, bb = RA.T @ RA, RT.T @ RT, RA.T @ b, float(b @ b)
    M = GA + 1e-3 * GT
    exp = np.linalg.solve(M, d)
    z, got, D2, st = B.projected_solve(dev(GA), dev(GT), dev(d), bb, 0.0, fixed_lambda=1e-3)
    assert st == 0 and got == 1e-3
    assert np.abs(z.cpu().numpy() - exp).max() <= 1e-14 * np.linalg.cond(M) * np.abs(exp).max() + 1e-14
    assert abs(D2 - float(np.sum((RA @ exp - b) ** 2))) <= 1e-12 * bb
    QA, RAq = np.linalg.qr(RA)
    _, RTq = np.linalg.qr(RT)
    lo = mmgks.discrepancy(RAq, QA.T @ b, RTq, 1e-8, bb)[0]
    hi = mmgks.discrepancy(RAq, QA.T @ b, RTq, 1e8, bb)[0]
    target = 0.7 * lo + 0.3 * hi
    lam0, st0 = mmgks.dp_lambda(RAq, QA.T @ b, RTq, bb, target)
    assert st0 == 0
    for prev in (0.0, lam0 * 1.3):
        z, lam, D2, st = B.projected_solve(dev(GA), dev(GT), dev(d), bb, target * target, prev_lambda=prev)
        assert st == 0
        assert abs(lam - lam0) <= 1e-9 * lam0
        assert abs(np.sqrt(D2) - target) <= 1e-10 * target


def test_big_no_factor_is_reported():
    import torch
    from paper_2501_12497_amd import binding as B
    K = 100
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    for at in (0, 63, 64, K - 1):
        G = np.eye(K)
        G[at, at] = -1.0
        z, lam, D2, st = B.projected_solve(dev(G), dev(np.zeros((K, K))), dev(np.ones(K)), float(K), 0.0,
                                           fixed_lambda=1.0)
        assert st == 4
        assert not z.cpu().numpy().any()
