"""GPU parity of the one-wave projected solve at the edges of its 16-column blocks: a fixed lambda against the dense
solve, and the discrepancy root from a cold start and from good and bad previous values, at a condition number of about
1e8.  The root to 1e-9 (the search stops at steps of 1e-11 in log10 lambda); the solution to the condition number
times 1e-14.  A matrix without a Cholesky factor is reported, not solved."""
import numpy as np
import pytest

from oracle import mmgks

pytestmark = pytest.mark.gpu


def _system(K, seed):
    r = np.random.default_rng(seed)
    RA = r.standard_normal((2 * K + 30, K)) * np.logspace(0, -4, K)
    RT = r.standard_normal((2 * K + 20, K))
    b = RA @ r.standard_normal(K) + 0.05 * r.standard_normal(2 * K + 30)
    return RA, RT, b


@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65])
def test_block_edges(K):
    import torch
    from paper_2501_12497_amd import binding as B
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    RA, RT, b = _system(K, 300 + K)
    GA, GT, d, bb = RA.T @ RA, RT.T @ RT, RA.T @ b, float(b @ b)
    for lam in (1e-6, 1.0):
        z, got, D2, st = B.projected_solve(dev(GA), dev(GT), dev(d), bb, 0.0, fixed_lambda=lam)
        M = GA + lam * GT
        exp = np.linalg.solve(M, d)
        assert st == 0 and got == lam
        assert np.abs(z.cpu().numpy() - exp).max() <= 1e-14 * np.linalg.cond(M) * np.abs(exp).max() + 1e-14
        res = float(np.sum((RA @ exp - b) ** 2))
        assert abs(D2 - res) <= 1e-12 * bb
    QA, RAq = np.linalg.qr(RA)
    _, RTq = np.linalg.qr(RT)
    lo = mmgks.discrepancy(RAq, QA.T @ b, RTq, 1e-8, bb)[0]
    hi = mmgks.discrepancy(RAq, QA.T @ b, RTq, 1e8, bb)[0]
    target = 0.7 * lo + 0.3 * hi
    exp, st0 = mmgks.dp_lambda(RAq, QA.T @ b, RTq, bb, target)
    assert st0 == 0
    for prev in (0.0, exp * 1.3, exp * 1e6, exp * 1e-6):
        z, lam, D2, st = B.projected_solve(dev(GA), dev(GT), dev(d), bb, target * target, prev_lambda=prev)
        assert st == 0
        assert abs(lam - exp) <= 1e-9 * exp, prev
        assert abs(np.sqrt(D2) - target) <= 1e-10 * target


@pytest.mark.parametrize("K", [5, 16, 40, 64])
def test_no_factor_is_reported(K):
    import torch
    from paper_2501_12497_amd import binding as B
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    G = np.eye(K)
    G[K - 1, K - 1] = -1.0
    z, lam, D2, st = B.projected_solve(dev(G), dev(np.zeros((K, K))), dev(np.ones(K)), float(K), 0.0, fixed_lambda=1.0)
    assert st == 4
    assert not z.cpu().numpy().any()
