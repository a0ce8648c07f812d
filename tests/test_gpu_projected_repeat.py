"""The projected solve beyond 64 columns gives the same bits every time: all waves that own rows factor a copy of a
diagonal block which one of them overwrites, so a wave that read it late would fail or change the solution.  The dense
solve bounds the value (the condition number times 1e-14, as for the other sizes)."""
import numpy as np
import pytest

from test_gpu_projected_blocks import _system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [65, 80, 128, 129, 192, 256])
def test_same_bits_every_time(K):
    import torch
    from paper_2501_12497_amd import binding as B
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    RA, RT, b = _system(K, 900 + K)
    GA, GT, d, bb = RA.T @ RA, RT.T @ RT, RA.T @ b, float(b @ b)
    args = (dev(GA), dev(GT), dev(d), bb, 0.0)
    M = GA + 1e-3 * GT
    exp = np.linalg.solve(M, d)
    first = None
    for _ in range(20):
        z, lam, D2, st = B.projected_solve(*args, fixed_lambda=1e-3)
        assert st == 0 and lam == 1e-3
        got = z.cpu().numpy()
        assert np.abs(got - exp).max() <= 1e-14 * np.linalg.cond(M) * np.abs(exp).max() + 1e-14
        if first is None:
            first = (got, D2)
        assert np.array_equal(got, first[0]) and D2 == first[1]
