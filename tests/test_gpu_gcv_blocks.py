"""GPU parity of the GCV search of Solve-OF where its factorization changes form: the register
blocks hold up to 16, 24 and 32 columns, and G_Y without a Cholesky factor takes the general
path.  Bars as in test_gpu_solve_of: fixed lambda 1e-10 (only summation order differs), GCV flows
1e-8 while the choices agree, every choice as good as the oracle's on the oracle's functional to
1e-9 (1e-6 where G_Y is singular: there the numerator is ||b||^2 - 2 z.d + z^T G_Y z, whose
cancellation loses up to that much)."""
import numpy as np
import pytest

from gpu_helpers import assert_close, pack
from test_gpu_solve_of import B, _frames, _gcv_choices_valid, _oracle, _run  # noqa: F401

pytestmark = pytest.mark.gpu

# the last projected solve has 16, 17, 24, 25 and 32 columns
SPLITS = [(6, 11), (6, 12), (8, 17), (8, 18), (9, 24)]


@pytest.mark.parametrize("ell,n_iter", SPLITS)
def test_fixed_lambda_at_block_edges(B, ell, n_iter):  # noqa: F811
    import torch
    us = _frames(31, [(2, 12, 13), (3, 11, 9)])   # even and odd pixel counts
    got, _, _ = _run(B, us, torch.float64, ell=ell, n_iter=n_iter, fixed_lambda=0.03)
    exp, _ = _oracle(us, ell, n_iter, 0.03)
    assert_close(got, pack(exp), 1e-10)


@pytest.mark.parametrize("ell,n_iter", SPLITS)
def test_gcv_at_block_edges(B, ell, n_iter):  # noqa: F811
    import torch
    us = _frames(32, [(2, 12, 13), (3, 11, 9)])
    got, _, lam = _run(B, us, torch.float64, ell=ell, n_iter=n_iter)
    exp, elams = _oracle(us, ell, n_iter)
    if _gcv_choices_valid(lam, us, ell, n_iter, 1e-9) == len(elams):
        assert_close(got, pack(exp), 1e-8)


def test_singular_data_rows(B):  # noqa: F811
    """One textured patch on a flat frame: Y has fewer independent rows than the basis columns."""
    import torch
    r = np.random.default_rng(33)
    u = np.zeros((2, 12, 11))
    u[0, 4:6, 4:6] = r.uniform(0.5, 1.0, (2, 2))
    u[1, 4:6, 5:7] = u[0, 4:6, 4:6]
    got, _, lam = _run(B, [u], torch.float64, ell=4, n_iter=28)
    assert np.all(np.isfinite(got)) and np.all(lam > 0)
    _gcv_choices_valid(lam, [u], 4, 28, 1e-6)
