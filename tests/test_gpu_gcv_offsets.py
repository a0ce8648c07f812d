"""Solve-OF on stacks whose pairs of an odd pixel count come before pairs of an even one: the left vectors of the even
pairs, read two values at a time, then start at an odd element of their array (an even ell).  Bars as in
test_gpu_solve_of: with a fixed lambda the flows match to 1e-10 (p = q = 2) and 1e-8 (p = q = 1)."""
import pytest

from gpu_helpers import assert_close, pack
from test_gpu_solve_of import B, _frames, _oracle, _oracle_l1, _run  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [(2, 11, 9), (3, 14, 16), (2, 9, 7), (2, 8, 13)]


@pytest.mark.parametrize("ell", [3, 4, 10])
def test_even_pairs_after_odd_ones(B, ell):  # noqa: F811
    import torch
    us = _frames(41, SIZES)
    got, _, _ = _run(B, us, torch.float64, ell=ell, n_iter=7, fixed_lambda=0.05)
    assert_close(got, pack(_oracle(us, ell, 7, 0.05)[0]), 1e-10)
    got, _, _ = _run(B, us, torch.float64, ell=ell, n_iter=7, fixed_lambda=0.05, pq=1, eps=1e-3)
    assert_close(got, pack(_oracle_l1(us, ell, 7, 0.05, 1e-3)[0]), 1e-8)
