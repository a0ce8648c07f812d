"""A reverse velocity is a mean of velocities and no longer than the longest of them, also where the mean of many equal
ones rounds past them: columns of sources with one horizontal velocity and vertical ones that all lead to one pixel (and
the transposed case), below 8 pixels of displacement and, with one longer source in the frame, above.  FP64 1e-15 and FP32
1e-6 of the oracle's mean."""
import numpy as np
import pytest

from gpu_helpers import dev, host, roundtrip32
from oracle import optflow

pytestmark = pytest.mark.gpu


def _flow(r, far):
    """One pair of 64 x 640: a cluster of up to 15 sources every 20 columns; every other pixel moves out of the frame."""
    ny, nx = 64, 640
    v = np.zeros((1, 2, ny, nx))
    y, x = np.mgrid[0:ny, 0:nx]
    v[0, 0] = -7.0 * (x < 7)
    for i, cx in enumerate(range(30, nx - 20, 20)):
        q = int(r.integers(9, ny - 9))
        m, n = r.uniform(2.5, 7.4), int(r.integers(3, 8))
        rows = np.arange(q - n, q + n + 1)
        v[0, 0, rows, cx] = m
        v[0, 1, rows, cx] = q - rows
        v[0, :, q, int(np.rint(cx + m))] = 0.0, 1.0   # (the target's own velocity leads elsewhere)
    if far:
        v[0, 0, 0, 20] = 12.0
    return v


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("which", ["f64", "f32"])
def test_no_longer_than_the_sources(which, swap, far):
    import torch
    from paper_2501_12497_amd import binding as B
    dt = torch.float64 if which == "f64" else torch.float32
    v = _flow(np.random.default_rng(3), far)
    if swap:
        v = np.ascontiguousarray(v[:, ::-1].transpose(0, 1, 3, 2))
    if which == "f32":
        v = roundtrip32(v)
    ny, nx = v.shape[2:]
    got = host(B.reverse_flow(B.Stack.single(2, ny, nx), dev(v, dt))).reshape(v.shape)
    exp = optflow.reverse_flow(v)
    np.testing.assert_allclose(got, exp, rtol=1e-15 if which == "f64" else 1e-6, atol=0)
    y, x = np.mgrid[0:ny, 0:nx]
    tx, ty = np.rint(x + v[0, 0]).astype(int), np.rint(y + v[0, 1]).astype(int)
    ok = (tx >= 0) & (tx < nx) & (ty >= 0) & (ty < ny)
    for c in range(2):
        most = np.zeros((ny, nx))
        np.maximum.at(most, (ty[ok], tx[ok]), np.abs(v[0, c][ok]))
        assert (np.abs(got[0, c]) <= most).all()
