"""GPU parity of the parallel-beam projector.  The transpose on tiles of 32 rows; the forward at the edges of its row
groups and lines: frames of 2 and 3 columns, row counts around the groups of 4 and 8 and their split over waves, rays
along the axes, on the diagonal and nearly along an axis, detectors narrower and wider than the frame; every
angle grouping.  FP64 1e-12, FP32 1e-5 of the projection of |u|."""
import numpy as np
import pytest

from gpu_helpers import TOL32, TOL64, assert_close, dev, host, pack, roundtrip32
from oracle import forward

pytestmark = pytest.mark.gpu

SIZES = [(1, 2, 2), (1, 3, 2), (2, 2, 9), (1, 5, 3), (1, 8, 8), (1, 17, 33), (1, 64, 65), (1, 71, 66)]
BINS = [3, 7, 13, 4, 13, 41, 95, 61]
ANGLES = np.array([0.0, np.pi / 2, np.pi / 4, 3 * np.pi / 4, 1e-9, np.pi / 2 - 1e-9, 0.3, 1.3, 2.0, 2.9, 4.4])


@pytest.mark.parametrize("choice", range(4))
@pytest.mark.parametrize("which", ["f64", "f32"])
def test_forward(which, choice):
    import torch
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    r = np.random.default_rng(2)
    us = [r.standard_normal(s) for s in SIZES]
    if which == "f32":
        us = [roundtrip32(u) for u in us]
    angs = [np.tile(ANGLES, (s[0], 1)) for s in SIZES]
    plan = B.plan_radon(B.Stack(SIZES), [ANGLES.size] * len(SIZES), BINS, np.concatenate([a.ravel() for a in angs]))
    plan.set_tile("radon_fwd", choice, dt)
    got = host(B.apply_A(plan, dev(pack(us), dt)))
    exp = pack([forward.radon_fwd(u, a, n) for u, a, n in zip(us, angs, BINS)])
    sc = pack([forward.radon_fwd(np.abs(u), a, n) for u, a, n in zip(us, angs, BINS)])
    assert_close(got, exp, tol, sc)


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("shape,n_ang", [((260, 49, 33), 11), ((260, 49, 33), 35), ((1030, 49, 33), 35),
                                         ((90, 81, 97), 33), ((130, 33, 97), 11)])
def test_transpose_of_many_tiles(which, shape, n_ang):
    # stacks of 4 or more 32 x 32 tiles per CU (FP64) and of 16 or more (FP32, the third): rows and columns past whole
    # tiles, more angles than one chunk; the last shape overhangs so far that the lower tiles stay.  Ten frames, repeated.
    import torch
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    r = np.random.default_rng(3)
    nt, ny, nx = shape
    ang = np.concatenate([ANGLES, r.uniform(0, np.pi, 24)])[:n_ang]
    n_bins = 2 * int(max(ny, nx) / np.sqrt(2)) + 1
    b = r.standard_normal((10, n_ang, n_bins))
    if which == "f32":
        b = roundtrip32(b)
    angs = np.tile(ang, (10, 1))
    plan = B.plan_radon(B.Stack([shape]), [n_ang], [n_bins], np.tile(ang, nt))
    got = host(B.apply_At(plan, dev(np.tile(b.ravel(), nt // 10), dt)))
    exp = np.tile(forward.radon_adj(b, angs, ny, nx).ravel(), nt // 10)
    assert_close(got, exp, tol, np.tile(forward.radon_adj(np.abs(b), angs, ny, nx).ravel(), nt // 10))
