"""A pixel that is not finite reaches the rays that weigh on it and no others: the parallel-beam forward over frames
below and above the sizes where its row groups change form, at angles where neighbours of a ray have the weight 0
exactly and at others.  Other rays keep their values (FP64 1e-12, FP32 1e-5 of the projection of |u|)."""
import numpy as np
import pytest

from gpu_helpers import TOL32, TOL64, dev, host
from oracle import forward

pytestmark = pytest.mark.gpu

ANGLES = np.array([0.0, np.pi / 2, np.pi / 4, 3 * np.pi / 4, 0.1, 0.7, 1.2, 2.2, 3.0])


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("shape", [(24, 31), (130, 70), (400, 430)])
def test_forward(shape, value, which):
    import torch
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    r = np.random.default_rng(7)
    u = np.asarray(r.standard_normal((1,) + shape), dtype=np.float32).astype(np.float64)
    at = [(0, shape[0] // 2, shape[1] // 2), (0, 0, shape[1] // 3), (0, shape[0] // 3, shape[1] - 1)]
    nb = int(1.5 * max(shape))
    plan = B.plan_radon(B.Stack([(1,) + shape]), [ANGLES.size], [nb], ANGLES)
    d = np.arange(nb) - 0.5 * (nb - 1)
    for p in at:
        hit, rest, bad = np.zeros_like(u), u.copy(), u.copy()
        hit[p], rest[p], bad[p] = 1.0, 0.0, value
        w = forward.radon_fwd(hit, ANGLES[None], nb).ravel()
        exp = forward.radon_fwd(rest, ANGLES[None], nb).ravel()
        sc = forward.radon_fwd(np.abs(rest), ANGLES[None], nb).ravel()
        got = host(B.apply_A(plan, dev(bad, dt)))
        with np.errstate(invalid="ignore"):
            if np.isnan(value):
                assert np.isnan(got[w > 1e-6]).all()
            else:
                assert (got[w > 1e-6] == value).all()
            # a distance of 1 or more is a weight of 0, of more than 1 by rounding's measure off the axis
            tau = (p[2] - 0.5 * (shape[1] - 1)) * np.cos(ANGLES) + (p[1] - 0.5 * (shape[0] - 1)) * np.sin(ANGLES)
            out = (np.abs(tau[:, None] - d) >= np.where(ANGLES == 0.0, 1.0, 1.0 + 1e-6)[:, None]).ravel()
            assert np.isfinite(got[out]).all()
            assert np.all(np.abs(got[out] - exp[out]) <= tol * (sc[out] + 1e-2 * np.sqrt(np.mean(sc ** 2))))
