"""The FP32 projectors' weights, seen through frames of a single pixel (no sum rounds anything): positions are good to
the rounding of the weight itself, not to that of a position held in FP32 (which is off by up to 1e-6 px)."""
import numpy as np
import pytest

from gpu_helpers import dev, host, pack
from oracle import forward

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
SIZES = [(24, 100, 90), (6, 33, 190), (6, 130, 17), (2, 400, 410)]
N_ANG = 20


def _frames(r):
    us = []
    for nt, ny, nx in SIZES:
        u = np.zeros((nt, ny, nx))
        u[np.arange(nt), r.integers(0, ny, nt), r.integers(0, nx, nt)] = 1.0
        us.append(u)
    return us, [np.concatenate([r.uniform(0, 2 * np.pi, (s[0], N_ANG - 3)), np.tile([0.0, np.pi / 4, 1e-7], (s[0], 1))], 1)
                for s in SIZES]


def test_parallel_beam():
    import torch
    from paper_2501_12497_amd import binding as B
    us, angs = _frames(np.random.default_rng(5))
    nb = [int(1.5 * max(s[1:])) for s in SIZES]
    plan = B.plan_radon(B.Stack(SIZES), [N_ANG] * len(SIZES), nb, pack(angs))
    exp = pack([forward.radon_fwd(u, a, n) for u, a, n in zip(us, angs, nb)])
    got = host(B.apply_A(plan, dev(pack(us), torch.float32)))
    # 1 - |a| x with x = |k - f| < sqrt(2), |a| x < 1: |a| and the result rounded (1 unit of 2^-24 and half a one), f
    # to half a unit, k - f (or the constant it is folded into) to one
    assert exp.max() > 0.99 and np.abs(got - exp).max() <= 3.0 * U32


def test_fan_beam():
    import torch
    from paper_2501_12497_amd import binding as B
    us, angs = _frames(np.random.default_rng(6))
    geo = dict(dso=700.0, dsd=1100.0, du=1.5)
    nb = [int(1.5 * max(s[1:])) for s in SIZES]
    plan = B.plan_fan(B.Stack(SIZES), [N_ANG] * len(SIZES), nb, pack(angs), **geo)
    exp = pack([forward.fan_fwd(u, a, n, **geo) for u, a, n in zip(us, angs, nb)])
    got = host(B.apply_A(plan, dev(pack(us), torch.float32)))
    # a weight 1 - f or f (f and 1 - f rounded to half a unit each) times a length of at most 1.5 (one unit relative),
    # the product rounded (one unit relative)
    assert exp.max() > 1.0 and np.abs(got - exp).max() <= 1.5 * 3.0 * U32
