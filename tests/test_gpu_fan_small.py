"""GPU parity of the fan-beam transpose on frames of up to 48 pixels (half a tile per workgroup, candidates by the lane's
own half-width) and just beyond: sides at the edges of the half tiles, source distances that give from one to many
candidate rays per pixel, rays of both kinds.  FP64 1e-12, FP32 1e-5 of the transpose of |b|."""
import numpy as np
import pytest

from gpu_helpers import TOL32, TOL64, assert_close, dev, host, pack, roundtrip32
from oracle import forward

pytestmark = pytest.mark.gpu

SIZES = {"small": [(2, 8, 32), (1, 9, 33), (1, 17, 7), (1, 48, 48), (1, 2, 48)], "beyond": [(1, 49, 20), (2, 8, 33)]}
# source distance over the frame's side, magnification, pixels per bin
GEO = [(0.85, 1.6, 1.0), (1.5, 5 / 3, 1.0), (4.0, 1.5, 0.5), (1.2, 2.0, 2.0), (0.9, 1.3, 0.25)]


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("geo", range(len(GEO)))
@pytest.mark.parametrize("sizes", ["small", "beyond"])
def test_transpose(sizes, geo, which):
    import torch
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    r = np.random.default_rng(geo)
    sz = SIZES[sizes]
    side = max(max(s[1:]) for s in sz)
    far, mag, per = GEO[geo]
    g = dict(dso=far * side, dsd=far * mag * side, du=mag * per)
    na = 19
    nb = [int(1.3 * side / per)] * len(sz)
    angs = [np.concatenate([r.uniform(0, 2 * np.pi, (s[0], na - 2)), np.tile([0.0, np.pi / 4], (s[0], 1))], 1) for s in sz]
    bs = [r.standard_normal((s[0], na, n)) for s, n in zip(sz, nb)]
    if which == "f32":
        bs = [roundtrip32(b) for b in bs]
    plan = B.plan_fan(B.Stack(sz), [na] * len(sz), nb, pack(angs), **g)
    adj = lambda v: pack([forward.fan_adj(b, a, s[1], s[2], **g) for b, a, s in zip(v, angs, sz)])
    assert_close(host(B.apply_At(plan, dev(pack(bs), dt))), adj(bs), tol, adj([np.abs(b) for b in bs]))
