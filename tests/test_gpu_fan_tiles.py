"""GPU parity of the fan-beam projector where its kernels change form: frames of one pixel tile and of
many (one or two pixels per lane of the transpose), rays split over four, two and one waves, frame
sides and line groups that end within a tile, detectors wider and narrower than the frame, windows too
wide for the staged form, and a source close to the frame.  Bars as in test_gpu_fan: FP64 1e-12,
FP32 1e-5 of the projection of |u|."""
import numpy as np
import pytest

from gpu_helpers import TOL32, TOL64, assert_close, dev, host, pack, roundtrip32
from oracle import forward

pytestmark = pytest.mark.gpu

CASES = [
    # sizes, angles, bins, geometry
    ([(1, 9, 33), (2, 2, 3)], 5, [45, 7], dict(dso=60.0, dsd=100.0, du=100.0 / 60.0)),
    ([(2, 47, 31)], 16, [81], dict(dso=50.0, dsd=80.0, du=1.6)),
    ([(1, 40, 52)], 17, [19], dict(dso=70.0, dsd=120.0, du=1.0)),        # narrow detector
    ([(1, 24, 24)], 6, [301], dict(dso=40.0, dsd=80.0, du=0.25)),         # 8 bins per pixel: not staged
    ([(1, 36, 34)], 9, [91], dict(dso=27.0, dsd=60.0, du=2.0)),          # source 2 px outside the frame
    ([(1, 20, 20)], 4, [25], dict(dso=900.0, dsd=2000.0, du=4.0)),        # 2 pixels per bin
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("which", ["f64", "f32"])
def test_forward_and_transpose(case, which):
    import torch
    from paper_2501_12497_amd import binding as B
    sizes, na, nb, geo = CASES[case]
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    r = np.random.default_rng(case)
    angs = [r.uniform(0, 2 * np.pi, (nt, na)) for nt, _, _ in sizes]
    for a in angs:
        a[0, :2] = 0.0, np.pi / 4
    us = [r.standard_normal(s) for s in sizes]
    bs = [r.standard_normal((s[0], na, n)) for s, n in zip(sizes, nb)]
    if which == "f32":
        us, bs = [roundtrip32(u) for u in us], [roundtrip32(b) for b in bs]
    plan = B.plan_fan(B.Stack(sizes), [na] * len(sizes), nb, np.concatenate([a.ravel() for a in angs]), **geo)
    fwd = lambda v: pack([forward.fan_fwd(u, a, n, **geo) for u, a, n in zip(v, angs, nb)])
    adj = lambda v: pack([forward.fan_adj(b, a, s[1], s[2], **geo) for b, a, s in zip(v, angs, sizes)])
    assert_close(host(B.apply_A(plan, dev(pack(us), dt))), fwd(us), tol, fwd([np.abs(u) for u in us]))
    assert_close(host(B.apply_At(plan, dev(pack(bs), dt))), adj(bs), tol, adj([np.abs(b) for b in bs]))


@pytest.mark.parametrize("nt", [1, 20, 40])
def test_ray_splits_and_tiles_agree(nt):
    """Frames of 130 x 130 with 24 angles and 187 bins: 1 frame (rays over four waves, one pixel per
    lane), 20 (two waves) and 40 (one wave, two pixels per lane) give each frame the same data to
    FP64 rounding."""
    import torch
    from paper_2501_12497_amd import binding as B
    geo = dict(dso=200.0, dsd=330.0, du=1.65)
    r = np.random.default_rng(9)
    u1, b1 = r.standard_normal((130, 130)), r.standard_normal((24, 187))
    ang = np.arange(24) * (np.pi / 24) + 0.1
    stack = B.Stack.single(nt, 130, 130)
    plan = B.plan_fan(stack, [24], [187], np.tile(ang, nt), **geo)
    got = host(B.apply_A(plan, dev(np.tile(u1.ravel(), nt), torch.float64))).reshape(nt, -1)
    exp = forward.fan_fwd(u1[None], ang[None], 187, **geo).ravel()
    sc = forward.fan_fwd(np.abs(u1)[None], ang[None], 187, **geo).ravel()
    for t in {0, nt - 1}:
        assert_close(got[t], exp, TOL64, sc)
    got = host(B.apply_At(plan, dev(np.tile(b1.ravel(), nt), torch.float64))).reshape(nt, -1)
    exp = forward.fan_adj(b1[None], ang[None], 130, 130, **geo).ravel()
    sc = forward.fan_adj(np.abs(b1)[None], ang[None], 130, 130, **geo).ravel()
    for t in {0, nt - 1}:
        assert_close(got[t], exp, TOL64, sc)
