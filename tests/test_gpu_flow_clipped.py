"""Flows that leave the frame: every displaced source past the border is clipped to it, up to 64 of them into the cell of
a corner, more than a whole list's in a small frame pulled together.  L(v)^T against the oracle (FP64 1e-12, FP32 1e-5 of
the transpose of the magnitudes), the same bits from every tile shape; the reverse flow of the same velocities turned
inwards (many sources per target) equal in FP64, to 1e-6 in FP32."""
import numpy as np
import pytest

from gpu_helpers import TOL32, TOL64, assert_close, dev, host, pack, roundtrip32
from oracle import optflow, regops

pytestmark = pytest.mark.gpu

SIZES = [(2, 20, 23), (3, 33, 47), (2, 70, 64)]


def _flows(r, top, inward):
    out = []
    for nt, ny, nx in SIZES:
        y, x = np.mgrid[0:ny, 0:nx]
        c = np.stack([x - (nx - 1) / 2, y - (ny - 1) / 2])
        v = np.clip(c * (0.93 if inward else 4.0), -top, top) + r.uniform(-0.05, 0.05, (nt - 1, 2, ny, nx))
        out.append(-v if inward else v)
    return out


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("inward", [False, True])
@pytest.mark.parametrize("top", [3.4, 7.9])
def test_crowded_cells(top, inward, which):
    import torch
    from paper_2501_12497_amd import _lib, binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    r = np.random.default_rng(8)
    vs = _flows(r, top, inward)
    rs = [r.standard_normal((s[0] - 1,) + s[1:]) for s in SIZES]
    if which == "f32":
        vs, rs = [roundtrip32(v) for v in vs], [roundtrip32(x) for x in rs]
    stack = B.Stack(SIZES)
    plan = B.plan_blur(stack)
    dv = dev(pack(vs), dt)
    for direction in (1, -1):
        exp = pack([regops.flow_adj(x, v, s[0], direction) for x, v, s in zip(rs, vs, SIZES)])
        sc = pack([np.abs(regops.flow_adj(np.abs(x), v, s[0], direction)) + 2 * np.abs(x).max() for x, v, s in
                   zip(rs, vs, SIZES)])
        got = []
        for choice in range(4):
            plan.set_tile("flow_adj", choice, dt)
            got.append(host(B.apply_flow_op(stack, _lib.MMOF_FLOW_ADJ, direction, 0, None, dv, dev(pack(rs), dt))))
            assert np.array_equal(got[0], got[-1])
        assert_close(got[0], exp, tol, sc)
    back = host(B.reverse_flow(stack, dv))
    exp = pack([optflow.reverse_flow(v) for v in vs])
    if which == "f64":
        assert np.array_equal(back, exp)
    else:
        np.testing.assert_allclose(back, exp, rtol=1e-6, atol=1e-6 * top)
