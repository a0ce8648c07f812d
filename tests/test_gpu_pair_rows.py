"""GPU parity of the rows that belong to pairs of frames at the edges of their 4-pixel quads: frames of 1 to 9 pixels
width, of a tile (128, 256) and one beside it, a single frame among them, on and off a 16-byte boundary: the temporal
difference and its transpose, and the two flow directions, which share a kernel.  FP64 1e-12, FP32 1e-5 of the operator
applied to absolute values."""
import numpy as np
import pytest

from gpu_helpers import TOL32, TOL64, assert_close, host, pack, roundtrip32
from oracle import regops

pytestmark = pytest.mark.gpu

SIZES = [(3, 5, 2), (2, 3, 3), (1, 4, 4), (4, 6, 5), (2, 9, 7), (3, 2, 9), (2, 11, 127), (2, 3, 129), (3, 5, 257)]


def _dev(x, dt, shift):
    import torch
    t = torch.zeros(x.size + 4, dtype=dt, device="cuda")
    t[shift:shift + x.size] = torch.as_tensor(x, dtype=dt, device="cuda")
    return t[shift:shift + x.size]


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("which", ["f64", "f32"])
def test_rows_of_pairs(which, shift):
    import torch
    from paper_2501_12497_amd import _lib
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    rt = roundtrip32 if which == "f32" else np.asarray
    g = np.random.default_rng(50)
    us = [rt(g.standard_normal(s)) for s in SIZES]
    rs = [rt(g.standard_normal((s[0] - 1, s[1], s[2]))) for s in SIZES]
    vs = [rt(g.uniform(-2.0, 2.0, (s[0] - 1, 2, s[1], s[2]))) for s in SIZES]
    stack = B.Stack(SIZES)
    d = lambda a: _dev(pack(a), dt, shift)
    got = B.apply_tdiff(stack, d(us))
    assert_close(host(got), pack([regops.tdiff_fwd(u) for u in us]), tol,
                 pack([np.abs(u[1:]) + np.abs(u[:-1]) for u in us]))
    got = B.apply_tdiff(stack, d(rs), transpose=True)
    scale = []
    for x in rs:
        s = np.zeros((x.shape[0] + 1,) + x.shape[1:])
        s[1:] += np.abs(x)
        s[:-1] += np.abs(x)
        scale.append(s)
    assert_close(host(got), pack([regops.tdiff_adj(x) for x in rs]), tol, pack(scale))
    for direction in (1, -1):
        got = B.apply_flow_op(stack, _lib.MMOF_FLOW_FWD, direction, _lib.MMOF_INTERP_BILINEAR, d(us), d(vs))
        exp = pack([regops.flow_fwd(u, v, direction) for u, v in zip(us, vs) if len(v)])
        # |W||src| + |sub|: a bilinear sample of absolute values
        scale = pack([np.abs(regops.flow_fwd(np.abs(u), v, direction)) +
                      2 * np.abs(u[:-1] if direction > 0 else u[1:]) for u, v in zip(us, vs) if len(v)])
        assert_close(host(got), exp, tol, scale)
