"""GPU parity of the flow adjoint where its cells fill up: flows that converge on a point (from two sources per
cell to more than its list holds), odd and shifted frames, and every tile, which has to give the same bits.  The
radius of the flows is checked over one and several workgroups through a single large displacement.  FP64 1e-12,
FP32 1e-5 of the operator applied to absolute values."""
import numpy as np
import pytest

from gpu_helpers import TOL32, TOL64, assert_close, dev, host, pack, roundtrip32
from oracle import regops

pytestmark = pytest.mark.gpu


def _abs_adj(r, v, n_t, direction, interp):
    """|L|^T |r|: the warp part by the oracle on |r|, the direct part with its sign taken out."""
    a = np.abs(r)
    full = regops.flow_adj(a, v, n_t, direction, interp)
    if direction > 0:
        full[:-1] += 2 * a
    else:
        full[1:] += 2 * a
    return full


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("direction,interp", [(1, "bilinear"), (-1, "bilinear"), (1, "round")])
@pytest.mark.parametrize("pull,shape", [(0.3, (3, 40, 70)), (0.6, (2, 33, 65)), (0.9, (2, 31, 17)), (0.9, (3, 80, 81))])
def test_converging_flow(which, direction, interp, pull, shape):
    import torch
    from paper_2501_12497_amd import _lib
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    rt = roundtrip32 if which == "f32" else np.asarray
    nt, ny, nx = shape
    g = np.random.default_rng(7)
    # sources move a share `pull` of the way to the centre, 7.5 pixels at most (the LDS path)
    yy, xx = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
    c = np.stack([nx / 2 - xx, ny / 2 - yy]).astype(float)
    v = rt(np.clip(pull * c + 0.1 * g.standard_normal((nt - 1, 2, ny, nx)), -7.5, 7.5))
    r = rt(g.standard_normal((nt - 1, ny, nx)))
    stack = B.Stack.single(nt, ny, nx)
    ip = _lib.MMOF_INTERP_BILINEAR if interp == "bilinear" else _lib.MMOF_INTERP_ROUND
    exp = regops.flow_adj(r, v, nt, direction, interp)
    scale = _abs_adj(r, v, nt, direction, interp)
    plan = B.plan_blur(stack, 3, 1.0)
    dv, dr = dev(pack([v]), dt), dev(pack([r]), dt)
    first = None
    for tile in range(4):
        plan.set_tile("flow_adj", tile, dt)
        got = B.apply_flow_op(stack, _lib.MMOF_FLOW_ADJ, direction, ip, None, dv, dr)
        assert_close(host(got), exp.ravel(), tol, scale.ravel())
        first = got if first is None else first
        assert torch.equal(first, got), tile


@pytest.mark.parametrize("which", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(2, 8, 9), (2, 128, 128), (2, 128, 129), (3, 181, 187)])
def test_one_large_displacement(which, shape):
    """The radius is that of the largest displacement, wherever it stands (32768 values per workgroup)."""
    import torch
    from paper_2501_12497_amd import _lib
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    nt, ny, nx = shape
    stack = B.Stack.single(nt, ny, nx)
    r = roundtrip32(np.random.default_rng(8).standard_normal((nt - 1, ny, nx)))
    n = 2 * r.size
    for at in (0, n // 2 - 1, n - 1):
        v = np.zeros(n)
        v[at] = -5.25 if at else 5.25
        v = v.reshape(nt - 1, 2, ny, nx)
        for shift in (0, 1):   # (the flow on and off a 16-byte boundary)
            t = torch.zeros(n + 4, dtype=dt, device="cuda")
            t[shift:shift + n] = torch.as_tensor(v.ravel(), dtype=dt, device="cuda")
            got = B.apply_flow_op(stack, _lib.MMOF_FLOW_ADJ, 1, _lib.MMOF_INTERP_BILINEAR, None, t[shift:shift + n],
                                  dev(pack([r]), dt))
            exp = regops.flow_adj(r, v, nt, 1)
            assert_close(host(got), exp.ravel(), tol, _abs_adj(r, v, nt, 1, "bilinear").ravel())
