"""GPU parity of the any-width gradient pair and the 9-tap blur at the edges of their quads, waves and
tiles: widths around multiples of 4, of a wave (256 pixels) and of a blur tile, frames of 2 rows, rows
that end in the middle of a wave, and arrays that start off a 16-byte boundary.  FP64 1e-12, FP32 1e-5
of the operator applied to absolute values."""
import numpy as np
import pytest

from gpu_helpers import TOL32, TOL64, assert_close, host, pack, roundtrip32
from oracle import forward, regops

pytestmark = pytest.mark.gpu

SIZES = [(1, 2, 2), (2, 2, 3), (1, 5, 4), (1, 9, 5), (2, 33, 7), (1, 64, 65), (1, 31, 129), (1, 67, 255), (1, 3, 257),
         (1, 70, 62)]


def _dev(x, dt, shift):
    """x on the GPU, starting `shift` elements after an aligned address."""
    import torch
    t = torch.zeros(x.size + 4, dtype=dt, device="cuda")
    t[shift:shift + x.size] = torch.as_tensor(x, dtype=dt, device="cuda")
    return t[shift:shift + x.size]


@pytest.mark.parametrize("sizes,shift", [(SIZES, 0), (SIZES, 1), ([(2, 9, 8), (1, 6, 260)], 3)])
@pytest.mark.parametrize("which", ["f64", "f32"])
def test_gradient_pair(which, sizes, shift):
    import torch
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    r = np.random.default_rng(4)
    rt = roundtrip32 if which == "f32" else np.asarray
    us = [rt(r.standard_normal(s)) for s in sizes]
    gx = [rt(r.standard_normal((t, ny, nx - 1))) for t, ny, nx in sizes]
    gy = [rt(r.standard_normal((t, ny - 1, nx))) for t, ny, nx in sizes]
    wx = [rt(r.uniform(0.5, 2.0, g.shape)) for g in gx]
    wy = [rt(r.uniform(0.5, 2.0, g.shape)) for g in gy]
    stack = B.Stack(sizes)
    d = lambda a: _dev(pack(a), dt, shift)
    for w in (False, True):
        kw = dict(wx=d(wx), wy=d(wy)) if w else {}
        ow = lambda a, b: (a, b) if w else (None, None)
        ox, oy = B.apply_grad(stack, d(us), **kw)
        exp = [regops.grad_fwd(u, *ow(a, b)) for u, a, b in zip(us, wx, wy)]
        # |Op||u|: both ends of a difference, weighted
        ax = [np.abs(u[:, :, 1:]) + np.abs(u[:, :, :-1]) for u in us]
        ay = [np.abs(u[:, 1:]) + np.abs(u[:, :-1]) for u in us]
        if w:
            ax, ay = [a * b for a, b in zip(ax, wx)], [a * b for a, b in zip(ay, wy)]
        assert_close(host(ox), pack([e[0] for e in exp]), tol, pack(ax))
        assert_close(host(oy), pack([e[1] for e in exp]), tol, pack(ay))
        got = B.apply_grad(stack, gx=d(gx), gy=d(gy), transpose=True, **kw)
        exp = pack([regops.grad_adj(a, b, *ow(p, q)) for a, b, p, q in zip(gx, gy, wx, wy)])
        sx = [np.abs(a) * (p if w else 1.0) for a, p in zip(gx, wx)]
        sy = [np.abs(b) * (q if w else 1.0) for b, q in zip(gy, wy)]
        scale = []
        for a, b in zip(sx, sy):
            s = np.zeros((a.shape[0], a.shape[1], b.shape[2]))
            s[:, :, 1:] += a
            s[:, :, :-1] += a
            s[:, 1:] += b
            s[:, :-1] += b
            scale.append(s)
        assert_close(host(got), exp, tol, pack(scale))


@pytest.mark.parametrize("choice", range(5))
@pytest.mark.parametrize("which", ["f64", "f32"])
def test_blur(which, choice):
    import torch
    from paper_2501_12497_amd import binding as B
    dt, tol = (torch.float64, TOL64) if which == "f64" else (torch.float32, TOL32)
    r = np.random.default_rng(5)
    us = [r.standard_normal(s) for s in SIZES]
    if which == "f32":
        us = [roundtrip32(u) for u in us]
    plan = B.plan_blur(B.Stack(SIZES), 9, 2.0)
    plan.set_tile("blur", choice, dt)
    for shift in (0, 1):
        got = host(B.apply_A(plan, _dev(pack(us), dt, shift)))
        assert_close(got, pack([forward.blur(u) for u in us]), tol, pack([forward.blur(np.abs(u)) for u in us]))
