"""GPU parity of the tiled Horn-Schunck sweeps with every strip height: stacks for which the launch takes 3, 4 and 5
rows per strip, with frames that end at, before and after a tile's edge.  All forms give the same bits on a frame (a
sequence alone and as the first of a larger stack), and the oracle's values: FP64 1e-12, FP32 1e-4 norm-wise and 2e-4 in
the max-norm after 25 sweeps."""
import numpy as np
import pytest

from gpu_helpers import assert_close, dev, host, pack, roundtrip32
from oracle import optflow

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("first", [(2, 66, 105), (2, 104, 52), (2, 53, 113), (3, 64, 65)])
@pytest.mark.parametrize("rest", [[], [(8, 120, 120)], [(16, 128, 128)], [(16, 256, 256)], [(5, 500, 250)]])
def test_strip_heights(dtype, first, rest):
    import torch
    from paper_2501_12497_amd import binding as B
    dt = torch.float64 if dtype == "f64" else torch.float32
    r = np.random.default_rng(9)
    rt = roundtrip32 if dtype == "f32" else np.asarray
    t, ny, nx = first
    u, v = rt(r.standard_normal(first)), rt(r.standard_normal((t - 1, 2, ny, nx)))
    big = torch.Generator(device="cuda").manual_seed(1)
    more = sum((a - 1) * b * c for a, b, c in rest)
    alone, stack = B.Stack([first]), B.Stack([first] + rest)
    ua = dev(pack([u]), dt)
    us = torch.cat([ua, torch.randn(stack.n - alone.n, dtype=dt, device="cuda", generator=big)])
    va = dev(pack([v]), dt)
    vs = torch.cat([va, torch.zeros(2 * more, dtype=dt, device="cuda")])
    B.flow_update(alone, ua, va, 0.3, 25)
    B.flow_update(stack, us, vs, 0.3, 25)
    assert torch.equal(va, vs[:va.numel()])
    exp = pack([optflow.flow_update(u, v, 0.3, 25)])
    if dtype == "f64":
        assert_close(host(va), exp, 1e-12)
    else:
        assert_close(host(va), exp, 1e-4, tol_inf=2e-4)
