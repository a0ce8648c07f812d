"""GPU parity of the Horn-Schunck sweeps on frames that one workgroup holds whole (strips of 1 to 4
rows, up to 1024 of them) and just beyond, against the oracle.  Bars as for the tiled sweeps:
FP64 1e-12, FP32 1e-4 norm-wise and 2e-4 in the max-norm after 25 sweeps."""
import numpy as np
import pytest

from gpu_helpers import assert_close, dev, host, pack, roundtrip32
from oracle import optflow

pytestmark = pytest.mark.gpu

STACKS = [
    [(3, 32, 32)],                             # 1 row per strip, every thread used
    [(2, 33, 32)],                             # 2 rows, the last strip of one row
    [(2, 64, 32), (3, 5, 7)],                  # 2 rows, 1024 strips; a small frame beside it
    [(2, 49, 60)],                             # 3 rows (17 strips of 60)
    [(2, 64, 64)],                             # 4 rows, 1024 strips
    [(2, 63, 65)],                             # one column too many: tiled
    [(2, 2, 1024), (2, 130, 2)],               # long and flat
    [(1, 300, 310), (4, 20, 21)],              # a large frame without a pair
]


@pytest.mark.parametrize("sizes", STACKS)
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_flow_update(sizes, dtype):
    import torch
    from paper_2501_12497_amd import binding as B
    dt = torch.float64 if dtype == "f64" else torch.float32
    r = np.random.default_rng(5)
    us = [r.standard_normal(s) for s in sizes]
    vs = [r.standard_normal((t - 1, 2, ny, nx)) for t, ny, nx in sizes]
    if dtype == "f32":
        us, vs = [roundtrip32(u) for u in us], [roundtrip32(v) for v in vs]
    stack = B.Stack(sizes)
    v = dev(pack(vs), dt)
    B.flow_update(stack, dev(pack(us), dt), v, 0.3, 25)
    exp = pack([optflow.flow_update(u, w, 0.3, 25) for u, w in zip(us, vs)])
    if dtype == "f64":
        assert_close(host(v), exp, 1e-12)
    else:
        assert_close(host(v), exp, 1e-4, tol_inf=2e-4)


def test_more_sweeps_than_one_launch():
    """2100 sweeps (three launches) in place equal 2000 and then 100 more, bit for bit."""
    import torch
    from paper_2501_12497_amd import binding as B
    r = np.random.default_rng(6)
    stack = B.Stack([(3, 12, 10)])
    u = dev(r.standard_normal(stack.n), torch.float64)
    a = torch.zeros(2 * stack.n_pair_px, dtype=torch.float64, device="cuda")
    b = a.clone()
    B.flow_update(stack, u, a, 0.3, 2100)
    B.flow_update(stack, u, b, 0.3, 2000)
    B.flow_update(stack, u, b, 0.3, 100)
    assert torch.equal(a, b)
