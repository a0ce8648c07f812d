"""Arguments of the Python binding: the ways a device can be named."""
import pytest
import torch

from paper_2501_12497_amd import binding as B


def test_device_index():
    assert B._device_index(3) == 3
    assert B._device_index("cuda:2") == 2
    assert B._device_index(torch.device("cuda", 1)) == 1
    with pytest.raises(ValueError):
        B._device_index("cpu")


@pytest.mark.gpu
@pytest.mark.parametrize("device", [None, 0, "cuda", "cuda:0", torch.device("cuda"), torch.device("cuda:0")])
def test_context_of_a_named_device(device):
    stack = B.Stack.single(2, 6, 5)
    u = torch.arange(60, dtype=torch.float64, device="cuda")
    for ctx in (B.Context(device), B.context(device)):
        gx, gy = B.apply_grad(stack, u, ctx=ctx)
        assert (gx == 1.0).all() and (gy == 5.0).all()
    assert B.context(device) is B.context()
