"""Arguments of the Python binding: the ways a device can be named, the shapes of the projected matrices."""
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


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(5,), (1, 5), (5, 1), (1, 1), (), (4, 4), (6, 6), (2, 5, 5)])
@pytest.mark.parametrize("which", [0, 1])
def test_projected_matrices_of_another_shape_are_refused(shape, which):
    G = [torch.eye(5, dtype=torch.float64, device="cuda") for _ in range(2)]
    G[which] = torch.ones(shape, dtype=torch.float64, device="cuda")
    with pytest.raises(ValueError):
        B.projected_solve(G[0], G[1], torch.ones(5, dtype=torch.float64, device="cuda"), 5.0, 0.0, fixed_lambda=1.0)


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["plain", "one of a batch", "transposed view", "float32"])
def test_projected_matrices_of_their_shape_are_taken(form):
    G = torch.diag(torch.arange(1.0, 6.0, dtype=torch.float64, device="cuda"))
    as_form = {"plain": lambda M: M, "one of a batch": lambda M: M[None], "transposed view": lambda M: M.T,
               "float32": lambda M: M.float()}[form]
    z, lam, _, st = B.projected_solve(as_form(G), as_form(G), torch.ones(5, dtype=torch.float64, device="cuda"), 5.0, 0.0,
                                      fixed_lambda=1.0)
    assert st == 0 and lam == 1.0
    assert torch.allclose(z, 0.5 / G.diagonal(), rtol=1e-14, atol=0.0)
