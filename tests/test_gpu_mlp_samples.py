"""Samples that start at any float: gradient and training step on rows that are
not 16-byte aligned give the bits of the aligned ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_unaligned_samples(shift):
    import torch
    from paper_2408_15115_amd import turret as T
    n = 130
    gen = torch.Generator(device="cuda").manual_seed(4)
    X = torch.randn((n, T.MLP_IN), device="cuda", generator=gen)
    Y = torch.randn((n, 3), device="cuda", generator=gen)
    Xs = torch.empty(shift + X.numel(), device="cuda")[shift:].view(n, T.MLP_IN).copy_(X)
    assert Xs.data_ptr() % 16 != 0
    nets = [T.MLP(max_batch=n, seed=2) for _ in range(2)]
    g = [net.grad(x, Y) for net, x in zip(nets, (X, Xs))]
    assert torch.equal(g[0][0], g[1][0]) and torch.equal(g[0][1], g[1][1])
    for net, x in zip(nets, (X, Xs)):
        net.train_step(x, Y)
    assert np.array_equal(nets[0].params(), nets[1].params())
