"""Calls made while an error of an earlier, unrelated runtime call is pending
(here: the choice of a device that does not exist)."""
import ctypes as C

import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture
def leave_an_error():
    import torch
    torch.zeros(1, device="cuda")
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = C.CDLL(path)
    yield lambda: hip.hipSetDevice(1 << 20)
    hip.hipGetLastError()


def test_training_step_that_fails_leaves_the_parameters(leave_an_error):
    import torch
    from paper_2408_15115_amd import turret as T
    gen = torch.Generator(device="cuda").manual_seed(4)
    X = torch.randn((100, T.MLP_IN), device="cuda", generator=gen)
    Y = torch.randn((100, 3), device="cuda", generator=gen)
    net, ref = T.MLP(max_batch=100, seed=2), T.MLP(max_batch=100, seed=2)
    torch.cuda.synchronize()
    assert leave_an_error() != 0
    with pytest.raises(T.TurretError):
        net.train_step(X, Y)
    assert np.array_equal(net.params(), ref.params())
    for _ in range(2):   # and the step count
        net.train_step(X, Y)
        ref.train_step(X, Y)
    assert np.array_equal(net.params(), ref.params())
