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


def test_step_log_is_read(leave_an_error):
    import torch
    from paper_2408_15115_amd import turret as T
    case = W.make_case(24, 24, 40, 0.7, W.BC_FREESLIP, W.BC_FREESLIP, 4, 2e-5)
    S = T.Solver([case], [W.sphere_fibonacci_body(3.0, 150, 2.0, [11.5, 11.5, 20.0])])
    S.run(40)
    torch.cuda.synchronize()
    assert leave_an_error() != 0
    first, lost = S.log_read(0, 3)
    assert first[:, 28].tolist() == [1, 2, 3] and lost == 0
    rest, _ = S.log_read(0)
    assert rest[:, 28].tolist() == list(range(4, 41))
    S.close()


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
