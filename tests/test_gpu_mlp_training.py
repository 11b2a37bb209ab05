"""The training pass of the warm-start network at the edges of its work split
(64 samples per workgroup and round, at most 256 workgroups): one sample, one
below, at and above a round, one above a full chip, against the FP64 reference
gradient; the fused Adam step against the reference update over several steps;
saturated activations; and bitwise reproducibility.  FP32 sums of n terms with
FP16-exact weights: gradient and loss within 1e-5 of the largest entry, the
bar of the other gradient tests."""
import numpy as np
import pytest

from oracle import mlp as ref
from tests.gpu_util import say

pytestmark = pytest.mark.gpu
NIN = ref.LAYERS[0][0]


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2408_15115_amd import turret
    return turret


def dev(a):
    import torch
    return torch.tensor(np.ascontiguousarray(a, np.float32), device="cuda")


def problem(n, seed, scale=1.0):
    rng = np.random.default_rng(seed)
    theta = np.asarray(scale * (ref.init_params(seed) + 0.05 * rng.standard_normal(ref.N_PARAMS)), np.float16)
    return (theta.astype(np.float32), rng.standard_normal((n, NIN)).astype(np.float32),
            rng.standard_normal((n, 3)).astype(np.float32))


@pytest.mark.parametrize("n,scale", [(1, 1.0), (63, 1.0), (64, 1.0), (65, 1.0), (200, 8.0), (16385, 1.0), (20000, 1.0)])
def test_gradient_at_the_edges_of_the_split(T, n, scale):
    theta, X, Y = problem(n, 7 + n, scale)
    net = T.MLP(max_batch=n, params=theta)
    g, loss = net.grad(dev(X), dev(Y))
    th, X64, Y64 = theta.astype(np.float64), X.astype(np.float64), Y.astype(np.float64)
    gr, lr_ = ref.grad(th, X64, Y64), ref.loss(th, X64, Y64)
    err = np.max(np.abs(g.cpu().numpy() - gr)) / np.max(np.abs(gr))
    say(f"  n={n} scale={scale}: gradient error {err:.2e}, loss {loss.item():.4e} (reference {lr_:.4e})")
    assert err < 1e-5 and abs(loss.item() - lr_) < 1e-5 * lr_
    g2, loss2 = net.grad(dev(X), dev(Y))
    assert np.array_equal(g.cpu().numpy(), g2.cpu().numpy()) and loss.item() == loss2.item()


def test_adam_steps_follow_the_gradient(T):
    """Each step is the reference update of the gradient that the same
    parameters give (compared one step at a time: the FP16 copy feeds back)."""
    import torch
    theta, X, Y = problem(300, 5)
    net, probe = T.MLP(max_batch=300, params=theta), T.MLP(max_batch=300, params=theta)
    m, v, cur = np.zeros(ref.N_PARAMS), np.zeros(ref.N_PARAMS), theta.astype(np.float64)
    loss = torch.zeros(1, device="cuda")
    for step in range(1, 4):
        probe.set_params(net.params())
        g, l0 = probe.grad(dev(X), dev(Y))
        net.train_step(dev(X), dev(Y), lr=2e-3, loss=loss)
        cur, m, v = ref.adam(cur, m, v, g.cpu().numpy().astype(np.float64), step, lr=2e-3)
        assert loss.item() == l0.item()
        assert np.max(np.abs(net.params() - cur)) < 1e-6 * step
