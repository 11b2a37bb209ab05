"""Moving no-slip walls give the same bits in every form of the step: every
schedule of the lattice kernel, and a case alone or among others in a batch
(where moment storage cuts it into other tiles), with and without a body near a
wall."""
import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W
from tests.gpu_util import oracle_to_soa

pytestmark = pytest.mark.gpu

U_WALL = (-0.03, 0.05)


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2408_15115_amd import turret
    return turret


def plates(nx, ny, nz):
    return W.make_case(nx, ny, nz, 0.62, W.BC_NOSLIP, W.BC_NOSLIP, 0, 2e-5, u_wall=U_WALL)


def sphere(nx, ny):
    # its stencils reach the bottom row
    return W.sphere_fibonacci_body(4.0, 260, 2.0, [nx / 2 - 0.3, ny / 2 + 0.2, 7.3], force_offset=0.0)


def step(S, f, steps, bodies):
    for b, x in enumerate(f):
        S.set_populations(x, b)
    if bodies:
        S.run(steps)
    else:
        for _ in range(steps):
            S.lbm_step()
    out = [S.populations(b) for b in range(S.n)]
    st = [S.body_state(b, check=False) for b in range(S.n)]
    S.close()
    assert all(s["err"] == 0 for s in st)
    return out, st


@pytest.mark.parametrize("with_body", [False, True])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_schedules_agree(T, storage, with_body):
    nx, ny, nz = 37, 29, 26
    f = [oracle_to_soa(W.random_populations(3, nx, ny, nz))]
    bodies = [sphere(nx, ny)] if with_body else None
    ref = None
    for opts in ({}, {"block": 64}, {"schedule": 1}, {"schedule": 2, "persist_wgs": 16}, {"schedule": 3}, {"schedule": 4}):
        (pop,), (st,) = step(T.Solver([plates(nx, ny, nz)], bodies, storage=storage, **opts), f, 8, bodies)
        if ref is None:
            ref = pop, st
        assert np.array_equal(pop, ref[0]), opts
        assert np.array_equal(st["F"], ref[1]["F"]) and np.array_equal(st["r"], ref[1]["r"]), opts


@pytest.mark.parametrize("with_body", [False, True])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16", "mom"])
def test_batch_equals_alone(T, storage, with_body):
    # the second box makes moment storage take tiles of 11 rows for both
    dims = [(37, 29, 26), (130, 45, 90)]
    cases = [plates(*d) for d in dims]
    f = [oracle_to_soa(W.random_populations(3 + b, *d)) for b, d in enumerate(dims)]
    bodies = [sphere(d[0], d[1]) for d in dims] if with_body else None
    both, st = step(T.Solver(cases, bodies, storage=storage), f, 6, bodies)
    (alone,), (st1,) = step(T.Solver(cases[:1], bodies[:1] if bodies else None, storage=storage), f[:1], 6, bodies)
    assert np.array_equal(both[0], alone)
    assert np.array_equal(st[0]["F"], st1["F"]) and np.array_equal(st[0]["r"], st1["r"])
