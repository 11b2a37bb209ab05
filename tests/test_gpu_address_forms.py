"""The two forms of a cell's place in its plane (scalar base and 32-bit offset, or
64-bit offsets) give the same bits: FP32 boxes on both sides of the sizes where
the plain schedule changes form (28 and 40 MB of buffers; with a body
256 MB and 1.75 GiB), against the persistent
schedule, which always takes the 64-bit one; and the D3Q19 kernel in a box of
2^30 cells, whose planes pass 4 GiB, against a box that it repeats along z."""
import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W
from tests.gpu_util import oracle_to_soa, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2408_15115_amd import turret
    return turret


@pytest.mark.parametrize("nx,ny,nz", [(50, 50, 50), (55, 54, 53), (75, 92, 27), (60, 60, 59)])
@pytest.mark.parametrize("bc", [(W.BC_FREESLIP,) * 2, (W.BC_NOSLIP, W.BC_PRESSURE)])
def test_forms_agree(T, nx, ny, nz, bc):
    case = W.make_case(nx, ny, nz, 0.6, bc[0], bc[1], 5)
    f = oracle_to_soa(W.random_populations(nx, nx, ny, nz))
    out = []
    for opts in ({}, {"schedule": 1}, {"schedule": 2, "persist_wgs": 64}):
        S = T.Solver([case], **opts)
        S.set_populations(f)
        for _ in range(3):
            S.lbm_step()
        out.append(S.populations())
        assert S.body_state(0, check=False)["err"] == 0
        S.close()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])


@pytest.mark.parametrize("n,warm", [(110, 0), (215, 0), (215, 1)])
def test_forms_agree_beside_a_body(T, n, warm):
    # 110: past the memory-side cache, the 64-bit form for the body's sake; 215
    # (past 1.75 GiB): for a warm start alone
    import torch
    case = W.make_case(n, n + 1, n, 0.7, W.BC_FREESLIP, W.BC_FREESLIP, 8, 2e-5)
    body = W.sphere_fibonacci_body(5.0, 400, 2.0, [n / 2 - 0.7, n / 2 + 0.1, n / 2 - 0.2])
    runs = []
    for opts in ({}, {"schedule": 4}):
        S = T.Solver([case], [body], **opts)
        S.set_warm_start(warm, None, 2)
        S.run(6)
        runs.append((S, S.body_state(), next(b for b in S.bufs[:2] if b.data_ptr() == S.current_buffer()).view(torch.int32)))
    (A, a, fa), (B, b, fb) = runs
    assert all(np.array_equal(a[k], b[k]) for k in a)
    assert a["err"] == 0 and torch.equal(fa, fb)
    A.close()
    B.close()


@pytest.mark.parametrize("collision", [0, 1])
def test_d3q19_planes_past_4_gib(T, collision):
    import torch
    torch.cuda.empty_cache()
    nx, ny, nz, period = 1024, 1024, 1024, 16
    need = 2 * 19 * 4 * nx * ny * (nz + 4 * period)
    if torch.cuda.mem_get_info()[0] < need + (8 << 30):
        pytest.skip(f"needs {need >> 30} GiB of device memory")
    say(f"D3Q19 {nx}x{ny}x{nz} against its period of {period}, collision {collision}")

    def planes(S, z):
        raw = next(b for b in S.bufs[:2] if b.data_ptr() == S.current_buffer()).view(torch.float32)
        return torch.as_strided(raw, (19, z, ny * nx), (S.plane_stride(), ny * nx, 1), S.pop_offset())

    make = lambda z: W.make_case(nx, ny, z, 0.6, W.BC_PERIODIC, W.BC_PERIODIC)  # noqa: E731
    small = T.Solver([make(period)], lattice=19, collision=collision)
    large = T.Solver([make(nz)], lattice=19, collision=collision)
    gen = torch.Generator(device="cuda").manual_seed(9)
    a, b = planes(small, period), planes(large, nz)
    for i in range(19):
        a[i].copy_(1e-3 * torch.rand(a[i].shape, device="cuda", generator=gen))
        for z in range(0, nz, period):
            b[i, z:z + period].copy_(a[i])
    for _ in range(3):
        small.lbm_step()
        large.lbm_step()
    torch.cuda.synchronize()
    a, b = planes(small, period), planes(large, nz)
    assert small.body_state(0, check=False)["err"] == 0 and large.body_state(0, check=False)["err"] == 0
    for i in range(19):
        assert all(torch.equal(b[i, z:z + period], a[i]) for z in range(0, nz, period)), i
    small.close()
    large.close()
    del small, large, a, b
    torch.cuda.empty_cache()
