"""The window's rows in a box far wider than the body's region: a library-
sequenced step with a shift, whose correction resets the rows with more
workgroups than the region has, against the separate window_shift, bit for bit."""
import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W
from tests.gpu_util import oracle_to_soa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,rows", [(97, 83, 16), (40, 33, 1)])
@pytest.mark.parametrize("storage", ["f32", "f16", "mom"])
def test_rows_of_a_wide_box(storage, nx, ny, rows):
    import torch
    from paper_2408_15115_amd import turret as T
    nz, h_end = 64, 30.0
    case = W.make_case(nx, ny, nz, 0.7, W.BC_FREESLIP, W.BC_FREESLIP, 0, 1e-5, h_ini=h_end + rows, h_end=h_end)
    body = W.sphere_fibonacci_body(3.0, 150, 2.0, [nx / 2, ny / 2, h_end + 0.055], force_offset=0.0)
    body["v0"] = np.array([0.0, 0.0, -0.02])
    f = oracle_to_soa(W.random_populations(5, nx, ny, nz))
    A, B = (T.Solver([case], [body], storage=storage, stream=torch.cuda.Stream()) for _ in range(2))
    for S in (A, B):
        S.set_populations(f)
    A.run(6)
    for _ in range(6):
        B.body_advance()
        B.lbm_step()
        B.ibm_couple()
        B.window_shift()
    a, b = A.body_state(), B.body_state()
    assert a["shifts"] >= 1
    assert all(np.array_equal(a[k], b[k]) for k in a)
    assert np.array_equal(A.populations(), B.populations())
    A.close()
    B.close()
