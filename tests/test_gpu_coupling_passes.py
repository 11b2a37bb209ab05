"""GPU parity of the coupling's launch forms against the FP64 oracle: with one
forcing cycle (the force totals in a kernel of their own), two (formed in the
last update pass), four (the default) and five (more cycles than accumulators,
the unfused sequence), the force on the markers or on the surface outside them
(beside the first update pass, or its own kernel), on population and moment
storage.  The sparse, tilted marker set has stencil boxes of every size, those
past the tile kernels' box limit among them."""
import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W
from tests.gpu_util import max_rel, oracle_to_soa, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2408_15115_amd import turret
    return turret


def tilted_sphere(cycles, offset, markers):
    n = 32
    case = W.make_case(n, n, 48, 0.75, W.BC_FREESLIP, W.BC_FREESLIP, 0, 3e-5, ibm_cycles=cycles)
    body = W.sphere_fibonacci_body(4.0, markers, 2.0, [(n - 1) / 2 + 0.3, (n - 1) / 2 - 0.2, 23.5],
                                   w0=np.array([1e-3, -2e-3, 3e-3]), force_offset=offset,
                                   d0=W.rotation_matrix([1.0, 2.0, 0.5], 0.4).T)
    return case, body


# the bounds of the coupled step's parity tests: FP32 populations 1e-5, force
# and torque 1e-4
@pytest.mark.parametrize("storage", ["f32", "mom"])
@pytest.mark.parametrize("cycles,offset,markers", [(1, 3.0, 300), (2, 3.0, 90), (4, 3.0, 90), (5, 3.0, 300),
                                                   (1, 0.0, 90), (5, 0.0, 90)])
def test_launch_forms_match_oracle(T, orc, storage, cycles, offset, markers):
    case, body = tilted_sphere(cycles, offset, markers)
    say(f"coupling passes: {storage}, {cycles} cycles, force surface {offset}, {markers} markers, 20 steps")
    o = orc.OracleSim(case, body)
    S = T.Solver([case], [body], storage=storage, ibm_cycles=cycles)
    D = T.Solver([case], [body], storage=storage, ibm_cycles=cycles, ibm_diag=1)
    o.step(20)
    S.run(20)
    D.run(20)
    st, ost, dg = S.body_state(), o.body_state(), D.body_state()
    Fs = np.linalg.norm(ost["F"])
    err = max_rel(S.populations(), oracle_to_soa(o.post_collision()))
    say(f"  populations {err:.3e}, force {np.max(np.abs(st['F'] - ost['F'])) / Fs:.3e}, "
        f"torque {np.max(np.abs(st['T'] - ost['T'])) / (Fs * 4.0):.3e}")
    assert err < 1e-5
    assert np.max(np.abs(st["F"] - ost["F"])) < 1e-4 * Fs
    assert np.max(np.abs(st["T"] - ost["T"])) < 1e-4 * max(np.linalg.norm(ost["T"]), Fs * 4.0)
    assert np.allclose(st["w"], ost["w"], rtol=1e-6, atol=1e-12)
    # reading every cycle's residual changes nothing else
    for k in ("F", "T", "r", "v", "w"):
        assert np.array_equal(st[k], dg[k]), k
    assert S.ibm_stats()["resid"] == D.ibm_stats()["resid"]
