"""The moment-storage step in tiles of 11 rows and 64 columns, whose side columns
come from the side wave, against the FP64 oracle: with z walls and a sponge, and
coupled, with the forcing box across a tile's side and in the rows of another.
(Boxes large enough for the planner to take 11 rows; FP32 state against FP64:
populations within 1e-5 relative, force within 1e-4, as for every FP32 form.)"""
import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W
from tests.gpu_util import max_rel, oracle_to_soa, say

pytestmark = pytest.mark.gpu

PAPER, PLATES = (W.BC_NOSLIP, W.BC_PRESSURE), (W.BC_NOSLIP,) * 2


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2408_15115_amd import turret
    return turret


@pytest.mark.parametrize("nx,ny,nz,bc,u_wall,sponge", [
    (127, 60, 150, PAPER, (0.0, 0.0), 13),
    (128, 62, 140, PLATES, (-0.03, 0.05), 0),
])
def test_walls_beside_the_side_wave(T, orc, nx, ny, nz, bc, u_wall, sponge):
    steps, tau = 3, 0.62
    say(f"moment tiles of 11 rows nx={nx} ny={ny} nz={nz} bc={bc} sponge={sponge}")
    case = W.make_case(nx, ny, nz, tau, bc[0], bc[1], sponge, u_wall=u_wall)
    C = orc.collide_grid(W.random_populations(nx + nz, nx, ny, nz, amp=0.03), tau, sponge)
    S = T.Solver([case], storage="mom")
    S.set_populations(oracle_to_soa(C))
    for _ in range(steps):
        S.lbm_step()
        C = orc.collide_grid(orc.stream_grid(C, bc[0], bc[1], u_wall), tau, sponge)
    gpu = S.populations()
    err = S.body_state(0, check=False)["err"]
    S.close()
    assert err == 0
    assert max_rel(gpu, oracle_to_soa(C)) < 1e-5


@pytest.mark.parametrize("x,y", [(63.6, 30.2), (126.4, 59.3)])   # two tiles' common side; the periodic edges
@pytest.mark.parametrize("forcing", [0, 1])
def test_body_beside_the_side_wave(T, orc, x, y, forcing):
    nx, ny, nz = 127, 60, 150
    case = W.make_case(nx, ny, nz, 0.7, PAPER[0], PAPER[1], 13, 2e-5)
    body = W.sphere_fibonacci_body(4.0, 300, 2.0, [x, y, 70.3], force_offset=0.0)
    say(f"moment tiles of 11 rows with a body at x={x} y={y}, forcing {forcing}")
    o = orc.OracleSim(dict(case, forcing=forcing), body)
    S = T.Solver([case], [body], storage="mom", forcing=forcing)
    o.step(6)
    S.run(6)
    gpu, st = S.populations(), S.body_state()
    S.close()
    ref, ost = oracle_to_soa(o.post_collision()), o.body_state()
    assert max_rel(gpu, ref) < 1e-5
    assert np.max(np.abs(st["F"] - ost["F"])) < 1e-4 * np.linalg.norm(ost["F"])
