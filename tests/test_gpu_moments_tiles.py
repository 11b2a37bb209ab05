"""The moment-storage step at the edges of its column tiles, against the FP64
oracle: boxes one column below, at and above the widths where the tiles change
(62 columns with the side columns in the lanes, 64 with the side wave, 65 in
two tiles), both row capacities, several z chunks with a ragged last one, all
kinds of walls; and a body across the periodic x and y edges, whose forcing
box wraps.  FP32 state against FP64: populations within 1e-5 relative, force
within 1e-4, as for every FP32 form."""
import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W
from tests.gpu_util import max_rel, oracle_to_soa, say

pytestmark = pytest.mark.gpu

SLIP, PAPER = (W.BC_FREESLIP,) * 2, (W.BC_NOSLIP, W.BC_PRESSURE)
PERIODIC, PLATES = (W.BC_PERIODIC,) * 2, (W.BC_NOSLIP,) * 2


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2408_15115_amd import turret
    return turret


@pytest.mark.parametrize("nx,ny,nz,bc,u_wall,sponge", [
    (62, 12, 13, PERIODIC, (0.0, 0.0), 0),
    (63, 11, 20, PAPER, (0.0, 0.0), 5),
    (64, 23, 24, SLIP, (0.0, 0.0), 0),
    (65, 40, 33, PLATES, (-0.03, 0.05), 0),
    (130, 45, 90, PAPER, (0.0, 0.0), 11),     # 11 rows a tile, widths of 44
    (127, 60, 150, PERIODIC, (0.0, 0.0), 0),   # 11 rows a tile, widths of 64
])
def test_tile_edges_match_oracle(T, orc, nx, ny, nz, bc, u_wall, sponge):
    steps, tau = 3, 0.62
    say(f"moment tiles nx={nx} ny={ny} nz={nz} bc={bc} sponge={sponge}")
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


@pytest.mark.parametrize("nx,ny,forcing", [(66, 26, 0), (62, 31, 1), (64, 24, 0)])
def test_forcing_box_across_the_periodic_edges(T, orc, nx, ny, forcing):
    case = W.make_case(nx, ny, 40, 0.7, SLIP[0], SLIP[1], 0, 2e-5)
    body = W.sphere_fibonacci_body(3.0, 200, 2.0, [0.4, ny - 0.7, 19.5], force_offset=0.0)
    say(f"moment forcing box across the edges nx={nx} ny={ny} forcing={forcing}")
    o = orc.OracleSim(dict(case, forcing=forcing), body)
    S = T.Solver([case], [body], storage="mom", forcing=forcing)
    o.step(20)
    S.run(20)
    gpu, st = S.populations(), S.body_state()
    S.close()
    ref, ost = oracle_to_soa(o.post_collision()), o.body_state()
    assert max_rel(gpu, ref) < 1e-5
    assert np.max(np.abs(st["F"] - ost["F"])) < 1e-4 * np.linalg.norm(ost["F"])
