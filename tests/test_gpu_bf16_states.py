"""BF16 states bit for bit: checksums of the codes that the solver held after
some steps when its BF16 store rounded in integer arithmetic.  A code that is
off by one stays visible for many steps, so a change of a rounding anywhere in
the step (a product contracted into an FMA, say) shows here; the inputs come
from numpy's PCG64 streams."""
import zlib

import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W
from tests.gpu_util import oracle_to_soa, say

pytestmark = pytest.mark.gpu

PAPER, SLIP = (W.BC_NOSLIP, W.BC_PRESSURE), (W.BC_FREESLIP,) * 2
CRC = {"fluid": 0xc6afa9ff, "bgk": 0xdea1f9bb, "queue": 0xc6afa9ff, "coupled": 0x93fc9f36, "coupled_store": 0x1621a7bb}


@pytest.mark.parametrize("name", list(CRC))
def test_states_are_those_of_the_integer_rounding(name):
    import torch
    from paper_2408_15115_amd import turret as T
    nx, ny, nz = 37, 29, 34
    bc = PAPER if name in ("fluid", "bgk", "queue") else SLIP
    case = W.make_case(nx, ny, nz, 0.62, bc[0], bc[1], 0 if name == "bgk" else 5, 2e-5)
    bodies, opts = None, {"bgk": {"collision": 1}, "queue": {"schedule": 4}, "coupled_store": {"fine_box": 0}}.get(name, {})
    if name.startswith("coupled"):
        bodies = [W.sphere_fibonacci_body(4.0, 260, 2.0, [18.3, 14.6, 17.2], force_offset=0.0)]
    S = T.Solver([case], bodies, storage="bf16", **opts)
    S.set_populations(oracle_to_soa(W.random_populations(11, nx, ny, nz)))
    for _ in range(12):
        S.run(1) if bodies else S.lbm_step()
    torch.cuda.synchronize()
    raw = next(b for b in S.bufs[:2] if b.data_ptr() == S.current_buffer()).view(torch.int16)
    codes = torch.as_strided(raw, (27, nz * ny * nx), (S.plane_stride(), 1), S.pop_offset()).cpu().numpy()
    assert S.body_state(0, check=False)["err"] == 0
    S.close()
    got = zlib.crc32(np.ascontiguousarray(codes).tobytes())
    say(f"  bf16 {name}: checksum {got:#010x}")
    assert got == CRC[name]
