"""How the lattice kernels round and store a step: the bfloat16 rounding of the
BF16 store against torch's on the FP32 result of the same step, code by code
(large and tiny values, both signs, a ragged box); and the D3Q19 kernel in a box
whose buffers pass the memory-side cache, where its stores take the other form,
against the FP64 oracle (1e-5 relative, the bar of the FP32 forms)."""
import numpy as np
import pytest

from paper_2408_15115_amd import workloads as W
from tests.gpu_util import max_rel, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2408_15115_amd import turret
    return turret


@pytest.mark.parametrize("amp", [0.05, 1e-6, 1e-30])
def test_bf16_codes_are_the_rounded_fp32_step(T, amp):
    import torch
    nx, ny, nz = 37, 21, 19
    case = W.make_case(nx, ny, nz, 0.6)
    scale = torch.tensor([2.0 ** (14 + 2 * sum(abs(k) for k in (i % 3 - 1, (i // 3) % 3 - 1, i // 9 - 1)))
                          for i in range(27)], device="cuda")[:, None]
    gen = torch.Generator(device="cuda").manual_seed(3)
    codes = (amp * 4096 * torch.randn((27, nx * ny * nz), device="cuda", generator=gen)).to(torch.bfloat16)
    out = {}
    for storage in ("bf16", "f32"):
        S = T.Solver([case], storage=storage)
        typ = torch.bfloat16 if storage == "bf16" else torch.float32
        view = lambda k: torch.as_strided(S.bufs[k].view(typ), (27, nx * ny * nz), (S.plane_stride(), 1))
        view(0).copy_(codes if storage == "bf16" else codes.float() / scale)
        S.lbm_step()
        torch.cuda.synchronize()
        out[storage] = view(1).clone()
        S.close()
    want = (out["f32"] * scale).to(torch.bfloat16)
    same = (out["bf16"].view(torch.int16) == want.view(torch.int16)).float().mean().item()
    say(f"  bf16 codes, amplitude {amp}: {same:.6f} equal the rounded FP32 step")
    # the two kernels may contract a product differently: an FP32 rounding
    # apart, which moves a code across its rounding boundary now and then, by
    # one unit of its 8 bits
    assert same > 0.999
    far = (out["bf16"].float() - want.float()).abs() > 2.0 ** -7 * want.float().abs()
    assert not far.any()


def test_d3q19_beyond_the_cache_matches_oracle(T, orc):
    nx, ny, nz, tau = 121, 120, 122, 0.6
    C = orc.collide_grid19(W.random_populations19(5, nx, ny, nz), tau)
    S = T.Solver([W.make_case(nx, ny, nz, tau, W.BC_PERIODIC, W.BC_PERIODIC)], lattice=19)
    S.set_populations(np.ascontiguousarray(np.moveaxis(C, -1, 0)))
    S.lbm_step()
    gpu = S.populations()
    S.close()
    ref = np.moveaxis(orc.collide_grid19(orc.stream19(C), tau), -1, 0)
    assert max_rel(gpu, ref) < 1e-5


@pytest.mark.parametrize("lattice,nx,ny,nz", [(27, 62, 61, 60), (19, 72, 66, 65)])
def test_boxes_that_the_cache_holds_match_oracle(T, orc, lattice, nx, ny, nz):
    """FP32 buffers past the L2s that the memory-side cache still holds: their
    stores are ordinary ones."""
    tau = 0.7
    rnd, collide, stream = ((W.random_populations, orc.collide_grid, orc.stream_grid) if lattice == 27 else
                            (W.random_populations19, orc.collide_grid19, orc.stream19))
    C = collide(rnd(9, nx, ny, nz), tau)
    S = T.Solver([W.make_case(nx, ny, nz, tau, W.BC_PERIODIC, W.BC_PERIODIC)], lattice=lattice)
    S.set_populations(np.ascontiguousarray(np.moveaxis(C, -1, 0)))
    S.lbm_step()
    gpu = S.populations()
    S.close()
    ref = np.moveaxis(collide(stream(C), tau), -1, 0)
    assert max_rel(gpu, ref) < 1e-5


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("schedule", [3, 4])
def test_queue_takes_every_tile_once(T, storage, schedule):
    """The work queue with fewer workgroups than counters, a few, and more than
    tiles, in chunks of 1 to 4 tiles (the largest box has 1,425), on uneven
    boxes: the fields of the plain schedule, bit for bit, over several steps."""
    dims = [(48, 76, 100), (9, 8, 11), (33, 21, 40)]
    cases = [W.make_case(*d, 0.6, W.BC_NOSLIP, W.BC_FREESLIP, 4) for d in dims]
    rng = np.random.default_rng(7)
    start = [W.D3Q27_W[:, None, None, None] * (1 + 0.02 * rng.standard_normal((27, *d[::-1]))) for d in dims]
    out = []
    for kw in [dict()] + [dict(schedule=schedule, persist_wgs=n) for n in (1, 5, 8, 61, 120, 700, 4000)]:
        S = T.Solver(cases, None, storage=storage, **kw)
        for c in range(3):
            S.set_populations(start[c], c)
        S.run(3)
        out.append([S.populations(c) for c in range(3)])
        S.close()
        for c in range(3):
            assert np.array_equal(out[-1][c], out[0][c]), (kw, c)
