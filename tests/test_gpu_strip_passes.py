"""The strip pass bit for bit against the one-cycle pass at sizes that step in strips, which each
case asserts (the passes of a size follow from rules that may move): both storages, odd
periodic widths and half pairs at walls in both, uniform and Ergun media, strips of four
cycles, and a recorded run. Equal inputs and the same per-node arithmetic, so the tolerance is
zero."""
import pytest
import torch

from paper_1311_7239_amd import inputs as I
from paper_1311_7239_amd import lbm
from tests.test_gpu_strip import _case

pytestmark = pytest.mark.gpu

P, W = I.PERIODIC, I.WALLS
CASES = [
    # (bc_x, bc_y, nx, ny, ergun, storage, four: strips of four cycles too)
    (P, W, 4099, 2401, True, lbm.FP16_DEV, True),     # odd pairs in binary16, one across the seam
    (P, P, 4097, 2500, True, lbm.FP16_DEV, True),
    (W, P, 4097, 2400, True, lbm.FP16_DEV, True),     # ends in half a pair
    (W, W, 4100, 2401, True, lbm.FP16_DEV, True),
    (P, W, 4103, 4101, False, lbm.FP16_DEV, False),
    (W, W, 4101, 4103, False, lbm.FP16_DEV, False),
    (P, W, 2731, 2049, True, lbm.FP32_DEV, True),
    (W, P, 16385, 351, True, lbm.FP32_DEV, True),
    (P, P, 1161, 5003, True, lbm.FP32_DEV, True),     # its last strip is a column wide before it takes its ring
    (P, W, 2901, 2307, True, lbm.FP32_DEV, False),
    (W, W, 2931, 2901, False, lbm.FP32_DEV, False),
    (P, W, 2933, 2903, False, lbm.FP32_DEV, False),
]


@pytest.mark.parametrize("bc_x,bc_y,nx,ny,ergun,storage,four", CASES)
def test_strip_pass_is_bitwise_the_one_cycle_pass(bc_x, bc_y, nx, ny, ergun, storage, four):
    case = _case(bc_x, bc_y, nx, ny, ergun)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    df = 2e-3 * (torch.rand((8, ny, nx), generator=g, device="cuda") - 0.5)
    a, b = (lbm.solver_for_case(case, storage=storage) for _ in range(2))
    a.set_time_blocking(1)
    for s in (a, b):
        s.set_populations(df)
    del df
    for chunk in (7, 4, 6, 13):
        if b.time > 0:
            assert b.next_pass(6) == ("strips", 6) and b.next_pass(4) == ("strips" if four else "tiles", 4)
        a.step(chunk)
        b.step(chunk)
        fa, fb = a.populations()[0], b.populations()[0]
        torch.cuda.synchronize()
        assert torch.equal(fa, fb), (chunk, a.time)
        del fa, fb
        assert a.reduce() == b.reduce(), (chunk, a.time)


def test_a_recorded_run_in_strips():
    """The gradient recomputes from the checkpoints, so equal gradients need equal checkpoints."""
    case = _case(P, W, 2731, 2049, True)
    out = []
    for cycles in (1, 0):
        s = lbm.solver_for_case(case, ckpt_every=9, max_steps_recorded=24)
        if cycles:
            s.set_time_blocking(cycles)
        s.step(1)
        assert s.next_pass(20) == (("tiles", 1) if cycles else ("strips", 4))   # to the checkpoint at 9: four and four
        s.step(8)
        assert s.next_pass(20) == (("tiles", 1) if cycles else ("strips", 6))
        s.step(15)
        _, u, _ = s.macroscopic()
        g, _ = s.backward(u)
        torch.cuda.synchronize()
        out.append((u, g))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
