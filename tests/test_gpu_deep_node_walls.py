"""Deep passes of small domains with on-node walls, whose plan cuts a wall axis into tiles of
few nodes, against the one-cycle pass, bit for bit: calls of one, two, three and many steps.
Equal inputs and the same per-node arithmetic, so the tolerance is zero."""
import pytest
import torch

from paper_1311_7239_amd import inputs as I
from paper_1311_7239_amd import lbm
from tests.test_gpu_deep import _cavity, _heat, _one_cycle

pytestmark = pytest.mark.gpu

CASES = {
    "cavity_23x23": lambda: _cavity(23, 23, nee=True),
    "cavity_24x24_grf": lambda: _cavity(24, 24, grf=True, nee=True),
    "cavity_31x31": lambda: _cavity(31, 31, nee=True),
    "cavity_27x29": lambda: _cavity(27, 29, nee=True),
    "cavity_3x200": lambda: _cavity(3, 200, nee=True),
    "cavity_511x4": lambda: _cavity(511, 4, nee=True),
    "channel_8x80": lambda: I.poiseuille_channel(nx=8, ny=80, nee=True),
    "channel_8x96": lambda: I.poiseuille_channel(nx=8, ny=96, nee=True),
    "channel_16x33": lambda: I.poiseuille_channel(nx=16, ny=33, nee=True),
    "heat_24x24": lambda: _heat(24, 24, nee=True),
    "heat_16x33": lambda: _heat(16, 33, nee=True),
}


@pytest.mark.parametrize("storage", [lbm.FP32_DEV, lbm.FP16_DEV])
@pytest.mark.parametrize("name", list(CASES))
def test_deep_pass_is_bitwise_the_one_cycle_pass(name, storage):
    case = CASES[name]()
    df = torch.from_numpy(I.random_deviation_state(case.ny, case.nx, 1e-3, seed=5)).cuda()
    dg = (torch.from_numpy(I.random_deviation_state(case.ny, case.nx, 1e-1, seed=6, channels=5)).cuda()
          if case.thermal else None)
    a, b = (lbm.solver_for_case(case, storage=storage) for _ in range(2))
    _one_cycle(a, case)
    for s in (a, b):
        s.set_populations(df, dg)
    for chunk in (1, 1, 2, 3, 11, 1, 40):
        a.step(chunk)
        b.step(chunk)
        fa, ga = a.populations(thermal=case.thermal)
        fb, gb = b.populations(thermal=case.thermal)
        torch.cuda.synchronize()
        assert torch.equal(fa, fb), (chunk, a.time)
        assert ga is None or torch.equal(ga, gb), (chunk, a.time)
        assert a.reduce() == b.reduce(), (chunk, a.time)
