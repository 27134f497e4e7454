"""Recomputation for the adjoint in rolling passes (the default on mid-size domains) against
tile passes: the gradients and the parameter gradients, whose reverse passes are the same
in both, bit for bit. Segments of every remainder, every medium, with and without the D2Q5
field. Equal inputs and the same per-node arithmetic, so the tolerance is zero."""
import pytest
import torch

from paper_1311_7239_amd import inputs as I
from paper_1311_7239_amd import lbm
from tests.test_gpu_roll import _case, _solver

pytestmark = pytest.mark.gpu

P, W = I.PERIODIC, I.WALLS


@pytest.mark.parametrize("bc_x,bc_y,nx,ny,medium,heat,every,steps", [
    (P, W, 701, 700, "ergun", False, 13, 29),
    (W, P, 129, 4001, "ergun", False, 6, 19),
    (W, W, 901, 555, "kappa", False, 11, 30),
    (P, P, 650, 651, "uniform", False, 14, 24),
    (W, W, 600, 500, "ergun", True, 9, 20),
    (W, P, 640, 513, "kappa", True, 7, 17),
    (W, W, 600, 450, "uniform", True, 10, 18),
])
def test_recording_in_rolling_passes_is_bitwise_that_in_tiles(bc_x, bc_y, nx, ny, medium, heat, every, steps):
    case = _case(bc_x, bc_y, nx, ny, medium, heat)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    df = 2e-3 * (torch.rand((8, ny, nx), generator=g, device="cuda") - 0.5)
    dg = 0.2 * (torch.rand((5, ny, nx), generator=g, device="cuda") - 0.5) if heat else None
    w = torch.randn((2, ny, nx), generator=g, device="cuda")
    out = []
    for tiles in (False, True):
        s = _solver(case, medium, ckpt_every=every, max_steps_recorded=steps)
        if tiles:
            s.set_time_blocking(2)   # the default's reverse passes
        s.set_populations(df, dg)
        s.step(steps)
        if medium == "uniform":
            out.append(s.backward_params(w, want_phi=False))
        else:
            out.append(s.backward_params(w) + s.backward(w))
        torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y
