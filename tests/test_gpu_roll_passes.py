"""The rolling pass bit for bit against the one-cycle pass at sizes that roll, which each case
asserts: binary16 storage with a 1/K plane, and per-node viscosity ratios with each medium, with
and without the D2Q5 field, alone, recorded and in batches. Equal inputs and the same per-node
arithmetic, so the tolerance is zero."""
import numpy as np
import pytest
import torch

from paper_1311_7239_amd import inputs as I
from paper_1311_7239_amd import lbm
from tests.test_gpu_batch_roll import _batch
from tests.test_gpu_roll import _case, _solver

pytestmark = pytest.mark.gpu

P, W = I.PERIODIC, I.WALLS


def _with_J(case, J):
    if J:
        x, y = np.arange(case.nx), np.arange(case.ny)
        case.Jfield = (2.5 + np.outer(np.sin(0.07 * y), np.cos(0.05 * x))).astype(np.float32)
    return case


def _made(case, medium, storage=lbm.FP32_DEV, **kw):
    s = _solver(case, medium, storage, **kw)
    if getattr(case, "Jfield", None) is not None:
        s.set_viscosity_ratio(torch.from_numpy(case.Jfield).cuda())
    return s


CASES = [
    (W, P, 1201, 351, "kappa", False, False, lbm.FP16_DEV),
    (P, W, 777, 533, "kappa", False, True, lbm.FP32_DEV),
    (W, W, 701, 650, "uniform", False, True, lbm.FP32_DEV),
    (P, P, 901, 601, "ergun", False, True, lbm.FP32_DEV),
    (W, P, 901, 601, "ergun", False, True, lbm.FP16_DEV),
    (W, W, 600, 450, "uniform", True, True, lbm.FP32_DEV),
    (W, P, 513, 640, "kappa", True, True, lbm.FP32_DEV),
    (P, W, 2501, 2111, "kappa", False, True, lbm.FP32_DEV),   # threes and fours in tiles
]


@pytest.mark.parametrize("bc_x,bc_y,nx,ny,medium,heat,J,storage", CASES)
def test_rolling_pass_is_bitwise_the_one_cycle_pass(bc_x, bc_y, nx, ny, medium, heat, J, storage):
    case = _with_J(_case(bc_x, bc_y, nx, ny, medium, heat), J)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    df = 2e-3 * (torch.rand((8, ny, nx), generator=g, device="cuda") - 0.5)
    dg = 0.2 * (torch.rand((5, ny, nx), generator=g, device="cuda") - 0.5) if heat else None
    a, b = (_made(case, medium, storage) for _ in range(2))
    a.set_time_blocking(1)
    for s in (a, b):
        s.set_populations(df, dg)
    for chunk in (7, 4, 6, 13, 3):
        if b.time > 0:
            assert b.next_pass(6) == ("rolling", 3 if heat else 6)
        a.step(chunk)
        b.step(chunk)
        fa, ga = a.populations(heat)
        fb, gb = b.populations(heat)
        torch.cuda.synchronize()
        assert torch.equal(fa, fb), (chunk, a.time)
        assert not heat or torch.equal(ga, gb), (chunk, a.time)
        assert a.reduce() == b.reduce(), (chunk, a.time)


@pytest.mark.parametrize("bc_x,bc_y,nx,ny,medium,heat,every,steps", [
    (P, W, 777, 533, "kappa", False, 13, 29),
    (W, W, 701, 650, "ergun", False, 11, 24),
    (W, W, 600, 500, "uniform", True, 10, 21),
])
def test_recording_in_rolling_passes_with_viscosity_ratios(bc_x, bc_y, nx, ny, medium, heat, every, steps):
    case = _with_J(_case(bc_x, bc_y, nx, ny, medium, heat), True)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    df = 2e-3 * (torch.rand((8, ny, nx), generator=g, device="cuda") - 0.5)
    dg = 0.2 * (torch.rand((5, ny, nx), generator=g, device="cuda") - 0.5) if heat else None
    w = torch.randn((2, ny, nx), generator=g, device="cuda")
    out = []
    for tiles in (False, True):
        s = _made(case, medium, ckpt_every=every, max_steps_recorded=steps)
        if tiles:
            s.set_time_blocking(2)   # the default's reverse passes
        s.set_populations(df, dg)
        s.step(1)
        assert tiles or s.next_pass(6)[0] == "rolling"
        s.step(steps - 1)
        out.append(s.backward_params(w, want_phi=medium != "uniform"))
        torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y


@pytest.mark.parametrize("heat", [False, True])
def test_batched_rolling_pass_with_viscosity_ratios(heat):
    shapes = [(W, W, 16, 16), (W, W, 65, 140), (P, W, 64, 16), (P, P, 67, 129), (P, W, 301, 90)]
    kinds = ["kappa", "uniform", "ergun", "kappa", "uniform"]
    cases = [_with_J(_case(bx, by, nx, ny, m, heat), k != 2) for k, ((bx, by, nx, ny), m) in enumerate(zip(shapes, kinds))]
    b = _batch(cases, kinds, lbm.FP32_DEV)
    singles = []
    for k, (case, medium) in enumerate(zip(cases, kinds)):
        g = torch.Generator(device="cuda")
        g.manual_seed(k)
        df = 2e-3 * (torch.rand((8, case.ny, case.nx), generator=g, device="cuda") - 0.5)
        dg = 0.2 * (torch.rand((5, case.ny, case.nx), generator=g, device="cuda") - 0.5) if heat else None
        if getattr(case, "Jfield", None) is not None:
            b.set_viscosity_ratio(k, torch.from_numpy(case.Jfield).cuda())
        s = _made(case, medium)
        s.set_time_blocking(1)
        s.set_populations(df, dg)
        b.set_populations(k, df, dg)
        singles.append(s)
    for chunk in (7, 4, 6, 11, 3):
        b.step(chunk)
        assert b.next_pass(6) == ("rolling", 3 if heat else 6)
        for k, s in enumerate(singles):
            s.step(chunk)
            fb, fs = b.populations(k, thermal=heat), s.populations(thermal=heat)
            torch.cuda.synchronize()
            for x, y in zip(fb if heat else (fb,), fs if heat else fs[:1]):
                assert torch.equal(x, y), (k, shapes[k], chunk, s.time)
            assert b.reduce(k) == s.reduce(), (k, shapes[k], chunk)
