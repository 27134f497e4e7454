"""The rolling pass (six, four and three cycles per launch on mid-size domains, the default
there) against the one-cycle pass, bit for bit: periodic and walled axes, strips from two
wide to many, runs of a few rows and of hundreds, every medium, both storages, with and
without the D2Q5 field, calls of every remainder, the residual's u(t - 1) planes and a
recorded pass. Equal inputs and the same per-node arithmetic, so the tolerance is zero."""
import numpy as np
import pytest
import torch

from paper_1311_7239_amd import inputs as I
from paper_1311_7239_amd import lbm

pytestmark = pytest.mark.gpu

P, W = I.PERIODIC, I.WALLS


def _phi(nx, ny):
    x, y = np.arange(nx, dtype=np.float32), np.arange(ny, dtype=np.float32)
    g = np.outer(np.sin(0.05 * y), np.cos(0.03 * x)) + np.outer(np.cos(0.011 * y), np.sin(0.2 * x))
    return np.clip(0.45 + 0.15 * g, 0.1, 0.95).astype(np.float32)


def _case(bc_x, bc_y, nx, ny, medium, heat):
    c = I.natural_convection(n=64) if heat else I.lid_cavity(n=64)
    c.nx, c.ny, c.bc_x, c.bc_y, c.nu, c.ax, c.ay = nx, ny, bc_x, bc_y, 0.1, 1e-6, -2e-6
    c.lid_ux = 0.05 if bc_y == I.WALLS else 0.0
    if heat:
        c.gbeta *= 100.0
    if medium != "uniform":
        c.phi, c.dp, c.Fphi = _phi(nx, ny), I.ergun_dp(30.0, 0.4), None
    return c


def _solver(case, medium, storage=lbm.FP32_DEV, **kw):
    desc = lbm.desc_from_case(case, storage=storage, **{k: v for k, v in kw.items() if k == "ckpt_every"})
    kap = phi = None
    if medium != "uniform":
        phi = torch.from_numpy(case.phi).cuda()
    if medium == "kappa":
        kap = (150.0 * (1 - phi) ** 2 / (phi ** 3 * case.dp ** 2)).contiguous()
        desc.medium = lbm.MEDIUM_PHI_KAPPA
    return lbm.Solver(desc, phi=phi, kappa=kap, **{k: v for k, v in kw.items() if k != "ckpt_every"})


CASES = [
    (P, W, 777, 1000, "kappa", False, lbm.FP32_DEV),
    (W, W, 701, 650, "uniform", False, lbm.FP32_DEV),
    (W, P, 129, 3001, "ergun", False, lbm.FP32_DEV),
    (P, P, 130, 2701, "ergun", False, lbm.FP32_DEV),
    (P, W, 5001, 70, "ergun", False, lbm.FP32_DEV),     # runs of a few rows
    (W, W, 128, 2900, "uniform", False, lbm.FP32_DEV),  # each strip next to a wall
    (P, P, 2049, 2048, "ergun", False, lbm.FP32_DEV),
    (W, P, 1201, 333, "kappa", False, lbm.FP16_DEV),
    (P, W, 901, 601, "ergun", False, lbm.FP16_DEV),
    (W, W, 900, 401, "uniform", False, lbm.FP16_DEV),
    (W, W, 600, 450, "uniform", True, lbm.FP32_DEV),
    (W, P, 129, 2001, "ergun", True, lbm.FP32_DEV),
    (W, W, 3001, 90, "kappa", True, lbm.FP32_DEV),
    (W, P, 640, 513, "uniform", True, lbm.FP16_DEV),
]


@pytest.mark.parametrize("bc_x,bc_y,nx,ny,medium,heat,storage", CASES)
def test_rolling_pass_is_bitwise_the_one_cycle_pass(bc_x, bc_y, nx, ny, medium, heat, storage):
    case = _case(bc_x, bc_y, nx, ny, medium, heat)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    df = 2e-3 * (torch.rand((8, ny, nx), generator=g, device="cuda") - 0.5)
    dg = 0.2 * (torch.rand((5, ny, nx), generator=g, device="cuda") - 0.5) if heat else None
    a, b = (_solver(case, medium, storage) for _ in range(2))
    a.set_time_blocking(1)
    for s in (a, b):
        s.set_populations(df, dg)
    for chunk in (7, 4, 6, 11, 13, 3, 5):
        a.step(chunk)
        b.step(chunk)
        fa, ga = a.populations(heat)
        fb, gb = b.populations(heat)
        torch.cuda.synchronize()
        assert torch.equal(fa, fb), (chunk, a.time)
        assert not heat or torch.equal(ga, gb), (chunk, a.time)
        assert a.reduce() == b.reduce(), (chunk, a.time)


@pytest.mark.parametrize("heat", [False, True])
def test_rolling_passes_stop_at_checkpoints(heat):
    """The gradient recomputes from the checkpoints, so equal gradients need equal checkpoints."""
    case = _case(W if heat else P, W, 700, 601, "ergun", heat)
    out = []
    for cycles in (1, 0):
        s = _solver(case, "ergun", ckpt_every=9, max_steps_recorded=24)
        if cycles:
            s.set_time_blocking(cycles)
        s.step(24)
        _, u, _ = s.macroscopic()
        g, _ = s.backward(u)
        torch.cuda.synchronize()
        out.append((u, g))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
