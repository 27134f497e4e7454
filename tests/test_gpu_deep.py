"""The deep pass (many cycles per launch on small domains, the default there) against the
one-cycle pass, bit for bit: every boundary kind, medium, storage, whole domains in one
workgroup and tiled ones, the three frame sizes, passes of every length, the residual's
u(t - 1) planes and a recorded pass's checkpoints. Equal inputs and the same per-node
arithmetic, so the tolerance is zero."""
import numpy as np
import pytest
import torch

from paper_1311_7239_amd import inputs as I
from paper_1311_7239_amd import lbm

pytestmark = pytest.mark.gpu


def _cavity(nx, ny, grf=False, nee=False):
    c = I.lid_cavity(n=max(nx, ny), heterogeneous=grf, ell=6.0, nee=nee)
    c.nx, c.ny = nx, ny
    if grf:
        c.phi = np.ascontiguousarray(c.phi[:ny, :nx])
    return c


def _channel(n, ny):
    c = I.lognormal_channel(n=max(n, ny), seed=3, ell=8.0, K_ref=30.0, drive=0.05)
    c.nx, c.ny = n, ny
    c.phi = np.ascontiguousarray(c.phi[:ny, :n])
    return c


def _heat(nx, ny, nee=False):
    c = I.natural_convection(n=max(nx, ny), nee=nee)
    c.nx, c.ny, c.gbeta = nx, ny, c.gbeta * 1e2
    return c


def _layered(nx, ny):
    return I.partial_couette(nx=nx, ny=ny)


def _periodic(nx, ny):
    c = I.poiseuille_channel(nx=nx, ny=ny)
    c.bc_y, c.ay = I.PERIODIC, 2e-5
    return c


CASES = {
    "one_row": lambda: _periodic(300, 1),
    "poiseuille_8x64": lambda: I.poiseuille_channel(),
    "poiseuille_node_8x64": lambda: I.poiseuille_channel(nee=True),
    "layered_2x80": lambda: _layered(2, 80),
    "layered_3x600": lambda: _layered(3, 600),
    "periodic_27x29": lambda: _periodic(27, 29),
    "periodic_61x67": lambda: _periodic(61, 67),
    "cavity_33x21": lambda: _cavity(33, 21),
    "cavity_70x131_grf": lambda: _cavity(70, 131, grf=True),
    "cavity_300x7": lambda: _cavity(300, 7),
    "cavity_511x257": lambda: _cavity(511, 257),
    "cavity_node_65x40": lambda: _cavity(65, 40, grf=True, nee=True),
    "cavity_node_601x590": lambda: _cavity(601, 590, nee=True),
    "channel_129x200": lambda: _channel(129, 200),
    "heat_25x24": lambda: _heat(25, 24),
    "heat_100x37": lambda: _heat(100, 37),
    "heat_400x301": lambda: _heat(400, 301),
    "heat_node_20x20": lambda: _heat(20, 20, nee=True),
    "heat_node_90x33": lambda: _heat(90, 33, nee=True),
}


def _one_cycle(s, case):
    if I.NEE in (case.bc_x, case.bc_y):
        s.set_schedule(128, 1, 2, 1)     # on-node walls: the one-cycle kernel in the caller's shape
    else:
        s.set_time_blocking(1)


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
    for chunk in (1, 4, 10, 3, 23, 2, 61):    # t = 0, the frame sizes, several passes of unequal length
        a.step(chunk)
        b.step(chunk)
        fa, ga = a.populations(thermal=case.thermal)
        fb, gb = b.populations(thermal=case.thermal)
        torch.cuda.synchronize()
        assert torch.equal(fa, fb), (chunk, a.time)
        assert ga is None or torch.equal(ga, gb), (chunk, a.time)
        assert a.reduce() == b.reduce(), (chunk, a.time)


@pytest.mark.parametrize("every", [1, 7, 16])
def test_recorded_deep_passes_leave_the_checkpoints_of_one_cycle_passes(every):
    """The gradient recomputes from the checkpoints, so equal gradients need equal checkpoints."""
    case = _channel(90, 50)
    out = []
    for cycles in (1, 0):
        s = lbm.solver_for_case(case, ckpt_every=every, max_steps_recorded=45)
        if cycles:
            s.set_time_blocking(cycles)
        s.step(30)
        s.step(15)
        _, u, _ = s.macroscopic()
        g, _ = s.backward(u)
        torch.cuda.synchronize()
        out.append((u, g))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
