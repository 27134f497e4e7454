"""Deep passes of the recorded run and of its reverse mode (the default on small domains)
against one step per launch: the medium gradients bit for bit, the parameter gradients to
the rounding of their sums, the tangent bit for bit. Both boundary kinds and periodic axes, with and without the
thermal model, whole domains in one workgroup and tiled ones, frames of both sizes and
segments of every length, over two calls."""
import numpy as np
import pytest
import torch

from paper_1311_7239_amd import inputs as I
from paper_1311_7239_amd import lbm

pytestmark = pytest.mark.gpu


def _cut(c, nx, ny):
    c.nx, c.ny = nx, ny
    if c.phi is not None:
        c.phi = np.ascontiguousarray(c.phi[:ny, :nx])
    return c


def _channel(nx, ny):
    return _cut(I.lognormal_channel(n=max(nx, ny), seed=3, ell=8.0, K_ref=30.0, drive=0.05), nx, ny)


def _cavity(nx, ny):
    return _cut(I.lid_cavity(n=max(nx, ny), heterogeneous=True, ell=6.0), nx, ny)


def _periodic(nx, ny):
    c = _channel(nx, ny)
    c.bc_x = c.bc_y = I.PERIODIC
    return c


def _heat(nx, ny):
    c, m = I.natural_convection(n=max(nx, ny)), _cavity(nx, ny)
    c.nx, c.ny, c.phi, c.dp = nx, ny, m.phi, m.dp
    c.gbeta *= 1e2
    return c


CASES = {
    # name: (case, checkpoint distance, 1/K plane)
    "channel_8x64": (lambda: _channel(8, 64), 40, False),
    "cavity_27x29": (lambda: _cavity(27, 29), 7, True),
    "periodic_31x40": (lambda: _periodic(31, 40), 23, False),
    "channel_100x37": (lambda: _channel(100, 37), 23, True),
    "cavity_190x203": (lambda: _cavity(190, 203), 30, False),
    "channel_401x350": (lambda: _channel(401, 350), 11, False),
    "heat_20x30": (lambda: _heat(20, 30), 40, False),
    "heat_111x90": (lambda: _heat(111, 90), 23, False),
    "channel_520x500": (lambda: _channel(520, 500), 23, False),
    "heat_330x301": (lambda: _heat(330, 301), 13, False),
    "heat_450x417": (lambda: _heat(450, 417), 13, False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_deep_gradients_are_those_of_single_steps(name):
    make, every, kappa_plane = CASES[name]
    case = make()
    kap = None
    if kappa_plane:
        kap = torch.from_numpy((150.0 * (1 - case.phi) ** 2 / (case.phi ** 3 * case.dp ** 2)).astype(np.float32)).cuda()
    out = []
    for single in (True, False):
        desc = lbm.desc_from_case(case, ckpt_every=every)
        if kappa_plane:
            desc.medium = lbm.MEDIUM_PHI_KAPPA
        s = lbm.Solver(desc, phi=torch.from_numpy(case.phi).cuda(), kappa=kap, max_steps_recorded=60)
        if single:
            s.set_time_blocking(1)
        s.step(19)
        s.step(30)
        _, u, _ = s.macroscopic()
        w = torch.cos(torch.arange(u.numel(), device="cuda", dtype=torch.float32)).reshape(u.shape)
        g, gk = s.backward(w, want_kappa=kappa_plane)
        g2, _, theta = s.backward_params(w)
        torch.cuda.synchronize()
        assert torch.equal(g, g2)
        out.append((u, g, gk, np.array([theta[k] for k in sorted(theta)])))
    (u0, g0, k0, t0), (u1, g1, k1, t1) = out
    assert torch.equal(u0, u1) and torch.equal(g0, g1)
    assert k0 is None or torch.equal(k0, k1)
    # both add the same FP32 shares of a node and step in FP64, in another order: at most
    # 7e6 shares, 2^-53 of their moduli each, for a sum 1e2 times smaller than their moduli
    np.testing.assert_allclose(t1, t0, rtol=1e-7)


@pytest.mark.parametrize("name", [n for n in CASES if not n.startswith("heat")])
def test_deep_tangent_is_that_of_single_steps(name):
    make, every, kappa_plane = CASES[name]
    case = make()
    kap = None
    if kappa_plane:
        kap = torch.from_numpy((150.0 * (1 - case.phi) ** 2 / (case.phi ** 3 * case.dp ** 2)).astype(np.float32)).cuda()
    out = []
    for single in (True, False):
        desc = lbm.desc_from_case(case, ckpt_every=every)
        if kappa_plane:
            desc.medium = lbm.MEDIUM_PHI_KAPPA
        s = lbm.Solver(desc, phi=torch.from_numpy(case.phi).cuda(), kappa=kap, max_steps_recorded=60)
        if single:
            s.set_time_blocking(1)
        s.step(49)
        w = torch.cos(torch.arange(case.nx * case.ny, device="cuda", dtype=torch.float32)).reshape(case.ny, case.nx)
        out.append(s.tangent(w, (0.3 * case.nu, 0.1, 0.2, 0.05)))
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
