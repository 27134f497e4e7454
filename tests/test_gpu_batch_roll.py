"""Rolling passes of a batch (the default there) against one-cycle passes of each domain
alone, bit for bit: domains narrower than a strip and of a few rows, periodic axes of a
strip's width, every medium, both storages, with and without the D2Q5 field, one group of
domains and several, calls of every remainder, and the tiles after them. Equal inputs and
the same per-node arithmetic, so the tolerance is zero."""
import pytest
import torch

from paper_1311_7239_amd import inputs as I
from paper_1311_7239_amd import lbm
from tests.test_gpu_roll import _case, _solver

pytestmark = pytest.mark.gpu

P, W = I.PERIODIC, I.WALLS
SMALL = [(W, W, 16, 16), (W, W, 64, 17), (W, W, 65, 140), (P, W, 64, 16), (W, P, 118, 64), (P, P, 67, 129),
         (W, W, 119, 333), (P, W, 301, 90), (W, W, 700, 222)]
LARGE = [(W, W, 1000 + 7 * k, 1011 - 9 * k) for k in range(8)]   # several groups


def _batch(cases, media, storage):
    descs, phis, kappas = [], [], []
    for case, medium in zip(cases, media):
        d = lbm.desc_from_case(case, storage=storage)
        phi = kap = None
        if medium != "uniform":
            phi = torch.from_numpy(case.phi).cuda()
        if medium == "kappa":
            kap = (150.0 * (1 - phi) ** 2 / (phi ** 3 * case.dp ** 2)).contiguous()
            d.medium = lbm.MEDIUM_PHI_KAPPA
        descs.append(d)
        phis.append(phi)
        kappas.append(kap)
    return lbm.Batch(descs, phis=phis, kappas=kappas)


@pytest.mark.parametrize("shapes,media,heat,storage", [
    (SMALL, "mixed", False, lbm.FP32_DEV),
    (SMALL, "uniform", False, lbm.FP32_DEV),
    (SMALL, "mixed", False, lbm.FP16_DEV),
    (SMALL, "uniform", False, lbm.FP16_DEV),
    (SMALL, "mixed", True, lbm.FP32_DEV),
    (SMALL, "uniform", True, lbm.FP32_DEV),
    (SMALL, "uniform", True, lbm.FP16_DEV),
    (SMALL[:1], "uniform", False, lbm.FP32_DEV),
    (LARGE, "uniform", False, lbm.FP32_DEV),
    (LARGE, "mixed", True, lbm.FP32_DEV),
])
def test_batched_rolling_pass_is_bitwise_the_one_cycle_pass(shapes, media, heat, storage):
    kinds = ["uniform"] * len(shapes) if media == "uniform" else [("ergun", "uniform", "kappa")[k % 3] for k in range(len(shapes))]
    cases = [_case(bx, by, nx, ny, m, heat) for (bx, by, nx, ny), m in zip(shapes, kinds)]
    b = _batch(cases, kinds, storage)
    singles = []
    for k, (case, medium) in enumerate(zip(cases, kinds)):
        g = torch.Generator(device="cuda")
        g.manual_seed(k)
        df = 2e-3 * (torch.rand((8, case.ny, case.nx), generator=g, device="cuda") - 0.5)
        dg = 0.2 * (torch.rand((5, case.ny, case.nx), generator=g, device="cuda") - 0.5) if heat else None
        s = _solver(case, medium, storage)
        s.set_time_blocking(1)
        s.set_populations(df, dg)
        b.set_populations(k, df, dg)
        singles.append(s)
    for n, chunk in enumerate((7, 4, 6, 11, 13, 3, 5, 8)):
        if n == 7:
            b.set_time_blocking(2)   # tiles go on from the rolling passes' state
        b.step(chunk)
        for k, s in enumerate(singles):
            s.step(chunk)
            fb, fs = b.populations(k, thermal=heat), s.populations(thermal=heat)
            torch.cuda.synchronize()
            for x, y in zip(fb if heat else (fb,), fs if heat else fs[:1]):
                assert torch.equal(x, y), (k, shapes[k], chunk, s.time)
            assert b.reduce(k) == s.reduce(), (k, shapes[k], chunk)
