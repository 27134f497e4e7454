"""Which pass lbm_step launches (tests/plan/pass_driver.cpp on the null device): what
lbm_next_pass reports is what runs, for every kind of pass, and the passes of a call."""
import os
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_1311_7239_amd" / "csrc"
BUILD = ROOT / "paper_1311_7239_amd" / "_build"
OBJECTS = [BUILD / f for f in ("lbm_abi.cpp.o", "lbm_kernels.hip.o", "lbm_adjoint.hip.o")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CLANG = pathlib.Path(HIPCC).resolve().parent.parent / "llvm" / "bin" / "clang++"
P, W, N = 0, 1, 2                       # LBM_PERIODIC, LBM_WALLS, LBM_WALLS_NEE
UNIFORM, ERGUN, KAPPA = 0, 1, 2         # LBM_MEDIUM_*

pytestmark = pytest.mark.skipif(not (shutil.which(HIPCC) or os.path.exists(HIPCC)) or not CLANG.exists()
                                or not all(o.exists() for o in OBJECTS), reason="hipcc or kernel objects missing")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("passes")
    dev_o, exe = tmp / "null_device.o", tmp / "pass_driver"
    r = subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                        "-I", str(CSRC), "-c", str(ROOT / "tests" / "sanitize" / "null_device.cpp"), "-o", str(dev_o)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    # linked without the HIP runtime: every HIP symbol resolves to the null device
    r = subprocess.run([str(CLANG), "-O1", "-std=c++17", "-I", str(ROOT / "include"),
                        str(ROOT / "tests" / "plan" / "pass_driver.cpp"), str(dev_o), *map(str, OBJECTS), "-lm",
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def passes(n, nx, ny, bx=W, by=W, medium=UNIFORM, half=0, heat=0, j=0, every=0, mode=0, t=1, count=1):
        line = f"{count} {nx} {ny} {bx} {by} {medium} {half} {heat} {j} {every} {mode} {t} {n}\n"
        r = subprocess.run([str(exe)], input=line, capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        out = r.stdout.split()
        assert not any(q.endswith("?") for q in out), out
        return out

    def reverse(nx, ny, every, steps, theta=0, bx=P, by=W, medium=ERGUN, heat=0):
        r = subprocess.run([str(exe), "reverse"], input=f"{nx} {ny} {bx} {by} {medium} {heat} {every} {steps} {theta}\n",
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return dict(zip(("rec_deep", "rec_roll", "rec_tiles", "deep", "steps", "tan_deep", "tan_steps"),
                        map(int, r.stdout.split())))

    passes.reverse = reverse
    return passes


@pytest.mark.parametrize("want,kw", [
    ("deep", dict(nx=8, ny=64, bx=P)), ("deep", dict(nx=512, ny=512)), ("deep", dict(nx=200, ny=200, bx=N, by=N)),
    ("deep", dict(nx=300, ny=300, heat=1)), ("rolling", dict(nx=777, ny=1000, bx=P, medium=KAPPA, j=1)),
    ("rolling", dict(nx=1024, ny=1024, heat=1)), ("rolling", dict(nx=901, ny=601, medium=ERGUN, half=1)),
    ("strips", dict(nx=8192, ny=8192, bx=P, medium=ERGUN)), ("strips", dict(nx=4099, ny=3001, bx=P, medium=ERGUN, half=1)),
    ("tiles", dict(nx=2000, ny=2000, bx=N, by=N)), ("rolling", dict(nx=300, ny=200, count=5)),
    ("rolling", dict(nx=200, ny=200, heat=1, count=27)), ("tiles", dict(nx=200, ny=200, bx=N, by=N, count=3)),
    ("tiles", dict(nx=512, ny=512, mode=2)), ("tiles", dict(nx=1024, ny=1024, mode=3)),
    ("tiles", dict(nx=8192, ny=8192, bx=P, medium=ERGUN, mode=4)), ("tiles", dict(nx=300, ny=200, count=5, mode=4)),
])
def test_the_reported_pass_is_the_one_launched(driver, want, kw):
    out = driver(48, **kw)
    assert all(q.startswith(want) for q in out), out
    out = driver(48 if want == "deep" else 49, t=0, **kw)   # with the first cycle, which only deep passes take in
    assert out[0] == "tiles1" or want == "deep", out
    assert all(q.startswith(want) for q in out[1:]), out


def test_passes_stop_at_checkpoints(driver):
    for kw in (dict(nx=90, ny=50, bx=P), dict(nx=700, ny=601, medium=ERGUN), dict(nx=2800, ny=2001, medium=ERGUN)):
        t = 3
        for q in driver(40, every=11, t=t, **kw):
            k = int(q.lstrip("adeghilnoprst"))
            assert t // 11 == (t + k - 1) // 11, (kw, t, q)
            t += k
        assert t == 43


# Passes of three and four cycles beyond the caches: those of tiles, which are faster there.
@pytest.mark.parametrize("n,want,kw", [
    (4, "tiles4", dict(nx=8192, ny=8192, bx=P, medium=ERGUN)),
    (20, "strips6 strips6 tiles4 tiles4", dict(nx=8192, ny=8192, bx=P, medium=ERGUN)),
    (7, "tiles4 tiles3", dict(nx=3000, ny=3000)), (10, "strips6 tiles4", dict(nx=4096, ny=4096)),
    (4, "strips4", dict(nx=2300, ny=2300, bx=P, medium=ERGUN)),
    (4, "strips4", dict(nx=4099, ny=3001, bx=P, medium=ERGUN, half=1)), (4, "tiles4", dict(nx=4200, ny=4200, half=1)),
    (3, "tiles3", dict(nx=2800, ny=2800, bx=P, medium=KAPPA, j=1)),
    (8, "tiles4 tiles4", dict(nx=2800, ny=2800, bx=P, medium=KAPPA, j=1)),
    (10, "rolling6 tiles4", dict(nx=2800, ny=2800, bx=P, medium=KAPPA)),
    (7, "rolling4 rolling3", dict(nx=777, ny=1000, bx=P, medium=KAPPA, j=1)),
    (7, "rolling4 tiles3", dict(nx=2048, ny=2048, bx=P, medium=ERGUN)),
    (3, "tiles3", dict(nx=1221, ny=2126, medium=ERGUN)), (3, "rolling3", dict(nx=1221, ny=2000, medium=ERGUN)),
    (3, "tiles3", dict(nx=1700, ny=1700, half=1)), (3, "rolling3", dict(nx=688, ny=2264, half=1, medium=ERGUN)),
    (3, "rolling3", dict(nx=1100, ny=1100, half=1)),
    (4, "tiles2 tiles2", dict(nx=1000, ny=1000, heat=1, medium=KAPPA)),
    (7, "rolling3 tiles2 tiles2", dict(nx=1000, ny=1000, heat=1, medium=KAPPA)),
    (7, "rolling4 rolling3", dict(nx=1000, ny=1000, heat=1)), (7, "rolling4 tiles3", dict(nx=2100, ny=2100, heat=1)),
    (7, "tiles3 tiles3 tiles1", dict(nx=2100, ny=2100, heat=1, medium=KAPPA)),
    (4, "tiles3 tiles1", dict(nx=3000, ny=3000, mode=3)),
])
def test_short_passes_of_large_domains(driver, n, want, kw):
    assert " ".join(driver(n, **kw)) == want


# The same for batches, by the bytes of all their states (the null device's tuner takes tiles
# of four cycles, two with the thermal model).
@pytest.mark.parametrize("n,want,kw", [
    (3, "tiles3", dict(nx=500, ny=500, count=17)), (4, "tiles4", dict(nx=500, ny=500, count=17)),
    (5, "tiles3 tiles2", dict(nx=500, ny=500, count=17)), (8, "tiles4 tiles4", dict(nx=500, ny=500, count=17)),
    (20, "rolling6 rolling6 tiles4 tiles4", dict(nx=500, ny=500, count=17, medium=KAPPA)),
    (4, "tiles2 tiles2", dict(nx=500, ny=500, count=40, half=1, mode=0, heat=1, medium=KAPPA)),
    (20, "rolling6 rolling6 rolling4 rolling4", dict(nx=500, ny=500, count=16)),
    (4, "rolling4", dict(nx=500, ny=500, count=30, half=1)), (4, "tiles4", dict(nx=500, ny=500, count=34, half=1)),
    (7, "rolling4 rolling3", dict(nx=500, ny=500, count=17, heat=1)),
    (4, "rolling4", dict(nx=36, ny=40, count=2000)),   # rows of 64 elements, of which 36 count
    (4, "tiles2 tiles2", dict(nx=200, ny=200, count=9, heat=1, medium=KAPPA)),
])
def test_short_passes_of_large_batches(driver, n, want, kw):
    assert " ".join(driver(n, **kw)) == want


# Small domains: one, two and sometimes four cycles in tiles.
@pytest.mark.parametrize("n,want,kw", [
    (1, "deep1", dict(nx=128, ny=128)), (2, "deep2", dict(nx=128, ny=128)), (1, "tiles1", dict(nx=256, ny=256)),
    (2, "tiles2", dict(nx=200, ny=200, bx=P, medium=ERGUN)), (1, "deep1", dict(nx=200, ny=200, half=1)),
    (2, "tiles2", dict(nx=250, ny=250, heat=1)), (2, "deep2", dict(nx=100, ny=100, heat=1)),
    (2, "deep2", dict(nx=200, ny=200, bx=N, by=N)), (2, "tiles1 tiles1", dict(nx=512, ny=512, bx=N, by=N)),
    (4, "tiles2 tiles2", dict(nx=512, ny=512)), (4, "deep4", dict(nx=300, ny=300)),
    (3, "tiles2 tiles1", dict(nx=642, ny=274, bx=P, by=P, medium=ERGUN)), (3, "deep3", dict(nx=400, ny=400)),
    (3, "deep3", dict(nx=500, ny=500, medium=KAPPA)), (3, "deep3", dict(nx=500, ny=500, half=1)),
    (4, "tiles2 tiles2", dict(nx=317, ny=271, heat=1)), (4, "deep4", dict(nx=250, ny=250, heat=1)),
    (8, "deep4 deep4", dict(nx=400, ny=400, heat=1)),
    (6, "tiles2 tiles2 tiles2", dict(nx=540, ny=540)), (10, "rolling4 rolling4 tiles2", dict(nx=450, ny=450, heat=1)),
    (8, "tiles2 tiles2 tiles2 tiles2", dict(nx=540, ny=540)), (10, "deep5 deep5", dict(nx=540, ny=540)),
    (12, "deep5 deep5 tiles2", dict(nx=540, ny=540)), (16, "rolling4 rolling4 rolling4 rolling4", dict(nx=600, ny=330, bx=P, medium=ERGUN, heat=1)),
    (6, "tiles2 tiles2 tiles2", dict(nx=437, ny=577, half=1)), (6, "deep6", dict(nx=520, ny=505, half=1)),
    (6, "deep5 tiles1", dict(nx=1036, ny=1355, bx=P, by=N, half=1)), (9, "deep7 tiles1 tiles1", dict(nx=980, ny=980, bx=N, by=N)), (9, "deep5 deep4", dict(nx=700, ny=700, bx=N, by=N)),
    (3, "tiles1 tiles1 tiles1", dict(nx=1501, ny=557, bx=P, by=N)), (3, "deep3", dict(nx=900, ny=900, bx=N, by=P)),
    (3, "tiles1 tiles1 tiles1", dict(nx=557, ny=1501, bx=P, by=N, heat=1)), (5, "deep5", dict(nx=900, ny=900, bx=P, by=N, heat=1)),
    (7, "tiles2 deep5", dict(nx=789, ny=209, bx=P, heat=1)), (4, "tiles2 tiles2", dict(nx=400, ny=400, heat=1, half=1)),
    (8, "tiles2 deep6", dict(nx=400, ny=400, heat=1, half=1)), (14, "deep6 deep6 tiles2", dict(nx=430, ny=430, heat=1, half=1)), (7, "deep7", dict(nx=400, ny=400, heat=1)),
    (8, "tiles2 deep6", dict(nx=400, ny=400, heat=1, medium=ERGUN)), (9, "deep6 deep3", dict(nx=430, ny=430, heat=1, medium=ERGUN)),
    (14, "deep5 deep5 deep4", dict(nx=430, ny=430, heat=1)),
    (6, "rolling4 tiles2", dict(nx=1038, ny=230, heat=1)), (6, "rolling3 rolling3", dict(nx=560, ny=540, heat=1)),
    (12, "tiles2 tiles2 tiles2 tiles2 tiles2 tiles2", dict(nx=1038, ny=230, heat=1, half=1, medium=KAPPA)),
    (7, "deep4 deep3", dict(nx=900, ny=900, bx=N, by=N, half=1)), (6, "deep5 tiles1", dict(nx=900, ny=900, bx=N, by=N, half=1)),
    (7, "deep5 tiles1 tiles1", dict(nx=900, ny=900, bx=N, by=N)),
    (5, "rolling3 tiles2", dict(nx=1038, ny=230, heat=1, half=1, medium=KAPPA)),
    (9, "rolling3 tiles2 tiles2 tiles2", dict(nx=1038, ny=230, heat=1, half=1, medium=KAPPA)),
    (6, "rolling3 rolling3", dict(nx=560, ny=540, heat=1, half=1, medium=KAPPA)),
    (7, "deep6 tiles1", dict(nx=512, ny=512)), (8, "deep6 tiles2", dict(nx=500, ny=500, bx=P, medium=ERGUN)),
    (9, "deep5 tiles2 tiles2", dict(nx=512, ny=512)), (9, "deep9", dict(nx=400, ny=400)),
    (12, "deep6 deep6", dict(nx=512, ny=512)),
    (11, "deep6 deep5", dict(nx=100, ny=100)), (1030, "deep515 deep515", dict(nx=8, ny=64, bx=P)),
])
def test_short_passes_of_small_domains(driver, n, want, kw):
    assert " ".join(driver(n, **kw)) == want


def test_short_segments_of_the_reverse_and_the_forward_mode(driver):
    """Deep passes backward and of the tangent, but not for segments too short for them."""
    r = driver.reverse
    assert r(300, 300, 1, 12)["deep"] == 0 and r(300, 300, 1, 12)["steps"] == 12
    assert r(300, 300, 2, 12)["deep"] == 6 and r(500, 500, 2, 12)["deep"] == 0
    assert r(100, 100, 1, 12)["deep"] == 12 and r(100, 100, 1, 12, theta=1)["deep"] == 0
    assert r(8, 64, 1, 12, theta=1)["deep"] == 12 and r(27, 27, 1, 12, theta=1)["deep"] == 0
    assert r(16, 16, 1, 12)["deep"] == 12 and r(300, 300, 3, 12)["deep"] == 4
    q = r(300, 300, 10, 31, theta=1)   # the last segment is of one step
    assert q["deep"] == 3 and q["steps"] == 1
    for nx in (8, 100, 300):
        assert r(nx, 64, 2, 12)["tan_deep"] == 0 and r(nx, 64, 2, 12)["tan_steps"] == 12
    q = r(300, 300, 10, 32)
    assert q["tan_deep"] == 3 and q["tan_steps"] == 2


def test_recomputation_with_stress_moments_in_tiles_from_some_size_on(driver):
    r = driver.reverse
    for kw in (dict(medium=ERGUN), dict(medium=KAPPA), dict(medium=ERGUN, bx=W, heat=1)):
        q = r(1500, 1500, 12, 24, theta=1, **kw)
        assert q["rec_roll"] == 0 and q["rec_tiles"] > 0, kw
        assert r(1500, 1500, 12, 24, **kw)["rec_roll"] > 0 and r(700, 700, 12, 24, theta=1, **kw)["rec_roll"] > 0
    assert r(1900, 1900, 4, 24)["rec_roll"] == 5   # the first segment has three cycles after t = 0
    assert r(2048, 2048, 4, 24)["rec_roll"] == 0 and r(2048, 2048, 13, 26)["rec_roll"] == 3
    assert r(2040, 2040, 12, 24, bx=W, heat=1)["rec_roll"] == 0 and r(2040, 2040, 12, 24)["rec_roll"] > 0


@pytest.mark.parametrize("kw", [
    dict(nx=8, ny=64, bx=P), dict(nx=512, ny=512), dict(nx=200, ny=200, bx=N, by=N), dict(nx=1024, ny=1024, heat=1),
    dict(nx=2900, ny=2700, bx=P, medium=ERGUN), dict(nx=300, ny=200, count=5), dict(nx=200, ny=200, heat=1, count=9),
    dict(nx=2000, ny=2000, bx=N, by=N),
])
def test_default_passes_come_back_after_a_mode(driver, kw):
    want = driver(23, t=2, **kw)
    modes = [1] if N in (kw.get("bx"), kw.get("by")) else [1, 2] if "heat" in kw else [1, 2, 3, 4]
    for mode in modes:
        assert all(q[:5] == "tiles" for q in driver(23, t=2, mode=mode, **kw))
        assert driver(23, mode=-mode, **kw) == want   # t = 1 and the step in the mode
