"""Deep-pass plans followed on the host (tests/plan/deep_walk.cpp, which runs the kernels' own
index arithmetic): every LDS read of a launch is of the node that the collision needs, as the
cycle before left it, no position lies outside the frame, and the tiles cover the domain. All
pairs of boundary kinds, thin and odd sizes, and the sizes around the switches of the plan."""
import os
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parent.parent
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
P, W, N = 0, 1, 2   # LBM_PERIODIC, LBM_WALLS, LBM_WALLS_NEE
MOST = 1 << 30

pytestmark = pytest.mark.skipif(not (shutil.which(HIPCC) or os.path.exists(HIPCC)), reason="hipcc not available")


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = tmp_path_factory.mktemp("plan") / "deep_walk"
    r = subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-O2", "-std=c++17",
                        "-ffp-contract=off", "-I", str(ROOT / "paper_1311_7239_amd" / "csrc"),
                        str(ROOT / "tests" / "plan" / "deep_walk.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(lines):
        text = "".join(" ".join(map(str, q)) + "\n" for q in lines)
        r = subprocess.run([str(exe)], input=text, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr
        out = [tuple(map(int, q.split())) for q in r.stdout.splitlines()]
        assert len(out) == len(lines)
        return out

    return run


SIZES = [1, 2, 3, 4, 5, 7, 8, 9, 13, 16, 20, 22, 23, 24, 25, 27, 29, 31, 32, 33, 40, 47, 64, 80, 96, 131, 200, 301, 640]


def _check(walk, lines):
    planned = 0
    for q, (tx, ty, cycles, fits, bad) in zip(lines, walk(lines)):
        assert bad == 0, (q, (tx, ty, cycles), bad)
        assert cycles == 0 or fits == 1, q
        planned += cycles > 0
    return planned


@pytest.mark.parametrize("bx,by", [(N, N), (P, N), (N, P), (W, W), (P, W), (W, P), (P, P)])
@pytest.mark.parametrize("heat", [0, 1])
def test_every_read_of_a_plan_is_of_the_cycle_before(walk, bx, by, heat):
    least = {P: 1, W: 2, N: 3}
    lines = [(nx, ny, bx, by, heat, MOST, 0, 0) for nx in SIZES for ny in SIZES
             if nx >= least[bx] and ny >= least[by] and nx * ny <= 50000]
    assert _check(walk, lines) > len(lines) // 2


def test_tiles_of_one_node_at_an_on_node_wall_are_refused(walk):
    for q, want in [((24, 24, N, N, 0, MOST, 16, 16), 0), ((24, 24, N, N, 0, MOST, 12, 12), 1),
                    ((24, 24, N, N, 0, MOST, 12, 13), 0), ((8, 80, P, N, 0, MOST, 5, 51), 0),
                    ((3, 200, N, N, 0, MOST, 2, 16), 0), ((3, 200, N, N, 0, MOST, 1, 16), 1),
                    ((24, 24, W, W, 0, MOST, 16, 16), 1)]:
        assert walk([q])[0][3] == want, q


def test_tile_bounds_of_the_longest_axes_stay_in_range(walk):
    """One-column domains of 1.6 to 2.7 million on-node rows: tile bounds are products of the
    axis and its number of tiles in 32 bits, beyond which there is no plan."""
    lines = [(1, ny, P, N, heat, MOST, 0, 0) for heat in (0, 1)
             for ny in (1_500_000, 1_677_721, 1_700_000, 1_900_000, 2_079_000, 2_097_000, 2_500_000)]
    _check(walk, lines)
