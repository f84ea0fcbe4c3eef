"""The radius graph's choice of its grid, run on the host (no GPU): it ends for
every box, and points within the radius are in adjacent cells."""
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2402_15106_amd import build  # noqa: E402

INF, NAN, BIG = float("inf"), float("nan"), 3e38


@pytest.fixture(scope="module")
def grid_check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("grid") / "grid_check")
    subprocess.run([build._hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-ffp-contract=off",
                    os.path.join(ROOT, "tests", "native", "grid_check.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=120)

    def run(D, r, cap, pts):
        text = "%d %r %d %d %s\n" % (D, r, cap, len(pts), " ".join("%r" % float(v) for p in pts for v in p))
        out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True, timeout=10).stdout
        return tuple(int(v) for v in out.split())
    return run


@pytest.mark.parametrize("D,r,cap,pts,pairs", [
    (2, 0.1, 64, [(0, 0), (INF, 0), (0.05, 0), (1, 1)], 1),
    (3, 0.1, 64, [(-INF, NAN, INF), (1, 2, 3), (1, 2, 3.05)], 1),
    (2, 0.1, 64, [(INF, INF), (-INF, NAN)], 0),
    (2, 0.1, 1, [(INF, 0.0), (0.0, 0.0)], 0),
    (2, 1.0, 64, [(-BIG, -BIG), (BIG, BIG), (0, 0)], 0),
    (3, 0.0, 64, [(-BIG, BIG, 0), (BIG, -BIG, 0), (BIG, -BIG, 0)], 1),
    (2, 1e30, 64, [(BIG, 0), (-BIG, 1), (INF, 0)], 3),   # the square overflows: every distance but NaN passes
    (2, 0.5, 64, [], 0),
])
def test_grid_of_extreme_boxes(grid_check, D, r, cap, pts, pairs):
    ncell, got, apart = grid_check(D, r, cap, pts)
    assert 1 <= ncell <= cap and got == pairs and apart == 0


def test_far_points_leave_the_others_their_cells(grid_check):
    """Coordinates that are not finite do not coarsen the grid of the others."""
    pts = [tuple(p) for p in np.random.default_rng(3).uniform(0, 1, (200, 2)).astype(np.float32)]
    plain = grid_check(2, 0.05, 464, pts)
    assert grid_check(2, 0.05, 464, pts + [(INF, 0.5), (NAN, NAN)]) == plain and plain[0] > 300 and plain[2] == 0
