"""The Hilbert build's boundary cells, row by row: rows of few pairs by a
wavefront, of many pairs or cells by a bitmap, boxes wider than one bitmap,
windows whose border cells belong to them.  Runs and codes are those of the
global sorts, and of a handle the oracle answers alike."""
import time

import numpy as np
import pytest
import torch

from gen import polygons_from_rings, uniform_points
from test_gpu_parity import run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


def both(sba, polys, eps, **kw):
    """A handle by the rows and one by the global sorts: the runs and sets of each."""
    out = []
    for off in (0, 2):
        sba.lib().sba_debug_build_paths(off)
        try:
            A = sba.Approx.from_polygons(polys, eps, kind="hilbert", **kw)
            if A.info()["gw"]:  # something of a polygon lies in the window
                assert sba.lib().sba_debug_last_build_paths() & 2 == (0 if off else 2)
        finally:
            sba.lib().sba_debug_build_paths(0)
        starts, ids = A.runs()
        out.append((A, starts.cpu().numpy(), ids.cpu().numpy(), *A.sets()))
    return out


def same(sba, polys, eps, **kw):
    one, two = both(sba, polys, eps, **kw)
    for a, b in zip(one[1:], two[1:]):
        np.testing.assert_array_equal(a, b)
    return one[0]


def fans(n, width, height, seed):
    """n quadrilaterals of edges from flat to steep, anywhere in the box."""
    r = np.random.default_rng(seed)
    return polygons_from_rings(
        [[np.stack((r.integers(0, width, 4), r.integers(0, height, 4)), 1)] for _ in range(n)])


# boxes of one bitmap's width (65,536 cells), one more and several; flat edges
# make rows of few pairs and many cells
@pytest.mark.parametrize("width", [1500, 65_530 * 7, 65_545 * 7, 200_000 * 7])
@pytest.mark.parametrize("n", [1, 5, 40])
@pytest.mark.parametrize("kw", [dict(), dict(centre_sampled=True), dict(boundary_only=True)])
def test_few_pairs_a_row(sba, orc, width, n, kw):
    polys = fans(min(n, 12) if width < 2000 else n, width, 900, width + n)
    A = same(sba, polys, 10, **kw)
    xy = uniform_points(40_001, -50, width + 50, 3)
    xy[1::2] = np.random.default_rng(4).integers(-50, 950, size=40_001)
    okw = {"centre": True} if "centre_sampled" in kw else kw
    want = orc.Approx(polys, 10, **okw).aggregate(xy, None)
    np.testing.assert_array_equal(run_agg(A, xy)[0], want[0])


# windows of one row, one column, one cell and more, off the polygons too
@pytest.mark.parametrize("win", [(100, 100, 101, 101), (0, 300, 500_000, 301),
                                 (3000, 0, 3001, 900), (2000, 200, 470_000, 700),
                                 (-500, -500, 900_000, 1500)])
def test_windows(sba, win):
    for n in (1, 20):
        same(sba, fans(n, 480_000, 900, 17 * n), 10, window=win)


@pytest.mark.parametrize("pairs", [62, 63, 64, 65, 66])
def test_rows_at_the_edge_of_a_wavefront(sba, pairs):
    """Upright slivers: one pair a side and row but the last and the first."""
    rings = [[[(20 * k, 0), (20 * k + 3, 0), (20 * k + 3, 200), (20 * k, 200)]]
             for k in range((pairs + 1) // 2)]
    if pairs & 1:  # a triangle whose lower tip leaves one side out of the first rows
        rings[-1] = [[(20 * pairs, 90), (20 * pairs + 4, 200), (20 * pairs, 200)]]
    polys = polygons_from_rings(rings)
    same(sba, polys, 10)
    same(sba, polys, 10, window=(5, 5, 20 * pairs, 190))


def test_a_wide_ring_takes_little_longer_than_its_grid(sba):
    """Ten times as long while every row had a bitmap of the box's width."""
    t = np.linspace(0, 2 * np.pi, 64, endpoint=False)
    ring = np.stack((500_000 + 500_000 * np.cos(t), 500_000 + 500_000 * np.sin(t)), 1).astype(int)
    polys = polygons_from_rings([[ring]])
    t = [torch.from_numpy(a).cuda() for a in (polys.ring_off, polys.vert_off, polys.xy)]

    def best(kind):
        ms = []
        for _ in range(6):
            t0 = time.perf_counter()
            A = sba.Approx(*t, 2, kind=kind)
            ms.append(time.perf_counter() - t0)
            A.close()
        return min(ms)

    assert best("hilbert") < 2 * best("grid")
