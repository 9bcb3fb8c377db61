"""The block directory of a Hilbert handle covers the stored box: key grids much
larger than the polygons, boxes of one row, one column or a single cell, and of
sizes off the tiles' and squares' edges.  Compared with the oracle."""
import numpy as np
import pytest
import torch

from gen import Polygons, star_polygons, uniform_points, voronoi_partition
from test_gpu_parity import dev, run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


def check(sba, orc, polys, eps, lo, hi, **kw):
    A = sba.Approx.from_polygons(polys, eps, kind="hilbert", **kw)
    n = 30_001
    xy = uniform_points(n, lo, hi, 5)
    vals = np.random.default_rng(6).integers(-1000, 1000, size=n).astype(np.int64)
    want = orc.Approx(polys, eps).aggregate(xy, vals)
    c, s = run_agg(A, xy, vals)
    np.testing.assert_array_equal(c, want[0])
    np.testing.assert_array_equal(s, want[1])


@pytest.mark.parametrize("level", [10, 12, 16, 17, 21])
@pytest.mark.parametrize("corner", [0, 1])
def test_key_grids_larger_than_the_box(sba, orc, level, corner):
    polys = star_polygons(40, 12, 300.0, 6000.0, 60_000, 95)
    s = orc.cell_side(200)
    far = (1 << level) - 66_000 // s - 40 if corner else 60  # cells left of and below the box
    check(sba, orc, polys, 200, -5000, 66_000, key_grid=(level, -far, -far))


@pytest.mark.parametrize("wh", [(1, 1), (1, 5000), (5000, 1), (7, 4), (8, 4), (9, 5), (64, 64),
                                (65, 63), (3000, 40), (255, 1025)])
def test_shapes_of_the_box(sba, orc, wh):
    """Rectangles of one cell and more, in rows, over a box of wh cells."""
    s, (w, h) = orc.cell_side(20), wh
    r = np.random.default_rng(w * 10_000 + h)
    n = 12
    x, y = r.integers(1, w * s, size=n), r.integers(1, h * s, size=n)
    x[0] = y[0] = 1
    x1 = np.minimum(x + r.integers(1, max(2, w * s // 3), size=n), w * s - 1)
    y1 = np.minimum(y + r.integers(1, max(2, h * s // 3), size=n), h * s - 1)
    xy = np.stack((x, y, x1, y, x1, y1, x, y1), 1).astype(np.int32).reshape(-1)
    polys = Polygons(np.arange(n + 1, dtype=np.int32), 4 * np.arange(n + 1, dtype=np.int64), xy)
    check(sba, orc, polys, 20, -40, max(w, h) * s + 40)


def test_a_far_key_grid_takes_as_long(sba):
    """The same points over the same cells on a grid of 2^21 cells a side: 450
    times as long while its blocks were a fixed share of the grid."""
    polys = voronoi_partition(200, 4_000_000, (20, 60), seed=96, jitter_seed=97)
    xy = dev(uniform_points(50_000, 0, 4_000_000, 9))

    def best(key_grid):
        A = sba.Approx.from_polygons(polys, 1000, kind="hilbert", key_grid=key_grid)
        ms = []
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                A.aggregate(xy)
            b.record()
            b.synchronize()
            ms.append(a.elapsed_time(b))
        return min(ms)

    assert best((21, -2, -2)) < 2 * best((13, -2, -2))


@pytest.mark.parametrize("n", [20, 300, 3_000, 30_000])
def test_squares_of_every_size(sba, orc, n):
    """Directories whose squares of blocks have 16, 32 and 64 a side."""
    polys = voronoi_partition(n, 3_000_000, (1, 2), seed=n, jitter_seed=n + 1)
    eps = 3_000 if n < 3_000 else 800
    A = sba.Approx.from_polygons(polys, eps, kind="hilbert")
    xy = uniform_points(100_001, -5_000, 3_005_000, n)
    vals = np.random.default_rng(n).integers(-1000, 1000, 100_001).astype(np.int64)
    want = orc.Approx(polys, eps).aggregate(xy, vals)
    c, s = run_agg(A, xy, vals)
    np.testing.assert_array_equal(c, want[0])
    np.testing.assert_array_equal(s, want[1])
