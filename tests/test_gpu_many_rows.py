"""Builds of many rows of cells with few edges in each: the scan of the rows by
several workgroups, rows of few pairs and cells by a lane, the others among them by
its wavefront.  Runs and codes are those of the global sorts."""
import numpy as np
import pytest

from gen import polygons_from_rings, uniform_points
from test_gpu_parity import run_agg, sba  # noqa: F401
from test_gpu_row_cells import fans, same

pytestmark = pytest.mark.gpu

SIDE = 7  # of a cell at eps 10


def turned(polys):
    return type(polys)(polys.ring_off, polys.vert_off,
                       np.ascontiguousarray(polys.xy.reshape(-1, 2)[:, ::-1]).reshape(polys.xy.shape))


# rows around multiples of 8,192 from which the scan has a workgroup each
@pytest.mark.parametrize("rows", [8_191, 24_574, 24_575, 24_576, 24_577, 32_767, 32_768, 40_961])
def test_scan_in_parts(sba, orc, rows):
    height = rows * SIDE - 3
    r = np.random.default_rng(rows)
    rings = [[[(0, 0), (5, 0), (900, height), (880, height)]]]
    for _ in range(30):  # the rows' counts differ
        x, y = int(r.integers(0, 800)), int(r.integers(0, height - 9_000))
        rings.append([[(x, y), (x + 90, y + 200), (x + 40, y + int(r.integers(300, 9_000)))]])
    polys = polygons_from_rings(rings)
    A = same(sba, polys, 10)
    G = sba.Approx.from_polygons(polys, 10)
    xy = uniform_points(40_001, -50, 950, 3)
    xy[1::2] = r.integers(-50, height + 50, size=40_001)
    want = orc.Approx(polys, 10).aggregate(xy, None)
    np.testing.assert_array_equal(run_agg(A, xy)[0], want[0])
    np.testing.assert_array_equal(run_agg(G, xy)[0], want[0])


# n quadrilaterals: up to 2 n edges a row, above and below the four of a lane's row
@pytest.mark.parametrize("rows", [(1 << 17) - 1, 1 << 17, (1 << 17) + 300])
@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("kw", [dict(), dict(centre_sampled=True), dict(boundary_only=True)])
def test_rows_by_a_lane(sba, orc, rows, n, kw):
    polys = turned(fans(n, rows * SIDE, 1_500, rows + n))
    A = same(sba, polys, 10, **kw)
    xy = uniform_points(40_001, -50, 1_550, 3)
    xy[1::2] = np.random.default_rng(4).integers(-50, rows * SIDE + 50, size=40_001)
    okw = {"centre": True} if "centre_sampled" in kw else kw
    want = orc.Approx(polys, 10, **okw).aggregate(xy, None)
    np.testing.assert_array_equal(run_agg(A, xy)[0], want[0])


# flat edges (rows of many cells) and steep ones, more pairs in some rows than a
# wavefront takes; clip windows, whose border cells belong to them
@pytest.mark.parametrize("win", [None, (3, 3, 3_500, 140_000 * SIDE - 2), (1_000, -50, 1_001, 10**6),
                                 (2_000, 700, 2_600, 135_000 * SIDE)])
def test_mixed_rows(sba, win):
    h = 140_000 * SIDE
    rings = [[[(0, 0), (4_000, 3), (3_990, h), (10, h - 20)]],
             [[(5, 300), (3_900, 310), (3_900, 500), (5, 480)]]]
    for k in range(60):  # 120 pairs in each of a few rows
        rings.append([[(40 + 60 * k, 9_000), (70 + 60 * k, 9_000), (70 + 60 * k, 9_100),
                       (40 + 60 * k, 9_100)]])
    polys = polygons_from_rings(rings)
    same(sba, polys, 10, **({"window": win} if win else {}))
