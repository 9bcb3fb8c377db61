"""The grid build's numbering of mixed squares (csrc/build.hip) at the sizes
where it can go wrong: fewer squares than a workgroup's 2,048 and one more,
counts that are no multiple of four or eight, more squares than one launch
numbers (65,536), more mixed tiles than 16 bits number (the 32-bit format),
none at all; and few and many rows around the row scan's one chunk of 8,191.
Compared with the oracle; tolerance zero."""
import numpy as np
import pytest

from gen import polygons_from_rings, star_polygons
from test_gpu_parity import run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


def compare(sba, orc, polys, eps, hi, n=60_001, **kw):
    rng = np.random.default_rng(2)
    xy = np.empty(2 * n, np.int32)
    xy[0::2] = rng.integers(-20, hi[0] + 20, size=n)
    xy[1::2] = rng.integers(-20, hi[1] + 20, size=n)
    vals = rng.integers(-1000, 10_000, size=n).astype(np.int64)
    want = orc.Approx(polys, eps).aggregate(xy, vals)
    A = sba.Approx.from_polygons(polys, eps, **kw)
    got = run_agg(A, xy, vals)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])
    return A.info()


# cells of one unit (eps 2): the grid's size is the stars' box
@pytest.mark.parametrize("w,h", [(7, 5), (90, 90), (181, 181), (182, 180), (333, 101), (1023, 1025),
                                 (1100, 1024)])
@pytest.mark.parametrize("kw", [dict(tile_log2=2), dict(tile_log2=2, sub_log2=1),
                                dict(tile_log2=3, sub_log2=1), dict()])
def test_numbers_of_squares(sba, orc, w, h, kw):
    polys = star_polygons(12, 9, 2.0, max(w, h) / 3, max(w, h), 95)
    polys.xy[0::2] = np.clip(polys.xy[0::2], 0, w)
    polys.xy[1::2] = np.clip(polys.xy[1::2], 0, h)
    compare(sba, orc, polys, 2, (w, h), **kw)


def test_no_mixed_tile(sba, orc):
    sq = [[np.array([[0, 0], [3, 0], [3, 3], [0, 3]])]]
    compare(sba, orc, polygons_from_rings(sq), 300, (4, 4))


def test_more_mixed_tiles_than_sixteen_bits(sba, orc):
    """A chequerboard of triangles: nearly every tile of 4 x 4 cells is mixed."""
    rings = [[[(x, y), (x + 5, y + 1), (x + 2, y + 6)]] for x in range(0, 900, 8)
             for y in range(0, 900, 8)]
    info = compare(sba, orc, polygons_from_rings(rings), 2, (900, 900), tile_log2=2)
    assert info["n_blocks"] >= 0x8000 and not info["compact"]


@pytest.mark.parametrize("rows", [8188, 8189, 8190, 8191, 8192, 8193])
@pytest.mark.parametrize("kind", ["grid", "hilbert"])
def test_rows_of_one_chunk(sba, orc, rows, kind):
    tri = [[[(0, 0), (37, rows // 2), (3, rows)]], [[(20, 5), (90, rows - 9), (60, rows // 3)]]]
    info = compare(sba, orc, polygons_from_rings(tri), 2, (95, rows), kind=kind)
    assert info["gh"] >= rows
