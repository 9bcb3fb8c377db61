"""The point index's build (csrc/pindex.hip) at the sizes where it can go
wrong: one key, tiles of 4,096 and chunks of 1,024 distinct keys, the sort's
change of tile at 2^22, keys of more than 32 bits, many equal keys, more knots
a chunk than one pass keeps, points at an 8-byte address.  Compared with the
oracle; tolerance zero."""
import numpy as np
import pytest
import torch

from gen import star_polygons, uniform_points
from test_gpu_pindex import check_index, dev, pindex_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 5, 1023, 1024, 1025, 4095, 4096, 4097, 8193, (4 << 20) - 1,
                               4 << 20, (4 << 20) + 8193])
@pytest.mark.parametrize("eps,span", [(4, 3000), (300, 3000), (3, 400_000)])
def test_sizes(sba, orc, n, eps, span):
    if span == 400_000 and n > (4 << 20):
        eps = 9
    polys = star_polygons(10, 9, span / 100, span / 8, span, 91)
    xy = uniform_points(n, -span // 20, span + span // 20, n)
    vals = np.random.default_rng(n).integers(-2**40, 2**40, size=n).astype(np.int64)
    ix, _ = check_index(sba, orc, polys, xy, vals, eps, spline_err=1 if n < 10_000 else 32)
    cells = np.unique(np.floor_divide(xy.reshape(-1, 2), ix.info()["s"]), axis=0)
    assert ix.info()["n_distinct"] == len(cells)


def test_points_at_an_eight_byte_address(sba, orc):
    n = 70_001
    polys = star_polygons(10, 9, 30.0, 400.0, 3000, 92)
    xy = uniform_points(n + 1, -100, 3100, 5)
    vals = np.arange(n + 1, dtype=np.int64)
    txy, tv = dev(xy)[2:], dev(vals)[1:]
    assert txy.data_ptr() % 16 == 8
    want = orc.Approx(polys, 6).aggregate(xy[2:], vals[1:])
    ix = sba.PointIndex(txy, tv, 6)
    A = sba.Approx.from_polygons(polys, 6, kind="hilbert", key_grid=ix)
    c, s = pindex_agg(ix, A, "learned")
    np.testing.assert_array_equal(c, want[0])
    np.testing.assert_array_equal(s, want[1])
