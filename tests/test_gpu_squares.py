"""The tiled grid's squares (csrc/build.hip) for tiles of 64 cells and more, in
every shape the workgroups take: several tiles to a workgroup and several
workgroup heights to a tile, few and many sub-tiles, grids that end inside a
tile, rows with more segments than the staged window.  Compared with the
oracle, cell by cell and by aggregates; tolerance zero."""
import numpy as np
import pytest

from gen import star_polygons
from test_gpu_parity import run_agg, sba  # noqa: F401
from test_gpu_rows import check, slanted_strips

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tl,sl", [(6, 6), (6, 4), (6, 3), (6, 2), (6, 1), (7, 4), (8, 6), (8, 4),
                                   (8, 3), (9, 6), (10, 7), (10, 5)])
@pytest.mark.parametrize("eps", [3, 9])
def test_tiles_and_sub_tiles(sba, orc, tl, sl, eps):
    check(sba, orc, star_polygons(14, 9, 20.0, 900.0, 2600, 93), eps, step=7, tile_log2=tl,
          sub_log2=sl)


@pytest.mark.parametrize("tl,sl", [(6, 3), (8, 4)])
def test_rows_of_many_segments(sba, orc, tl, sl):
    check(sba, orc, slanted_strips(300), 3, step=11, tile_log2=tl, sub_log2=sl)


@pytest.mark.parametrize("width,height", [(15, 300), (2100, 40), (1025, 257), (4097, 16)])
def test_ragged_grids(sba, orc, width, height):
    polys = star_polygons(9, 7, 4.0, min(width, height) / 2.5, max(width, height), 94)
    polys.xy[0::2] = np.clip(polys.xy[0::2], 0, width)
    polys.xy[1::2] = np.clip(polys.xy[1::2], 0, height)
    xy = np.random.default_rng(1).integers(-20, max(width, height) + 20, size=80_002).astype(np.int32)
    vals = np.arange(40_001, dtype=np.int64)
    for tl, sl in ((6, 3), (8, 5), (9, 4)):
        want = orc.Approx(polys, 2).aggregate(xy, vals)
        got = run_agg(sba.Approx.from_polygons(polys, 2, tile_log2=tl, sub_log2=sl), xy, vals)
        np.testing.assert_array_equal(got[0], want[0])
        np.testing.assert_array_equal(got[1], want[1])
