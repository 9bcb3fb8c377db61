"""Polygons smaller than a cell, many in one row of cells: each leaves one pair and
two toggles, more toggles than the row's workgroup holds, which it finds in the
sweep; the build then takes the global sorts.  Compared with the oracle."""
import numpy as np
import pytest

from gen import polygons_from_rings
from test_gpu_parity import run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


def footprints(per_row, rows, pitch, side, seed):
    r = np.random.default_rng(seed)
    x = np.arange(per_row) * pitch + r.integers(0, pitch - side, (rows, per_row))
    y = np.broadcast_to(np.arange(rows)[:, None] * pitch + 1, x.shape)
    return polygons_from_rings(
        [[[(a, b), (a + side, b), (a + side, b + side), (a, b + side)]]
         for a, b in zip(x.ravel(), y.ravel())])


# 257 to 1,024 pairs hold 1,408 toggles, up to 4,096 pairs 4,096
@pytest.mark.parametrize("per_row,held", [(256, True), (690, True), (750, False), (2_040, True),
                                          (2_100, False)])
@pytest.mark.parametrize("kind", ["grid", "hilbert"])
def test_many_in_a_row(sba, orc, per_row, held, kind):
    # cells of 70 units: a footprint of 12 meets one or two of them
    polys = footprints(per_row, 3, 70, 12, per_row)
    A = sba.Approx.from_polygons(polys, 100, kind=kind)
    path = sba.lib().sba_debug_last_build_paths() & 2
    rng = np.random.default_rng(7)
    xy = np.stack((rng.integers(-50, 70 * per_row + 50, 200_001),
                   rng.integers(-50, 300, 200_001)), 1).astype(np.int32).ravel()
    vals = rng.integers(-1000, 1000, 200_001).astype(np.int64)
    want = orc.Approx(polys, 100).aggregate(xy, vals)
    c, s = run_agg(A, xy, vals)
    np.testing.assert_array_equal(c, want[0])
    np.testing.assert_array_equal(s, want[1])
    assert path == (2 if held else 0)
