"""Calls of few points against grids (csrc/probe.hip) around the size where the
probe changes its kernel, in every storage of the grid, with and without
values and sets.  Compared with the oracle; tolerance zero."""
import numpy as np
import pytest

from gen import star_polygons, uniform_points, voronoi_partition
from test_gpu_parity import run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu

LAST = 1 << 17


@pytest.mark.parametrize("what", ["stars", "partition", "many", "wide"])
@pytest.mark.parametrize("eps", [20, 400])
def test_few_points(sba, orc, what, eps):
    if what == "stars":
        polys = star_polygons(20, 12, 100.0, 3000.0, 20_000, 81)
    else:
        polys = voronoi_partition(4100 if what == "many" else 60, 20_000, (2, 5), seed=82,
                                  jitter_seed=83)
    O = orc.Approx(polys, eps)
    sba.lib().sba_debug_force_wide_grid(1 if what == "wide" else 0)
    try:
        A = sba.Approx.from_polygons(polys, eps)
    finally:
        sba.lib().sba_debug_force_wide_grid(0)
    for n in (1, 2, 3, 255, 511, 512, 513, 20_001, LAST - 1, LAST, LAST + 1):
        xy = uniform_points(n, -500, 20_500, n + eps)
        vals = np.random.default_rng(n).integers(-2**40, 2**40, size=n).astype(np.int64)
        want = O.aggregate(xy, vals)
        c, s = run_agg(A, xy, vals)
        np.testing.assert_array_equal(c, want[0])
        np.testing.assert_array_equal(s, want[1])
        c, _ = run_agg(A, xy)
        np.testing.assert_array_equal(c, want[0])
