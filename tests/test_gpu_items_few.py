"""Few points over Hilbert handles and grids of many polygons: the sizes between
which the probe takes more of them a lane, cells of polygon sets (which wait in
the wavefronts' queues) among them.  Compared with the oracle."""
import numpy as np
import pytest

from gen import Polygons, uniform_points, voronoi_partition
from test_gpu_parity import run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


def layered(n):
    """Two partitions of one box: every cell belongs to two polygons or more."""
    a = voronoi_partition(n, 1_000_000, (1, 2), seed=91, jitter_seed=92)
    b = voronoi_partition(n, 1_000_000, (1, 2), seed=93, jitter_seed=94)
    return Polygons(np.concatenate((a.ring_off, b.ring_off[1:] + a.ring_off[-1])),
                    np.concatenate((a.vert_off, b.vert_off[1:] + a.vert_off[-1])),
                    np.concatenate((a.xy, b.xy)))


@pytest.fixture(scope="module")
def sets(orc):
    polys = layered(2_200)  # more than a grid probe has a bin for
    return polys, orc.Approx(polys, 1500)


@pytest.mark.parametrize("kw", [dict(), dict(kind="hilbert"),
                                dict(kind="hilbert", search="learned")])
def test_edges_of_the_split(sba, sets, kw):
    polys, O = sets
    A = sba.Approx.from_polygons(polys, 1500, **kw)
    rng = np.random.default_rng(3)
    for n in (2047, 2048, 2049, 4097, 1 << 18, (1 << 18) + 1, 1 << 19, (1 << 19) + 1):
        xy = uniform_points(n, -2000, 1_002_000, n)
        vals = rng.integers(-10**9, 10**9, size=n).astype(np.int64)
        want = O.aggregate(xy, vals)
        c, s = run_agg(A, xy, vals)
        np.testing.assert_array_equal(c, want[0])
        np.testing.assert_array_equal(s, want[1])
        c, _ = run_agg(A, xy)
        np.testing.assert_array_equal(c, want[0])
