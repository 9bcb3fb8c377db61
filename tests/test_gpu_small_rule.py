"""Grid handles of thousands of polygons whose small directory the staged probe
takes over from half as many points, and others from three quarters: both sides of
these sizes and of the general one, compared with the oracle."""
import numpy as np
import pytest

from gen import uniform_points, voronoi_partition
from test_gpu_parity import run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps,kernel", [(10_000, "k_probe_grid16<true, 0, 0,"),  # sets in memory
                                        (1_000, "k_probe_grid16<true, 1, 0,")])  # sub-directory
def test_small_directory(sba, orc, eps, kernel):
    polys = voronoi_partition(4_000, 4_000_000, (1, 2), seed=71, jitter_seed=72)
    A = sba.Approx.from_polygons(polys, eps)
    O = orc.Approx(polys, eps)
    assert A.probe_kernel(True).startswith(kernel)
    rng = np.random.default_rng(5)
    for n in (0, 1, 1 << 16, (1 << 16) + 1, 3 << 15, (3 << 15) + 1, 1 << 17, (1 << 17) + 1):
        xy = uniform_points(n, -2000, 4_002_000, n)
        vals = rng.integers(-10**9, 10**9, size=n).astype(np.int64)
        want = O.aggregate(xy, vals)
        c, s = run_agg(A, xy, vals)
        np.testing.assert_array_equal(c, want[0])
        np.testing.assert_array_equal(s, want[1])
        c, _ = run_agg(A, xy)
        np.testing.assert_array_equal(c, want[0])
