"""Batched lookups over Hilbert handles where some lanes' points all lie in mixed
blocks of the directory, some none and others between.  Compared with the oracle."""
import numpy as np
import pytest
import torch

from gen import star_polygons, uniform_points, voronoi_partition
from test_gpu_parity import dev, sba  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["partition", "stars"])
@pytest.mark.parametrize("search", ["binary", "learned"])
def test_lanes_of_any_mix(sba, orc, what, search):
    if what == "partition":
        polys = voronoi_partition(700, 100_000, (2, 5), seed=41, jitter_seed=42)
    else:
        polys = star_polygons(12, 30, 2_000.0, 40_000.0, 100_000, 43)
    A = sba.Approx.from_polygons(polys, 150, kind="hilbert", search=search)
    O = orc.Approx(polys, 150)
    rng = np.random.default_rng(8)
    for n in (1, 513, 50_001):
        xy = uniform_points(n, -2000, 102_000, n).reshape(-1, 2)
        # the first third along the polygons' own vertices, the second outside
        v = polys.xy.reshape(-1, 2)
        xy[:n // 3] = v[rng.integers(0, len(v), n // 3)] + rng.integers(-200, 200, (n // 3, 2))
        xy[n // 3:2 * n // 3] += 200_000
        for order in (xy, xy[rng.permutation(n)]):
            flat = np.ascontiguousarray(order).ravel()
            vals = rng.integers(-10**9, 10**9, size=n).astype(np.int64)
            want = O.aggregate(flat, vals)
            t = sba.Task(A, dev(flat), dev(vals), search=search)
            u = sba.Task(A, dev(flat), search=search, lo=n // 2)
            sba.aggregate_batch([t, u])
            torch.cuda.synchronize()
            np.testing.assert_array_equal(t.counts.cpu().numpy().astype(np.uint64), want[0])
            np.testing.assert_array_equal(t.sums.cpu().numpy(), want[1])
            half = O.aggregate(flat[2 * (n // 2):], None)
            np.testing.assert_array_equal(u.counts.cpu().numpy().astype(np.uint64), half[0])
