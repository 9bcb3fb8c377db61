"""Values on both sides of the 24 bits that a bin of the Hilbert layout's probe
packs beside its count: the answers where the second lines have places of their
own, take hashed ones, have none left and where all lines are hashed, and the
time beside that of small values."""
import numpy as np
import pytest
import torch

from gen import uniform_points, voronoi_partition
from test_gpu_parity import dev, run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


def signed(n, rng):
    """Cents of both signs, and a few of every size."""
    v = rng.integers(-10_000, 10_001, size=n).astype(np.int64)
    v[::97] = rng.choice(np.array([1 << 24, -(1 << 24), (1 << 62) + 5, -(1 << 63), (1 << 63) - 1]),
                         size=v[::97].size)
    return v


# 16 polygons a line; one workgroup a compute unit has 1,035 places, two 461
@pytest.mark.parametrize("polygons", [40, 7_376, 7_377, 8_272, 8_288, 16_560, 16_561])
def test_signed_values(sba, orc, polygons):
    polys = voronoi_partition(polygons, 1_000_000, (1, 2), seed=81, jitter_seed=82)
    A = sba.Approx.from_polygons(polys, 1000, kind="hilbert")
    n = 400_003
    xy = uniform_points(n, -2000, 1_002_000, 7)
    vals = signed(n, np.random.default_rng(8))
    want = orc.Approx(polys, 1000).aggregate(xy, vals)  # both wrap modulo 2^64
    c, s = run_agg(A, xy, vals)
    np.testing.assert_array_equal(c, want[0])
    np.testing.assert_array_equal(s, want[1])
    c, s = A.aggregate_partitioned(dev(xy), dev(vals))
    np.testing.assert_array_equal(c.cpu().numpy().astype(np.uint64), want[0])
    np.testing.assert_array_equal(s.cpu().numpy(), want[1])


def test_signed_values_take_about_as_long(sba):
    """Points in spatial order over few polygons, where an addition to the
    outputs for each point made them 100 times as long; twice the additions to
    LDS may take up to three times here."""
    polys = voronoi_partition(200, 1_000_000, (4, 9), seed=83, jitter_seed=84)
    A = sba.Approx.from_polygons(polys, 1000, kind="hilbert")
    n = 4_000_000
    xy, _, _ = sba.bucket_points(dev(uniform_points(n, 0, 1_000_000, 9)), None, 0, 0, 1000, 1000)
    small = torch.randint(0, 10_000, (n,), device="cuda")
    large = torch.randint(-10_000, 10_000, (n,), device="cuda")

    def best(v):
        ms = []
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                A.aggregate(xy, v)
            b.record()
            b.synchronize()
            ms.append(a.elapsed_time(b))
        return min(ms)

    assert best(large) < 3 * best(small)
