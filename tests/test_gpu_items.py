"""The probe over LDS lines of polygon bins and the block directory of the
Hilbert layout, at the sizes where they can go wrong: more lines than places,
values that leave a bin's 24 bits, sets, chunk edges, a bin's largest count,
directories of a few blocks, keys of more than 32 bits, boxes at the ends of
the coordinate range.  Compared with the oracle; whole numbers, tolerance
zero."""
import numpy as np
import pytest
import torch

from gen import Polygons, star_polygons, uniform_points, voronoi_partition
from test_gpu_parity import dev, run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def many(orc):
    """More polygons than one workgroup has lines for, in every workgroup size."""
    polys = voronoi_partition(20_000, 1_000_000, (1, 3), seed=61, jitter_seed=62)
    return polys, orc.Approx(polys, 700)


HANDLES = {"grid": dict(), "binary": dict(kind="hilbert"),
           "learned": dict(kind="hilbert", search="learned")}


def draw_values(kind, n, rng):
    if kind == "small":
        return rng.integers(0, 1 << 24, size=n).astype(np.int64)
    # on both sides of a bin's range
    return rng.choice(np.array([0, 1, (1 << 24) - 1, 1 << 24, -1, -(1 << 40), 1 << 40]), size=n)


@pytest.mark.parametrize("name", list(HANDLES))
@pytest.mark.parametrize("values", ["small", "wide"])
def test_more_lines_than_places(sba, many, name, values):
    polys, O = many
    A = sba.Approx.from_polygons(polys, 700, **HANDLES[name])
    rng = np.random.default_rng(5)
    for n in (1, 2, 3, 8191, 8192, 8193, 2_100_003):
        xy = uniform_points(n, -2000, 1_002_000, n)
        vals = draw_values(values, n, rng)
        want = O.aggregate(xy, vals)
        c, s = run_agg(A, xy, vals)
        np.testing.assert_array_equal(c, want[0])
        np.testing.assert_array_equal(s, want[1])
        c, _ = run_agg(A, xy)
        np.testing.assert_array_equal(c, want[0])
    for m in ((1 << 17), (1 << 17) + 1, 2_100_003):  # the partition's edges
        c, s = A.aggregate_partitioned(dev(xy[:2 * m]), dev(vals[:m]))
        want = O.aggregate(xy[:2 * m], vals[:m])
        np.testing.assert_array_equal(c.cpu().numpy().astype(np.uint64), want[0])
        np.testing.assert_array_equal(s.cpu().numpy(), want[1])


def test_bins_at_their_largest_count(sba, orc):
    """Every point in one cell, with the largest value a bin takes: each
    workgroup has more of them than one bin can count before it goes out."""
    polys = voronoi_partition(4200, 1_000_000, (1, 2), seed=63, jitter_seed=64)
    n = (1 << 28) + (1 << 20) + 7
    v = (1 << 24) - 1
    txy = torch.full((2 * n,), 500_123, dtype=torch.int32, device="cuda")
    tv = torch.full((n,), v, dtype=torch.int64, device="cuda")
    for eps in (2000, 100):  # a cell of two polygons, a cell of one
        one = orc.Approx(polys, eps).aggregate(np.array([500_123, 500_123], np.int32),
                                               np.array([v], np.int64))
        for kw in (dict(), dict(kind="hilbert")):
            A = sba.Approx.from_polygons(polys, eps, **kw)
            c, s = A.aggregate(txy, tv)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(c.cpu().numpy().astype(np.uint64), one[0] * n)
            np.testing.assert_array_equal(s.cpu().numpy(), one[1] * n)


# levels of 1 and more, keys of 32 bits (level 16) and of more, overlapping
# polygons (sets)
@pytest.mark.parametrize("eps", [2000, 400, 150, 60, 12])
@pytest.mark.parametrize("span", [1500, 60_000, 1_500_000])
@pytest.mark.parametrize("search", ["binary", "learned"])
def test_directory_levels(sba, orc, eps, span, search):
    polys = star_polygons(30, 12, span / 60, span / 5, span, 71)
    if eps * 40_000 < span:
        eps = max(eps, 17)
    try:
        A = sba.Approx.from_polygons(polys, eps, kind="hilbert", search=search)
    except sba.SbaError:
        assert search == "learned"  # keys of more than 32 bits have no learned index
        return
    n = 60_001
    xy = uniform_points(n, -span // 3, span + span // 3, 9)
    vals = draw_values("wide", n, np.random.default_rng(3))
    want = orc.Approx(polys, eps).aggregate(xy, vals)
    for srch in ("binary", search):
        c, s = run_agg(A, xy, vals, search=srch)
        np.testing.assert_array_equal(c, want[0])
        np.testing.assert_array_equal(s, want[1])


@pytest.mark.parametrize("at", [(1 - 2**30, 1 - 2**30), (2**30 - 3001, 2**30 - 3001),
                                (-1500, -1500)])
@pytest.mark.parametrize("eps", [7, 500])
def test_directory_at_the_ends_of_the_range(sba, orc, at, eps):
    base = star_polygons(20, 9, 40.0, 500.0, 3000, 73)
    xy0 = np.clip(base.xy, 0, 3000).astype(np.int64)
    xy0[0::2] += at[0]
    xy0[1::2] += at[1]
    polys = Polygons(base.ring_off, base.vert_off, xy0.astype(np.int32))
    rng = np.random.default_rng(4)
    n = 50_003
    pts = rng.integers(-200, 3200, size=(n, 2)) + np.array(at, np.int64)
    xy = pts.astype(np.int32).reshape(-1)
    xy[:8] = [-2**31, -2**31, 2**31 - 1, 2**31 - 1, -2**31, 2**31 - 1, at[0], at[1]]
    vals = rng.integers(-50, 5000, size=n).astype(np.int64)
    want = orc.Approx(polys, eps).aggregate(xy, vals)
    for kw in HANDLES.values():
        c, s = run_agg(sba.Approx.from_polygons(polys, eps, **kw), xy, vals)
        np.testing.assert_array_equal(c, want[0])
        np.testing.assert_array_equal(s, want[1])
