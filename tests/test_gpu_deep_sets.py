"""Cells of more than three polygons: their sets' numbers and members are those of
the sorted list of all keys, whether one workgroup numbers them with the others
or the rows' counts do, and in rows of every class; intervals over more than 64
pieces; the deepest cell that is taken."""
import numpy as np
import pytest

from gen import Polygons, polygons_from_rings, uniform_points
from test_gpu_parity import run_agg, sba  # noqa: F401

pytestmark = pytest.mark.gpu

BOX = 100_000


def rects(n, w, seed):
    r = np.random.default_rng(seed)
    x, y = r.integers(0, BOX - w, size=(2, n))
    a, b = r.integers(w // 4, w, size=(2, n))
    xy = np.stack((x, y, x + a, y + 1, x + a + 1, y + b, x, y + b), 1).astype(np.int32).reshape(-1)
    return Polygons(np.arange(n + 1, dtype=np.int32), 4 * np.arange(n + 1, dtype=np.int64), xy)


def both(sba, polys, eps, **kw):
    out = []
    for off in (0, 4):
        sba.lib().sba_debug_build_paths(off)
        try:
            out.append(sba.Approx.from_polygons(polys, eps, **kw))
            assert sba.lib().sba_debug_last_build_paths() & 2
        finally:
            sba.lib().sba_debug_build_paths(0)
    return out


# layers of 2 to 25 polygons; from some hundred to some hundred thousand sets of
# more than three; rows of a wavefront, of 4, 8 and 16
@pytest.mark.parametrize("n,w,eps", [(40, 30_000, 1500), (40, 30_000, 300), (40, 30_000, 40),
                                     (300, 12_000, 400), (300, 12_000, 60), (2500, 6000, 300),
                                     (6000, 3500, 150)])
def test_numbers_and_members(sba, orc, n, w, eps):
    polys = rects(n, w, n + eps)
    A, B = both(sba, polys, eps)
    for a, b in zip(A.sets(), B.sets()):
        np.testing.assert_array_equal(a, b)
    s = orc.cell_side(eps)
    ij = np.random.default_rng(4).integers(-2, BOX // s + 2, size=(40_000, 2)).astype(np.int64)
    np.testing.assert_array_equal(A.lookup(ij).cpu().numpy(), B.lookup(ij).cpu().numpy())
    A, B = both(sba, polys, eps, kind="hilbert")
    for a, b in zip(A.runs(), B.runs()):
        np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
    xy = uniform_points(60_001, -500, BOX + 500, 5)
    vals = np.random.default_rng(6).integers(-1000, 1000, size=60_001).astype(np.int64)
    want = orc.Approx(polys, eps).aggregate(xy, vals)
    got = run_agg(A, xy, vals)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])


@pytest.mark.parametrize("pieces", [63, 64, 65, 700])
def test_intervals_over_many_pieces(sba, orc, pieces):
    """Five boxes over a row of small polygons: six in each, five between them."""
    wide = [[[(-10 * k, -5 * k), (40 * pieces + 10 * k, -5 * k),
              (40 * pieces + 10 * k, 500 + 5 * k), (-10 * k, 500 + 5 * k)]] for k in range(5)]
    small = [[[(40 * q + 5, 20), (40 * q + 24, 25), (40 * q + 15, 480)]] for q in range(pieces // 2)]
    polys = polygons_from_rings(wide + small)
    A, B = both(sba, polys, 10)
    for a, b in zip(A.sets(), B.sets()):
        np.testing.assert_array_equal(a, b)
    xy = uniform_points(50_000, -100, 40 * pieces + 100, 7)
    xy[1::2] = np.random.default_rng(8).integers(-60, 560, size=50_000)
    np.testing.assert_array_equal(run_agg(A, xy)[0], orc.Approx(polys, 10).aggregate(xy, None)[0])


@pytest.mark.parametrize("depth", [31, 32, 33])
def test_deepest_cell(sba, orc, depth):
    polys = polygons_from_rings([[[(3 * k, 0), (900 + 3 * k, 0), (900 + 3 * k, 90), (3 * k, 90)]]
                                 for k in range(depth)])
    if depth > 32:
        with pytest.raises(sba.SbaError):
            sba.Approx.from_polygons(polys, 30)
        return
    A, B = both(sba, polys, 30)
    for a, b in zip(A.sets(), B.sets()):
        np.testing.assert_array_equal(a, b)
    xy = uniform_points(20_000, -20, 1100, 9)
    np.testing.assert_array_equal(run_agg(A, xy)[0], orc.Approx(polys, 30).aggregate(xy, None)[0])
