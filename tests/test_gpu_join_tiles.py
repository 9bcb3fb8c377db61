"""The join over tiles of merged runs (csrc/join.hip) at the sizes where it can
go wrong: lists of one run, a tile and its neighbours of one list only, equal
first keys everywhere, keys of more than 32 bits, more pairs than the first
table holds, sets on both sides.  Compared with the oracle; tolerance zero."""
import numpy as np
import pytest

from gen import polygons_from_rings, star_polygons, voronoi_partition
from test_gpu_join import check, gpu_join, sba  # noqa: F401

pytestmark = pytest.mark.gpu


def square(x0, y0, x1, y1):
    return [np.array([[x0, y0], [x1, y0], [x1, y1], [x0, y1]])]


@pytest.mark.parametrize("eps", [2, 30, 1000])
def test_few_runs_against_many(sba, orc, eps):
    one = polygons_from_rings([square(-5000, -5000, 9000, 9000)])
    many = voronoi_partition(60, 4000, (2, 6), seed=41, jitter_seed=42)
    check(sba, orc, one, one, eps)
    check(sba, orc, one, many, eps)
    check(sba, orc, many, one, eps)
    check(sba, orc, many, many, eps)


def test_wide_keys(sba, orc):
    a = star_polygons(8, 9, 500.0, 4000.0, 700_000, 43)
    b = star_polygons(8, 7, 500.0, 4000.0, 700_000, 44)
    want = check(sba, orc, polygons_from_rings([[r] for r in rings(a)] +
                                               [square(0, 0, 3000, 3000)]),
                 polygons_from_rings([[r] for r in rings(b)] +
                                     [square(1000, 1000, 4000, 4000)]), 12)
    assert want[0].size > 0


def rings(polys):
    return [polys.xy.reshape(-1, 2)[a:b] for a, b in zip(polys.vert_off[:-1], polys.vert_off[1:])]


def test_more_pairs_than_the_first_table(sba, orc):
    """Staircases of squares: each of 600 meets 600 of the other side (at most
    32 in one cell)."""
    def bars(horizontal):
        out = []
        for k in range(600):
            lo, hi = 40 * k, 40 * k + 70
            out.append(square(0, lo, 24_100, hi) if horizontal else square(lo, 0, hi, 24_100))
        return polygons_from_rings(out)

    want = check(sba, orc, bars(True), bars(False), 30)
    assert want[0].size > 8 * 2048 * 8
