"""The build's row sweep (csrc/rows.hip) at the sizes where it can go wrong:
rows of each workgroup class and past the last one, edges that a workgroup
cannot count in LDS, edges inside one cell, keys of large sets, boundary-cell
bitmaps wider than one LDS chunk.  Everything is compared with the oracle;
counts and sums are whole numbers, so the tolerance is zero."""
import numpy as np
import pytest

from gen import Polygons, polygons_from_rings, star_polygons
from test_gpu_parity import expected_sets, gpu_sets, run_agg, sba, window_of  # noqa: F401

pytestmark = pytest.mark.gpu


def slanted_strips(n, width=37, height=230, lean=90):
    """n leaning quadrilaterals side by side, each overlapping the next."""
    return polygons_from_rings([[[(k * width, 5), (k * width + width + 9, 3),
                                  (k * width + width + 9 + lean, height),
                                  (k * width + lean, height + 4)]] for k in range(n)])


def check(sba, orc, polys, eps, okw=None, n=40_001, seed=3, box=None, step=1, **kw):
    O = orc.Approx(polys, eps, **(okw or {}))
    x, y = polys.xy[0::2], polys.xy[1::2]
    lo = (int(x.min()) - 50, int(y.min()) - 50)
    hi = (int(x.max()) + 50, int(y.max()) + 50)
    rng = np.random.default_rng(seed)
    xy = np.empty(2 * n, np.int32)
    xy[0::2] = rng.integers(lo[0], hi[0], size=n)
    xy[1::2] = rng.integers(lo[1], hi[1], size=n)
    vals = rng.integers(1, 10_000, size=n).astype(np.int64)
    want = O.aggregate(xy, vals)
    A = sba.Approx.from_polygons(polys, eps, **kw)
    taken = sba.lib().sba_debug_last_build_paths()
    got = run_agg(A, xy, vals)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])
    info = A.info()
    i0, j0, nw, nh = window_of(polys, O.s, pad=1)
    js = range(0, nh, step)
    cells = [(i0 + i, j0 + j) for j in js for i in range(nw)]
    if len(cells) <= 400_000:
        ws = expected_sets(O, polys.n_polys, i0, j0, nw, nh)
        gs = gpu_sets(A, cells)
        bad = [c for c in cells if gs[c] != ws[c]]
        assert not bad, (len(bad), bad[:5])
    A.close()
    return taken, info


# the first and the last row hold three pairs per strip: workgroups of 1, 4, 8
# and 16 wavefronts take rows of up to 64, 256, 1024 and 4096 pairs, larger
# ones the global sorts
@pytest.mark.parametrize("n,swept", [(1, 2), (21, 2), (22, 2), (85, 2), (86, 2), (341, 2),
                                     (342, 2), (700, 2), (1365, 2), (1366, 0)])
@pytest.mark.parametrize("kind", ["grid", "hilbert"])
def test_rows_of_every_class(sba, orc, n, swept, kind):
    taken, _ = check(sba, orc, slanted_strips(n), 40, kind=kind, step=1 if n < 400 else 3)
    assert taken & 2 == swept and taken & 1


@pytest.mark.parametrize("kw,okw", [({"centre_sampled": True}, {"centre": True}),
                                    ({"boundary_only": True}, {"boundary_only": True})])
@pytest.mark.parametrize("kind", ["grid", "hilbert"])
@pytest.mark.parametrize("n", [40, 300])
def test_cell_rules_by_row(sba, orc, kw, okw, kind, n):
    check(sba, orc, slanted_strips(n), 40, okw=okw, kind=kind, **kw)


def test_sets_larger_than_three_beyond_the_small_keys(sba, orc):
    """Six squares on top of one another, shifted by their own widths' parts:
    fields of 4 bits leave 2^12 small set keys, and the rows hold more than
    2^12 segments of two or more polygons, many of them of four and more."""
    polys = polygons_from_rings([[[(70 * k, 11 * k), (70 * k + 900, 11 * k + 3),
                                   (70 * k + 905, 11 * k + 9000), (70 * k + 2, 11 * k + 9003)]]
                                 for k in range(6)])
    _, info = check(sba, orc, polys, 10, n=200_001, step=40)
    assert info["n_set_ids"] > 4 * info["n_sets"] > 4 * 4096
    check(sba, orc, polys, 10, n=100_001, step=80, kind="hilbert")


@pytest.mark.parametrize("off", [1, 2, 4, 5])
def test_same_sets_on_the_other_paths(sba, orc, off):
    polys = star_polygons(14, 11, 100.0, 900.0, 3000, 9)
    _, a = check(sba, orc, polys, 12, step=9)
    sba.lib().sba_debug_build_paths(off)
    try:
        _, b = check(sba, orc, polys, 12, step=9)
    finally:
        sba.lib().sba_debug_build_paths(0)
    for k in ("n_segments", "n_boundary", "n_sets", "n_set_ids", "bytes"):
        assert a[k] == b[k], k


@pytest.mark.parametrize("eps", [30, 900, 60_000])
def test_edges_inside_one_cell(sba, orc, eps):
    """Rings of 600 short edges: at the coarser bounds nearly every edge lies
    strictly inside one cell, at the last a whole ring does (it keeps the cell
    of its first edge)."""
    ang = np.linspace(0, 2 * np.pi, 600, endpoint=False)
    rings = []
    for k in range(9):
        r = 300 + 2500 * (k % 3) + 40 * np.sin(31 * ang)
        c = (7001 * (k % 3) + 900 * k, 6500 * (k // 3))
        rings.append([np.c_[c[0] + r * np.cos(ang), c[1] + r * np.sin(ang)].round().astype(np.int64)])
    polys = polygons_from_rings(rings)
    for kind in ("grid", "hilbert"):
        check(sba, orc, polys, eps, kind=kind, step=1 if eps > 100 else 50)


def test_edges_over_thousands_of_rows(sba, orc):
    """Edges of 20,000 rows (more than a workgroup counts in LDS) beside short
    ones, and one row-long horizontal edge."""
    polys = polygons_from_rings([[[(0, 0), (900, 10), (1000, 140_003), (40, 140_000)]],
                                 [[(500, 50), (560, 61), (551, 120), (505, 111)]],
                                 [[(-200, 70_000), (1500, 70_000), (1500, 70_090)]]])
    check(sba, orc, polys, 10, n=60_001, step=500)
    check(sba, orc, polys, 10, n=60_001, step=500, kind="hilbert")


def test_rows_wider_than_one_bitmap(sba, orc):
    """70,000 columns: the boundary-cell bitmap of a row takes two chunks."""
    polys = polygons_from_rings([[[(0, 0), (490_000, 300), (489_000, 700), (100, 400)]],
                                 [[(455_000, 100), (462_000, 250), (458_500, 800)]]])
    check(sba, orc, polys, 10, n=60_001, kind="hilbert", step=1000)


@pytest.mark.parametrize("win", [(400, 40, 2300, 150), (0, 0, 60, 60), (-500, 100, 90, 700)])
@pytest.mark.parametrize("kind", ["grid", "hilbert"])
def test_window_cuts_rows_and_columns(sba, orc, win, kind):
    polys = slanted_strips(80)
    eps = 20
    O = orc.Approx(polys, eps)
    rng = np.random.default_rng(8)
    n = 50_000
    xy = np.empty(2 * n, np.int32)
    xy[0::2] = rng.integers(win[0], win[2], size=n)
    xy[1::2] = rng.integers(win[1], win[3], size=n)
    vals = rng.integers(1, 99, size=n).astype(np.int64)
    want = O.aggregate(xy, vals)
    A = sba.Approx.from_polygons(polys, eps, window=win, kind=kind)
    assert sba.lib().sba_debug_last_build_paths() & 3 == 3
    got = run_agg(A, xy, vals)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])
    A.close()


def test_more_sets_than_one_workgroup_numbers(sba, orc):
    """A lattice of 8,100 overlapping squares: about 30,000 distinct sets,
    more than one workgroup sorts and fewer than the table holds."""
    m = 90
    polys = polygons_from_rings([[[(100 * i, 100 * j), (100 * i + 111, 100 * j + 1),
                                   (100 * i + 109, 100 * j + 112), (100 * i - 2, 100 * j + 108)]]
                                 for j in range(m) for i in range(m)])
    taken, info = check(sba, orc, polys, 12, n=200_001, step=97)
    assert info["n_sets"] > 8192 and taken & 3 == 3 and not taken & 4
    assert isinstance(polys, Polygons)


# a workgroup's edges with more than 4,096 pairs between them go to a launch of
# their own, 1,024 pairs a workgroup: one edge across all rows (too many to count
# in LDS), many across 600 of them (counted in LDS part by part), and both beside
# workgroups that stay in the first launch
@pytest.mark.parametrize("rows", [1023, 1025, 4095, 4097, 9000])
@pytest.mark.parametrize("kind", ["grid", "hilbert"])
def test_edges_across_many_rows(sba, orc, rows, kind):
    s = orc.cell_side(40)
    tall = [[[(10, 3), (90 * s, 7), (91 * s, rows * s - 9), (15, rows * s - 4)]]]
    taken, _ = check(sba, orc, polygons_from_rings(tall), 40, kind=kind, step=7)
    assert taken & 2


@pytest.mark.parametrize("kw,okw", [({}, {}), ({"centre_sampled": True}, {"centre": True}),
                                    ({"boundary_only": True}, {"boundary_only": True})])
def test_many_edges_across_many_rows(sba, orc, kw, okw):
    s, r = orc.cell_side(40), np.random.default_rng(12)
    rings = []
    for k in range(24):  # a comb of long teeth each, and small polygons between them
        x = 40 * s * k
        teeth = [(x + (q * 37 * s) // 20, (600 + r.integers(0, 9)) * s if q & 1 else r.integers(1, 5))
                 for q in range(20)]
        rings.append([teeth + [(x + 38 * s, 700 * s), (x, 701 * s)]])
        rings += [[[(x + 39 * s, y), (x + 39 * s + 30, y + 2), (x + 39 * s + 9, y + 40)]]
                  for y in range(50, 600 * s, 61 * s)]
    taken, _ = check(sba, orc, polygons_from_rings(rings), 40, okw=okw, step=5, **kw)
    assert taken & 2


def test_a_box_around_all_rows_costs_little(sba):
    """Its four edges' 100,000 pairs, by one workgroup, nearly doubled the build."""
    import time

    import torch

    from gen import voronoi_partition
    city = voronoi_partition(60, 4_000_000, (10, 40), seed=98, jitter_seed=99)
    box = Polygons(np.append(city.ring_off, city.ring_off[-1] + 1).astype(np.int32),
                   np.append(city.vert_off, city.vert_off[-1] + 4).astype(np.int64),
                   np.append(city.xy, [0, 0, 4_000_000, 0, 4_000_000, 4_000_000, 0, 4_000_000])
                   .astype(np.int32))

    def best(polys):
        t = [torch.from_numpy(a).cuda() for a in (polys.ring_off, polys.vert_off, polys.xy)]
        ms = []
        for _ in range(15):
            t0 = time.perf_counter()
            A = sba.Approx(*t, 100)
            ms.append(time.perf_counter() - t0)
            A.close()
        return min(ms)

    assert best(box) < 1.5 * best(city)
