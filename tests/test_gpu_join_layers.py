"""Joins of polygons in layers (cells of many polygons on both sides) and of few
runs: every pair summed in LDS, tables that are too small at first, tiles of every
size.  Compared with the oracle's pairs."""
import numpy as np
import pytest

from gen import Polygons
from test_gpu_join import check, sba  # noqa: F401

pytestmark = pytest.mark.gpu

BOX = 60_000


def rects(n, w, seed):
    r = np.random.default_rng(seed)
    x, y = r.integers(0, BOX - w, size=(2, n))
    a, b = r.integers(w // 4, w, size=(2, n))
    xy = np.stack((x, y, x + a, y + 1, x + a + 1, y + b, x, y + b), 1).astype(np.int32).reshape(-1)
    return Polygons(np.arange(n + 1, dtype=np.int32), 4 * np.arange(n + 1, dtype=np.int64), xy)


# polygons of both sides, their width, eps: one layer and many, few runs and
# hundreds of thousands; 900 and 2,500 a side meet in more pairs than the first
# table takes, 40 in few enough for a slot each
@pytest.mark.parametrize("n,w,eps", [(2, 30_000, 2000), (40, 15_000, 3000), (40, 15_000, 100),
                                     (300, 2000, 400), (900, 8000, 900), (900, 8000, 200),
                                     (2500, 4500, 700), (2500, 4500, 150)])
def test_layers(sba, orc, n, w, eps):
    P, Q = rects(n, w, n), rects(n, w, n + 1)
    assert check(sba, orc, P, Q, eps)[0].size > 0
    check(sba, orc, Q, P, eps)
