"""The row sweep's sets of more than three polygons (csrc/rows.hip), whose
members a wavefront finds together, and the sort of its pairs: many such pieces
in a row, rows of every workgroup class, sets up to the most a cell takes, the
first and the last of a row's intervals among the members.  Compared with the
oracle cell by cell; tolerance zero."""
import numpy as np
import pytest

from gen import polygons_from_rings
from test_gpu_parity import sba  # noqa: F401
from test_gpu_rows import check

pytestmark = pytest.mark.gpu


def fan(n, depth, width=40, height=60):
    """n leaning bars, `depth` of them over every place between."""
    return polygons_from_rings([[[(k * width, 3 + k % 5),
                                  (k * width + width * depth - 7, 2 + k % 3),
                                  (k * width + width * depth + 5, height + k % 7),
                                  (k * width + 9, height + 2)]] for k in range(n)])


@pytest.mark.parametrize("n", [5, 33, 66, 130, 260, 300, 520, 1100])
@pytest.mark.parametrize("depth", [4, 7, 28])
def test_many_large_sets(sba, orc, n, depth):
    taken, info = check(sba, orc, fan(n, depth), 6, step=5 if n > 100 else 1, n=20_001)
    assert taken & 1
    assert info["n_sets"] > 0 and info["n_set_ids"] >= 4
