"""The inverse of the Hilbert index, all levels at once (host copy): against
the index itself at every level, at the ends of the curve and at keys whose
levels all turn the frame the same way.  Exact."""
import numpy as np
import pytest

import paper_2010_12548_amd as sba


@pytest.mark.parametrize("L", list(range(1, 22)))
def test_inverse_of_the_index(L):
    rng = np.random.default_rng(L)
    top = 1 << (2 * L)
    keys = [0, 1, top - 1, top // 2, top // 2 - 1, top // 3, (top - 1) // 3 * 2]
    keys += [int(rng.integers(0, top)) for _ in range(200)]
    for d in keys:
        i, j = sba.hilbert_cell(L, d)
        assert 0 <= i < 1 << L and 0 <= j < 1 << L
        assert sba.hilbert(L, i, j) == d
