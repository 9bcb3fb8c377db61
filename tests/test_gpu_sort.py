"""The radix sort's large tiles (csrc/prims.hip, 2^22 keys and more) at the
sizes where they can go wrong: the first size they take, the last key of a
tile and one more, several tiles to a counting workgroup, all keys in one
digit.  Stable order by the low bits, exactly."""
import numpy as np
import pytest

from test_gpu_prims import check_sort, sba  # noqa: F401

pytestmark = pytest.mark.gpu

FIRST, TILE = 4 << 20, 8192


@pytest.mark.parametrize("n", [FIRST - 1, FIRST, FIRST + 1, FIRST + TILE - 1, FIRST + TILE + 1,
                               3 * 1024 * TILE - 7])
@pytest.mark.parametrize("kind", ["random", "equal", "few"])
def test_large_tiles(sba, n, kind):
    rng = np.random.default_rng(n)
    if kind == "random":
        keys = rng.integers(0, 2**62, n, dtype=np.int64)
    elif kind == "equal":
        keys = np.full(n, 255, np.int64)
    else:
        keys = rng.integers(0, 3, n, dtype=np.int64) * 127
    for bits in (8, 24) if kind != "random" else (21, 40):
        check_sort(sba, keys & ((1 << bits) - 1), bits, with_vals=bits != 24)
