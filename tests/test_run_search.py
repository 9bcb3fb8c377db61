"""The search for a key's run in a block of the Hilbert layout, as the kernels
make it, against numpy's; and its rounds of loads, which may not exceed the steps
of a halving search by more than two (one for the estimate, one for the start)."""
import math

import numpy as np
import pytest

import paper_2010_12548_amd as sba


def search(starts, keys, guess):
    run, rounds = np.empty(keys.size, np.int64), np.empty(keys.size, np.int32)
    rc = sba.lib().sba_debug_run_search(starts.ctypes.data, starts.size, keys.ctypes.data,
                                        keys.size, guess, run.ctypes.data, rounds.ctypes.data)
    assert rc == 0
    return run, rounds


@pytest.mark.parametrize("n", [*range(1, 70), 255, 1023, 1024, 1025, 4096, 16_384, 1_000_003])
def test_run_search(n):
    r = np.random.default_rng(n)
    starts = np.unique(np.concatenate(([0], r.integers(1, 1 << 42, size=4 * n))))[:n].astype(np.uint64)
    keys = np.concatenate((starts[-300:], starts[:300], starts[1:301] - np.uint64(1),
                           r.integers(0, 1 << 42, size=400).astype(np.uint64)))
    want = np.searchsorted(starts, keys, side="right") - 1
    most = math.ceil(math.log2(starts.size)) + 2 if starts.size > 1 else 1
    for guess in (-1, 0, n // 3, n - 1):
        run, rounds = search(starts, keys, min(guess, starts.size - 1))
        np.testing.assert_array_equal(run, want)
        assert rounds.max() <= most, (guess, rounds.max())
