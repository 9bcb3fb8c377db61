"""The radix sort on both sides of the size from which it takes large tiles, whose
digits are always of 8 bits: whole keys, the bits above the last digit ignored,
equal keys in their order."""
import numpy as np
import pytest
import torch

import paper_2010_12548_amd as sba

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(5 << 18) - 1, 5 << 18, (5 << 18) + 1, 2_100_003, 4_194_303])
@pytest.mark.parametrize("bits", [9, 20, 42, 64])
def test_sizes(n, bits):
    r = np.random.default_rng(n + bits)
    k = r.integers(0, 1 << min(bits, 16), size=n).astype(np.uint64) << np.uint64(max(bits - 16, 0))
    keys, vals = torch.from_numpy(k.view(np.int64)).cuda(), torch.arange(n, dtype=torch.int32,
                                                                       device="cuda")
    sba.radix_sort(keys, vals, bits=bits)
    order = np.argsort(k, kind="stable")
    np.testing.assert_array_equal(vals.cpu().numpy(), order)
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), k[order])
