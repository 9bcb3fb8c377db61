"""Offsets of many rings are checked to the last, wherever the decreasing one lies."""
import numpy as np
import pytest
import torch

from test_gpu_parity import sba  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 7_169, 8_192, 8_193, 20_000])
def test_decreasing_offsets_are_refused(sba, n):
    x = 20 * np.arange(n, dtype=np.int32)
    z = np.zeros_like(x)
    xy = np.stack((x, z, x + 9, z, x + 9, z + 9, x, z + 9), 1).ravel()
    ro = torch.tensor([0, n // 3, n] if n > 2 else [0, n], dtype=torch.int32, device="cuda")
    off = 4 * np.arange(n + 1, dtype=np.int64)
    xy = torch.from_numpy(xy).cuda()

    def build(o):
        A = sba.Approx(ro, torch.from_numpy(o).cuda(), xy, 50)
        torch.cuda.synchronize()
        return A

    assert build(off).n_polys == len(ro) - 1
    for r in {0, 1, 1023, 1024, 7_168, 8_191, 8_192, 16_384, n // 2, n - 1}:
        if r >= n:
            continue
        bad = off.copy()
        bad[r], bad[r + 1] = off[r + 1], off[r]  # every offset stays inside the vertices
        with pytest.raises(sba.SbaError):
            build(bad)
    build(off)
