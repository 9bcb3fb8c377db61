"""The name of the kernel that aggregates many points over a handle, with every
template argument, as profilers list it."""
import re

import pytest

from gen import star_polygons, voronoi_partition
from test_gpu_parity import sba  # noqa: F401

pytestmark = pytest.mark.gpu


def test_names(sba):
    polys = star_polygons(12, 9, 20.0, 400.0, 1500, 55)
    many = voronoi_partition(4_100, 100_000, (1, 2), seed=31, jitter_seed=32)
    for v in (False, True):
        t = "true" if v else "false"
        assert re.fullmatch(r"k_probe_grid16<%s, \d, \d, \d+>" % t,
                            sba.Approx.from_polygons(polys, 5).probe_kernel(v))
        for kw, layout in ((dict(kind="hilbert"), 1), (dict(kind="hilbert", search="learned"), 2)):
            A = sba.Approx.from_polygons(polys, 5, **kw)
            assert A.probe_kernel(v) == "k_probe_items<%d, %s, 1, 4>" % (layout, t)
        # a key grid above level 16: 64-bit keys
        A = sba.Approx.from_polygons(polys, 5, kind="hilbert", key_grid=(18, -100, -100))
        assert A.probe_kernel(v) == "k_probe_items<3, %s, 1, 4>" % t
        sba.lib().sba_debug_force_wide_grid(1)
        try:
            A = sba.Approx.from_polygons(polys, 5)
            M = sba.Approx.from_polygons(many, 100)
        finally:
            sba.lib().sba_debug_force_wide_grid(0)
        assert A.probe_kernel(v) == "k_probe_lds<%s, 4>" % t
        assert M.probe_kernel(v) == "k_probe_items<0, %s, 1, 4>" % t
