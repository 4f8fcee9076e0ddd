"""Device memory and tiles of batches of many FP64 scans (host-only plans)."""
import numpy as np
import pytest

from paper_1910_01965_amd import workloads as wl
from paper_1910_01965_amd import zmc


def _spec(points, samples, N=7):
    return wl.ScanSpec("sin_sum", [np.linspace(0.0, 1.0, points)], np.zeros(N), np.ones(N), samples, 1, "fp64")


# grids of one piece by the tuned table: what the finer cut adds to it is bounded for
# each scan, and a batch holds that times its scans
@pytest.mark.parametrize("points,samples", [(66000, 32768), (100000, 32768), (10 ** 6, 32768)])
def test_finer_fp64_tiles_are_bounded(points, samples):
    table = zmc.batch_plan([_spec(points, samples)], cu_count=256, pm_groups=8192, pm_min_points=1)
    assert table["merge_scans"] == 0
    for count in (1, 100):
        info = zmc.batch_plan([_spec(points, samples)] * count, cu_count=256)
        assert info["workspace_bytes"] <= count * (table["workspace_bytes"] + (8 << 20) + 16 * 2100)
        assert info["tiles"] <= count * max(table["tiles"], 2100)
