"""Automatic plans keep their split partials under 8 GiB (host-only plans)."""
import numpy as np

from paper_1910_01965_amd import workloads as wl
from paper_1910_01965_amd import zmc


def test_automatic_fp64_plans_stay_under_8_gib_at_any_compute_unit_count():
    spec = wl.ScanSpec("sin_sum", [np.linspace(0.0, 1.0, 120)] * 4, np.zeros(4), np.ones(4), 2049, 1, "fp64")
    for cu in (1, 256, 10 ** 5, 10 ** 6, 4 * 10 ** 6):
        assert zmc.plan(spec, cu_count=cu)["workspace_bytes"] <= 8 << 30, cu


def test_fp64_grids_of_one_wave_per_simd_are_cut():
    def plan(points, samples, precision="fp64"):
        return zmc.plan(wl.ScanSpec("sin_sum", [np.linspace(0.0, 1.0, points)], np.zeros(2), np.ones(2), samples, 1,
                                    precision), cu_count=256)

    for samples, pieces in ((128, 1), (188, 1), (189, 3), (256, 4), (511, 5)):
        p = plan(65536, samples)
        assert p["mode"] == "point_major" and p["splits"] == pieces, (samples, p)
    assert plan(65537, 256)["splits"] == 1 and plan(65536, 256, "fp32")["splits"] == 1
