"""Automatic plans keep their split partials under 8 GiB (host-only plans)."""
import numpy as np

from paper_1910_01965_amd import workloads as wl
from paper_1910_01965_amd import zmc


def test_automatic_fp64_plans_stay_under_8_gib_at_any_compute_unit_count():
    spec = wl.ScanSpec("sin_sum", [np.linspace(0.0, 1.0, 120)] * 4, np.zeros(4), np.ones(4), 2049, 1, "fp64")
    for cu in (1, 256, 10 ** 5, 10 ** 6, 4 * 10 ** 6):
        assert zmc.plan(spec, cu_count=cu)["workspace_bytes"] <= 8 << 30, cu
