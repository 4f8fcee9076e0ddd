"""The autotuner compares tiles that the planner would run (no GPU: plans only)."""
import pytest

from paper_1910_01965_amd import autotune, zmc


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_point_major_threshold_is_timed_on_the_planner_tiles(precision, monkeypatch):
    seen = []

    def fake(z, specs, reps, **opts):
        (sp,) = specs
        default = zmc.batch_plan(specs, cu_count=256, **{k: v for k, v in opts.items() if k == "pm_min_points"})
        tiles = zmc.batch_plan(specs, cu_count=256, **opts)["tiles"]
        seen.append((sp.G, opts, tiles, default["tiles"]))
        return float(opts["pm_min_points"] == 1)  # sample-major wins: every size is tried

    monkeypatch.setattr(autotune, "_time_batch", fake)
    autotune.tune_pm_min(zmc, "sin_sum", precision, 7, 8192, 1, lambda m: None)
    assert len(seen) == 2 * len(autotune.PM_MIN_CANDIDATES)
    for G, opts, tiles, default in seen:
        if precision == "fp64" or opts["pm_min_points"] > 1:
            assert tiles == default, (G, opts)
        else:
            assert opts["pm_groups"] == 8192
