"""FP64 scans of mid-sized grids: the planner's point-major pieces and the tree
merge of many pieces, at the edges of their ranges, against the oracle."""
import numpy as np
import parity
import pytest

from oracle import oracle as zo
from paper_1910_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01965_amd import zmc
    zmc.load()
    return torch


def _spec(family, lens, N, samples):
    box = {"sin_sum": (0.0, 1.0), "gauss": (0.1, 10.0), "cosexp": (-1.0, 1.0)}[family]
    return wl.ScanSpec(family, [np.linspace(*box, L) for L in lens], np.zeros(N), np.ones(N), samples,
                       77, "fp64")


def _check(spec, points, **kw):
    import torch
    from paper_1910_01965_amd import zmc
    f, s = zmc.scan(spec, **kw)
    torch.cuda.synchronize()
    idx = np.unique(np.linspace(0, spec.G - 1, points).astype(np.uint64))
    f_ref, s_ref = zo.scan(spec, idx)
    sel = torch.from_numpy(idx.astype(np.int64))
    parity.check(f.cpu()[sel].numpy(), s.cpu()[sel].numpy(), f_ref, s_ref, spec.samples, "fp64", "mid grid")


# below, at and past a multiple of 64 points and of the planner's 16-group
# pieces; one piece; a ragged last group; pieces past the tree's threshold
@pytest.mark.parametrize("family,lens,N,samples", [
    ("sin_sum", [65535], 2, 2), ("sin_sum", [40001], 3, 33), ("gauss", [100, 100], 4, 1025),
    ("cosexp", [9, 8, 8, 7], 2, 4099), ("sin_sum", [4097], 5, 4097), ("gauss", [211, 97], 12, 515)])
def test_mid_grid_plans_match_oracle(family, lens, N, samples):
    from paper_1910_01965_amd import zmc
    spec = _spec(family, lens, N, samples)
    print(family, lens, N, samples, zmc.plan(spec), flush=True)
    assert zmc.plan(spec)["mode"] == "point_major"
    _check(spec, 40)


@pytest.mark.parametrize("splits", [1, 2, 15, 16, 17, 31, 256, 257])
@pytest.mark.parametrize("G", [1, 15, 17, 300])
def test_merge_of_many_pieces_matches_oracle(G, splits):
    spec = _spec("sin_sum", [G], 2, 1031)
    print("merge", G, splits, flush=True)
    _check(spec, min(G, 20), mode="point_major", splits=splits)
