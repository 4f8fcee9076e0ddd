"""FP64 grids of just one wave per SIMD (65536 points on 256 compute units), around the
sample counts where they are cut, against the oracle."""
import numpy as np
import parity
import pytest

from oracle import oracle as zo
from paper_1910_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("samples", [188, 189, 259, 511])
@pytest.mark.parametrize("family,N", [("sin_sum", 1), ("gauss", 3), ("cosexp", 2)])
def test_one_wave_per_simd(family, N, samples):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01965_amd import zmc
    lens = {"sin_sum": [65536], "gauss": [256, 256], "cosexp": [16, 16, 16, 16]}[family]
    lo, hi = {"sin_sum": (0.0, 1.0), "gauss": (0.1, 10.0), "cosexp": (-1.0, 1.0)}[family]
    spec = wl.ScanSpec(family, [np.linspace(lo, hi, L) for L in lens], np.zeros(N), np.ones(N), samples, 7, "fp64")
    print("one wave", family, samples, zmc.plan(spec), flush=True)
    f, s = zmc.scan(spec)
    torch.cuda.synchronize()
    idx = np.unique(np.linspace(0, spec.G - 1, 300).astype(np.uint64))
    f_ref, s_ref = zo.scan(spec, idx)
    sel = torch.from_numpy(idx.astype(np.int64))
    parity.check(f.cpu()[sel].numpy(), s.cpu()[sel].numpy(), f_ref, s_ref, samples, "fp64", f"{family} n={samples}")
