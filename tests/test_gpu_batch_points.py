"""Sample-major batch tiles of several points: pieces of one, two and four waves
and one group more, point counts around a tile's, in both precisions, against the
oracle; each scan bitwise the same alone and in the mix."""
import numpy as np
import parity
import pytest

from oracle import oracle as zo
from paper_1910_01965_amd import workloads as wl

pytestmark = pytest.mark.gpu

SAMPLES = [2, 256, 257, 512, 513, 1027, 4100]  # 1, 64, 65, 128, 129, 257, 1025 groups


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01965_amd import zmc
    zmc.load()
    return torch


def _spec(G, samples, precision, seed):
    return wl.ScanSpec("sin_sum", [np.linspace(0.0, 1.0, G)], np.zeros(3), np.ones(3), samples, seed, precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("G", [1, 5, 1023, 1025, 8209])
def test_tiles_of_several_points(G, precision):
    import torch
    from paper_1910_01965_amd import zmc
    specs = [_spec(G, n, precision, 10 + i) for i, n in enumerate(SAMPLES)]
    print("points", G, precision, flush=True)
    mix = zmc.scan_batch(specs)
    idx = np.unique(np.linspace(0, G - 1, 12).astype(np.uint64))
    for sp, (f, s) in zip(specs, mix):
        (fa, sa), = zmc.scan_batch([sp])
        assert torch.equal(f, fa) and torch.equal(s, sa), sp.samples
        f_ref, s_ref = zo.scan(sp, idx)
        sel = torch.from_numpy(idx.astype(np.int64))
        parity.check(f.cpu()[sel].numpy(), s.cpu()[sel].numpy(), f_ref, s_ref, sp.samples, precision,
                     f"G={G} n={sp.samples}", small_n=precision == "fp32" and sp.samples < 4096)
