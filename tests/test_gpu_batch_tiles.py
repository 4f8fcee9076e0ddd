"""GAUSS and COSEXP in the tiles of batches and of the server: sample-major tiles of
several points and finely cut FP64 point-major tiles, at the edges of pieces and of
point blocks, against the oracle, and the server's bits against the batch's."""
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


def _spec(family, lens, N, samples, precision, seed):
    box = {"gauss": (0.1, 10.0), "cosexp": (-1.0, 1.0)}[family]
    return wl.ScanSpec(family, [np.linspace(*box, L) for L in lens], np.zeros(N), np.ones(N), samples, seed,
                       precision)


def _check(specs, points):
    import torch
    from paper_1910_01965_amd import zmc
    out = zmc.scan_batch(specs)
    srv = zmc.Server()
    tickets = [srv.submit(sp) for sp in specs]
    for sp, (f, s), t in zip(specs, out, tickets):
        assert srv.wait(t)[0] == 0
        g, r = srv.outputs(t)
        torch.cuda.synchronize()
        assert torch.equal(f, g) and torch.equal(s, r), (sp.family, sp.N, sp.samples)
        idx = np.unique(np.linspace(0, sp.G - 1, points).astype(np.uint64))
        f_ref, s_ref = zo.scan(sp, idx)
        sel = torch.from_numpy(idx.astype(np.int64))
        parity.check(f.cpu()[sel].numpy(), s.cpu()[sel].numpy(), f_ref, s_ref, sp.samples, sp.precision,
                     f"{sp.family} N={sp.N} G={sp.G} n={sp.samples}",
                     small_n=sp.precision == "fp32" and sp.samples < 4096)
    srv.close()


# pieces of 1, 64, 65, 128, 129 and 257 groups: one, two and four waves a point
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("family,lens", [("gauss", [33, 31]), ("gauss", [3, 3]), ("cosexp", [6, 6, 5, 7]),
                                         ("cosexp", [1, 2, 3, 1])])
def test_tiles_of_several_points(family, lens, precision):
    specs = [_spec(family, lens, N, n, precision, 20 + i)
             for i, n in enumerate([2, 256, 257, 512, 513, 1027]) for N in (2, 5)]
    print("tiles of several points", family, lens, precision, flush=True)
    _check(specs, 10)


# 7 and 15 pieces a grid, a ragged last group and a last block of few points
@pytest.mark.parametrize("family,lens,N,samples", [
    ("gauss", [257, 129], 2, 8195), ("gauss", [257, 256], 6, 8191), ("cosexp", [17, 16, 16, 16], 3, 8197),
    ("cosexp", [13, 13, 13, 31], 7, 6007)])
def test_finely_cut_fp64_tiles(family, lens, N, samples):
    from paper_1910_01965_amd import zmc
    spec = _spec(family, lens, N, samples, "fp64", 31)
    info = zmc.batch_plan([spec], cu_count=256)
    print("finely cut", family, lens, N, samples, info["tiles"], flush=True)
    assert info["tiles"] > 4 * ((spec.G + 255) // 256) and info["merge_scans"] == 1
    _check([spec], 24)
