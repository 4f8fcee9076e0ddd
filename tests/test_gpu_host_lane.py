"""Host-memory scans of one small chunk (kept stream and pinned staging): sizes
around the staging's limit equal the device scan bit for bit, also from several
threads at once and mixed with scans that take the chunk pipeline."""
import threading

import numpy as np
import pytest

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


def _spec(lens, precision, seed, samples=37):
    return wl.ScanSpec("cosexp", [np.linspace(-1.0, 1.0, L) for L in lens], np.zeros(2), np.ones(2), samples,
                       seed, precision)


def _device(spec):
    import torch
    from paper_1910_01965_amd import zmc
    f, s = zmc.scan(spec)
    torch.cuda.synchronize()
    return f.cpu().numpy(), s.cpu().numpy()


# 4 MiB of staging hold the lists and 16 B a point: the last two grids are just
# below and just above it
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("lens", [(1, 1, 1, 1), (3, 1, 7, 5), (64, 64, 8, 7), (64, 64, 63, 1), (64, 64, 8, 8)])
def test_host_scan_equals_device_scan(lens, precision):
    from paper_1910_01965_amd import zmc
    spec = _spec(lens, precision, 3)
    print("host lane", lens, precision, flush=True)
    f_ref, s_ref = _device(spec)
    for _ in range(2):
        f, s = zmc.scan_chunked(spec)
        assert np.array_equal(f, f_ref) and np.array_equal(s, s_ref)
    lo, hi = spec.G // 3, spec.G // 3 + max(1, spec.G // 2)
    f, s = zmc.scan_range(spec, lo, hi)
    assert np.array_equal(f, f_ref[lo:hi]) and np.array_equal(s, s_ref[lo:hi])


def test_host_scans_from_threads():
    from paper_1910_01965_amd import zmc
    specs = [_spec((5 + i, 9, 4, 64 if i % 3 == 0 else 3), "fp64" if i % 2 else "fp32", i, 600) for i in range(12)]
    refs = [_device(sp) for sp in specs]
    bad = []

    def work(k):
        for r in range(4):
            i = (k * 5 + r) % len(specs)
            f, s = zmc.scan_chunked(specs[i], chunk_points=0 if r % 2 else 10 ** 6)
            if not (np.array_equal(f, refs[i][0]) and np.array_equal(s, refs[i][1])):
                bad.append((k, i))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
