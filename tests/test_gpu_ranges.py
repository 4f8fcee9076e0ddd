"""Scans at the edges of their value ranges, against the oracle."""
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


def _check(spec, f, s, label):
    f_ref, s_ref = zo.scan(spec)
    parity.check(f.cpu().numpy(), s.cpu().numpy(), f_ref, s_ref, spec.samples, "fp64", label)


# sin of a phase as small as the box: an absolute error of 1e-16 would be 1e-4 of f
@pytest.mark.parametrize("N", [1, 3, 11])
@pytest.mark.parametrize("w", [1e-3, 1e-6, 1e-12, 1e-17])
def test_small_phases(w, N):
    import torch
    from paper_1910_01965_amd import zmc
    spec = wl.ScanSpec("sin_sum", [np.zeros(130)], np.zeros(N), w * np.ones(N), 1031, 5, "fp64")
    for mode in ("point_major", "sample_major"):
        print("small phases", w, N, mode, flush=True)
        f, s = zmc.scan(spec, mode=mode)
        torch.cuda.synchronize()
        _check(spec, f, s, f"w={w} N={N} {mode}")
    (f, s), = zmc.scan_batch([spec])
    _check(spec, f, s, f"w={w} N={N} batch")


# exponents -x3^2 y1 y2 of samples near the edge of [-1, 0]^2, where only small
# coordinates count
@pytest.mark.parametrize("x3", [1.0, 30.0, 1000.0])
@pytest.mark.parametrize("N", [2, 5, 12])
def test_cosexp_exponents_on_negative_boxes(N, x3):
    import torch
    from paper_1910_01965_amd import zmc
    axes = [np.array([0.0, 0.3]), np.array([0.1, 0.2]), x3 * np.array([0.5, 1.0]), np.array([0.0])]
    spec = wl.ScanSpec("cosexp", axes, -np.ones(N), np.zeros(N), 4099, 9, "fp64")
    for mode in ("point_major", "sample_major"):
        print("cosexp exponents", N, x3, mode, flush=True)
        f, s = zmc.scan(spec, mode=mode)
        torch.cuda.synchronize()
        _check(spec, f, s, f"x3={x3} N={N} {mode}")


# every sample is x4 to the last bit: a sum of n x4 overflows, the mean does not
@pytest.mark.parametrize("samples", [2, 200, 500, 1031, 4100, 70001])
def test_means_near_the_largest_double(samples):
    import torch
    from paper_1910_01965_amd import zmc
    axes = [np.array([0.2]), np.array([0.3]), np.array([0.4]), np.array([1e306, -1.7e308])]
    spec = wl.ScanSpec("cosexp", axes, np.zeros(3), np.ones(3), samples, 11, "fp64")
    runs = [zmc.scan(spec, mode=m) for m in ("sample_major", "point_major")]
    runs += [zmc.scan(spec, mode="sample_major", block=1024), zmc.scan_batch([spec])[0]]
    torch.cuda.synchronize()
    for i, (f, s) in enumerate(runs):
        print("large means", samples, i, flush=True)
        assert f.cpu().tolist() == [1e306, -1.7e308] and s.cpu().tolist() == [0.0, 0.0]


# phases that FP64 no longer resolves: bounded values, spread like a sine's
@pytest.mark.parametrize("box,x", [(1e15, 0.5), (1e18, 0.5), (1.0, 1e17), (1e300, 1e300)])
def test_sin_of_unresolved_phases_stays_bounded(box, x):
    import torch
    from paper_1910_01965_amd import zmc
    spec = wl.ScanSpec("sin_sum", [x * np.linspace(1.0, 1.5, 70)], np.zeros(2), np.array([box, 1.0]), 4099, 5, "fp64")
    for mode in ("point_major", "sample_major"):
        print("unresolved phases", box, x, mode, flush=True)
        f, s = zmc.scan(spec, mode=mode)
        torch.cuda.synchronize()
        f, s = f.cpu().numpy() / box, s.cpu().numpy() / box * np.sqrt(4099)
        assert np.all(np.abs(f) <= 1.0) and np.all(np.isfinite(s)) and np.all(s <= 1.0)
        if 1.0 < box < 1e20:
            assert np.all(np.abs(f) < 0.07) and np.all(np.abs(s - 0.5 ** 0.5) < 0.05)
