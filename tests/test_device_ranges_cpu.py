"""Host builds of the FP64 integrands at the edges of their ranges (no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1910_01965_amd", "csrc")


def _run(name, tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / name)
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "-O2", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "cpu_checks", name + ".cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    return out.stdout.split()


def test_sin_of_small_phases_keeps_its_relative_accuracy(tmp_path):
    """Within the roundings of 1/(2 pi), of A and of the phase (N - 1 additions and
    one fma) and the sine polynomial's own error."""
    e1, e3, bad, out = _run("small_phase", tmp_path)
    assert float(e1) < 1.0 and float(e3) < 1.0, (e1, e3)
    assert int(bad) == 0 and int(out) == 0


def test_cosexp_exponent_and_phase_over_their_ranges(tmp_path):
    """The exponent within the roundings of its factors where they are near 0 (boxes
    [-1, 0] and [-3, -1/2], x3 up to 1000), the phase within those of its terms, and
    2^t of an exponent that overflows as exp gives it."""
    e, c, bad = _run("cosexp_ranges", tmp_path)
    assert float(e) < 1.0 and float(c) < 1.0 and int(bad) == 0, (e, c, bad)


def test_sin_phases_are_reduced_without_the_rounding_of_the_whole(tmp_path):
    """No more error than one rounding of the sum and one of the reduced phase allow, none
    more than with the product rounded first (up to the noise of 20000 samples), and
    bounded values at phases of any size."""
    worst, ratio, out, flat = _run("sin_phases", tmp_path)
    assert float(worst) < 1.0 and float(ratio) < 1.02 and int(out) == 0 and int(flat) == 0, (worst, ratio, out, flat)
