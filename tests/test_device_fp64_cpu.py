"""Host builds of the FP64 set-up and sample functions of the kernels (no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1910_01965_amd", "csrc")


def test_exp2_table_and_phase_reduction_against_long_double(tmp_path):
    """2^t within half an ulp and the polynomial's own rounding (1.2e-16, below
    the 1.3e-16 of a polynomial without a table); e^-q with the rounding of
    q log2 e besides; a phase's fraction within 2^-53 of a revolution; the sine by the
    quarter turn within the sine polynomial's 2.8e-16 and that phase error."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "exp2_table")
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "-O2", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "cpu_checks", "exp2_table.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    e, q, t, s, bad = out.stdout.split()
    assert float(e) < 1.2e-16 and float(q) < 2.4e-16, out.stdout
    assert float(t) < 2.0 ** -53 and float(s) < 2.8e-16 + 6.3 * 2.0 ** -53 and int(bad) == 0, out.stdout
