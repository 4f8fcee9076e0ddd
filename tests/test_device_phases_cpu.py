"""Host builds of the phased Philox blocks of the point-major and sample-major
kernels and of the grid decoding (no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1910_01965_amd", "csrc")


@pytest.mark.parametrize("name", ["philox_phased", "philox_point", "param_cursor"])
def test_fast_path_equals_generic(name, tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / name)
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "-O2", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "cpu_checks", name + ".cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    bad, total = (int(t) for t in out.stdout.split())
    assert total >= 60000 and bad == 0 and out.returncode == 0
