"""Sample-major blocks of user integrands: up to 256 threads from a variant's first
build, larger ones from a kernel that only such a plan builds."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import sys
import numpy as np, torch
sys.path.insert(0, 'tests')
import parity
from oracle import oracle as zo
from paper_1910_01965_amd import zmc, workloads as wl
SRC = '''template <typename T> __device__ T integrand(const T* y, const T* x, const T* p) {
  return p[0] * exp(-(x[0] * y[0] * y[0] + y[1] * y[1])); }'''
ref = wl.ScanSpec('gauss', [np.linspace(0.1, 3.0, 7)], np.zeros(2), np.ones(2), 5001, 3, '%s')
sp = wl.ScanSpec('user', ref.axes, ref.lo, ref.hi, ref.samples, ref.seed, ref.precision, source=SRC, params=np.array([1.0]))
f_ref, s_ref = zo.scan(ref)
for block in (64, 256, 320, 1024, 512):
    f, s = zmc.scan(sp, mode='sample_major', block=block)
    torch.cuda.synchronize()
    parity.check(f.cpu().numpy(), s.cpu().numpy(), f_ref, s_ref, sp.samples, sp.precision, str(block))
    print('block', block, flush=True)
"""


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_large_blocks_build_one_kernel_more(precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("user blocks", precision, flush=True)
    r = subprocess.run([sys.executable, "-c", CODE % precision], cwd=ROOT, env=dict(os.environ, ZMC_LOG="1"),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
    built = [ln for ln in r.stderr.splitlines() if "compiled the" in ln and "N = 2, M = 1" in ln]
    assert len(built) == 2 and "large-block" not in built[0] and "large-block" in built[1], built
