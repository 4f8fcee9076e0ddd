"""Workspaces of scans on many streams, and what host-memory scans leave behind
(child processes, since the library reads its log level once)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01965_amd import zmc
    zmc.load()
    return torch


def _new_buffers(code):
    head = ("import numpy as np, torch\n"
            "from paper_1910_01965_amd import zmc, workloads as wl\n"
            "def spec(G, n, precision, N=8):\n"
            "    return wl.ScanSpec('sin_sum', [np.linspace(0, 1, G)], np.zeros(N), np.ones(N), n, 3, precision)\n")
    r = subprocess.run([sys.executable, "-c", head + code], cwd=ROOT, env=dict(os.environ, ZMC_LOG="2"),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return [ln for ln in r.stderr.splitlines() if ln.startswith("[zmc] workspace: new")]


def test_mid_sized_scans_on_eight_streams_have_their_own_workspaces():
    print("eight streams", flush=True)
    new = _new_buffers(
        "sp = spec(20467, 2049, 'fp64', 12)\n"
        "assert 0 < zmc.plan(sp)['workspace_bytes'] <= 8 << 20\n"
        "ax = zmc.axis_tensor(sp)\n"
        "out = [(torch.empty(sp.G, dtype=torch.float64, device='cuda'), torch.empty(sp.G, dtype=torch.float64,"
        " device='cuda')) for _ in range(8)]\n"
        "st = [torch.cuda.Stream() for _ in out]\n"
        "torch.cuda.synchronize()\n"
        "long = spec(20000, 300001, 'fp64'); assert zmc.plan(long)['workspace_bytes'] == 0\n"
        "zmc.scan(long)  # the eight scans wait for it\n"
        "for t in st: t.wait_stream(torch.cuda.current_stream())\n"
        "for (f, s), t in zip(out, st): zmc.scan_device(sp, ax, f, s, stream=t)\n"
        "torch.cuda.synchronize()\n"
        "assert all(torch.equal(f, out[0][0]) and torch.equal(s, out[0][1]) for f, s in out)\n")
    assert len(new) == 8, new


def test_large_host_scans_leave_no_buffer():
    """A host-memory scan of few points whose partials take 134 MB frees them."""
    print("large host scan", flush=True)
    new = _new_buffers(
        "import ctypes\n"
        "sp = spec(100000, 65536, 'fp32')\n"
        "assert zmc.plan(sp)['workspace_bytes'] > 100 << 20\n"
        "f, s = zmc.scan_chunked(sp)\n"
        "g, t = zmc.scan_range(sp, 0, 1000)\n"
        "assert np.array_equal(f[:1000], g) and np.array_equal(s[:1000], t) and np.all(np.isfinite(f))\n")
    assert len(new) == 1 and int(new[0].split("new ")[1].split("-byte")[0]) <= 8 << 20, new  # the range's own
