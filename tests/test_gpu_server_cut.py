"""The server cuts a request into the tiles that a batch would, whatever its budget:
FP64 requests whose finer pieces do not fit the budget still run, with the bits of
the batch, from host lists and from device lists."""
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


@pytest.mark.parametrize("budget", [1 << 20, 3 << 20, 0])
def test_small_budgets_keep_the_batch_bits(budget):
    import torch
    from paper_1910_01965_amd import zmc
    specs = [wl.ScanSpec("sin_sum", [np.linspace(0.0, 1.0, 33000 + i)], np.zeros(2), np.ones(2), 4093 + i, i, "fp64")
             for i in range(3)]
    assert zmc.batch_plan(specs, cu_count=256, pm_groups=1024)["merge_scans"] == 0  # one piece by the table
    info = zmc.batch_plan(specs, cu_count=256)
    assert info["merge_scans"] == 3 and info["workspace_bytes"] > 3 << 20  # each in pieces, above 1 MiB
    ref = zmc.scan_batch(specs)
    print("server cut", budget, flush=True)
    srv = zmc.Server(hbm_budget_bytes=budget)
    axes = [zmc.axis_tensor(sp) for sp in specs]
    torch.cuda.synchronize()
    tickets = [(i, srv.submit(sp, axis=a)) for i, sp in enumerate(specs) for a in (None, axes[i])]
    for i, t in tickets:
        status, _ = srv.wait(t)
        assert status == 0
        f, s = srv.outputs(t)
        torch.cuda.synchronize()
        assert torch.equal(f, ref[i][0]) and torch.equal(s, ref[i][1]), (budget, i)
    srv.close()
