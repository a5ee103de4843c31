"""What a call leaves beside histograms counted straight from the staged keys:
the table, and the per-host statistics whose staging cursor they share, against
the oracle (whole numbers, tolerance 0)."""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from tests._gpu import DEV, offsets_to_device, to_device
from tests.test_gpu_hist_direct import REGS
from tests.test_gpu_hosts import check as check_hosts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sites,n,grid,nw,hosts", [
    (64, 30_000, 0, 1, True), (1000, 9_999, 5, 1, True), (64, 102_400, 0, 2, True), (64, 5, 0, 1, True),
    (64, 40_001, 3, 1, False), (1000, 3_001, 0, 2, False)])
def test_table_and_hosts(sites, n, grid, nw, hosts):
    import torch
    print("case: beside direct histograms", sites, n, grid, nw, hosts, flush=True)
    r = flowgen.registry_for(REGS[sites])
    rec = flowgen.records_for(REGS[sites], reg=r, n=n)
    off = None if nw == 1 else np.array([0, n // 3, n], dtype=np.uint64)
    reg, orc = gnm.Registry.from_generated(r), oracle.Registry.from_generated(r)
    hist = gnm.make_rate_hist(reg, nw)
    table = gnm.HostTable(reg, 2 * n, n, grid, device=DEV) if hosts else None
    acc = torch.full((nw, reg.rows, 8), 7, dtype=torch.int64, device=DEV)
    gnm.classify_aggregate(reg, to_device(rec), acc, n=n, n_windows=nw, grid_blocks=grid, rate_hist=hist, hosts=table,
                           window_offsets=None if off is None else offsets_to_device(off),
                           workspace=gnm.make_workspace(reg, grid, n_records=n, n_windows=nw, hist=True))
    torch.cuda.synchronize()
    exp = orc.classify_aggregate(rec, window_offsets=off)
    assert (gnm.acc_to_numpy(acc) == exp.reshape(nw, reg.rows, 8)).all()
    eh = oracle.rate_histograms(orc, rec, window_offsets=off)[:, :2 * reg.n_sites]
    assert (hist.cpu().numpy().view(np.uint32).reshape(eh.shape) == eh).all()
    if hosts:
        check_hosts(table, orc, rec)
