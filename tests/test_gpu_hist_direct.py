"""Small calls' rate histograms, counted straight from the staged keys, against
the oracle: every count equal (tolerance 0), on both sides of the lines
between that and the partition kernels (records, records x rows), for both
piece lengths (up to 256 rows, and beyond), ranges that end on, before and
after a piece's end, empty ranges and windows, rows filled on top of others
(accumulate), one hot bucket, and the per-host statistics' shared staging
cursor."""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from tests._gpu import DEV, offsets_to_device, to_device

pytestmark = pytest.mark.gpu

REGS = {64: flowgen.PLAIN_SMALL, 1000: flowgen.PLAIN_LARGE}


def _run(sites, n, nw=1, grid=0, accumulate=False, hot=False, hosts=False):
    import torch
    print("case: direct histograms", sites, n, nw, grid, accumulate, hot, hosts, flush=True)
    r = flowgen.registry_for(REGS[sites])
    rec = flowgen.records_for(REGS[sites], reg=r, n=n)
    if hot:  # every second record a copy of one bulk flow
        i = int(np.argmax(rec.bytes))
        for f in ("src_ip", "dst_ip", "bytes", "packets", "first_ms", "last_ms"):
            getattr(rec, f)[::2] = getattr(rec, f)[i]
    off = None
    if nw > 1:  # uneven windows, the second of several empty
        cut = np.sort(np.random.default_rng(n + nw).integers(0, n + 1, nw - 1))
        off = np.concatenate([[0], cut, [n]]).astype(np.uint64)
        if nw > 2:
            off[2] = off[1]
    reg, orc = gnm.Registry.from_generated(r), oracle.Registry.from_generated(r)
    exp = oracle.rate_histograms(orc, rec, window_offsets=off)[:, :2 * reg.n_sites].astype(np.int64)
    hist = gnm.make_rate_hist(reg, nw)
    hist.fill_(3)
    table = gnm.HostTable(reg, 2 * n, n, grid, device=DEV) if hosts else None
    acc = torch.zeros((nw, reg.rows, 8), dtype=torch.int64, device=DEV)
    ws = gnm.make_workspace(reg, grid, n_records=n, n_windows=nw, hist=True)
    gnm.classify_aggregate(reg, to_device(rec), acc, n=n, n_windows=nw, grid_blocks=grid, workspace=ws, rate_hist=hist,
                           hosts=table,
                           window_offsets=None if off is None else offsets_to_device(off), accumulate=accumulate)
    torch.cuda.synchronize()
    got = hist.cpu().numpy().view(np.uint32).reshape(exp.shape).astype(np.int64)
    np.testing.assert_array_equal(got, exp + (3 if accumulate else 0))
    assert exp.sum() > 0


@pytest.mark.parametrize("sites,n,nw", [
    (64, 1, 1), (64, 5, 1), (64, 102_400, 1), (64, 102_401, 1),      # the line in records
    (64, 102_400, 2), (64, 65_536, 4), (64, 65_537, 4),              # 256 rows; the line in records x rows
    (64, 20_000, 3), (1000, 16_777, 1), (1000, 16_778, 1), (1000, 3_001, 2),
])
@pytest.mark.parametrize("accumulate", [False, True])
def test_lines(sites, n, nw, accumulate):
    _run(sites, n, nw, accumulate=accumulate)


# one, two and many ranges; keys per range about 1,024 and 2,048; more workgroups than records / 4, and past 2,048
@pytest.mark.parametrize("grid", [1, 2, 3, 31, 2048, 2049])
@pytest.mark.parametrize("sites,n", [(64, 4_099), (64, 8_000), (64, 40_001), (1000, 9_998)])
def test_ranges(sites, n, grid):
    _run(sites, n, grid=grid)


@pytest.mark.parametrize("n", [1_000, 102_400])
def test_hot_bucket(n):
    _run(64, n, hot=True)
    _run(64, n, nw=2, grid=7, hot=True)


def test_with_hosts():
    _run(64, 30_000, hosts=True)
    _run(1000, 9_999, grid=5, hosts=True)
