"""The vector path whose byte counts are loaded by whole lines and exchanged
between a wave's halves: tables beyond LDS at any length (tile, wave and
half-wave edges, arrays cut at every element of a 16-byte word), and tables in
LDS from 2^24 records on (both sides of that line, with windows that end
anywhere).  Every record's byte count is different, so that one exchanged wrongly
shows.  Whole numbers: tolerance 0 against the oracle."""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from tests._gpu import diff, run

pytestmark = pytest.mark.gpu


def _records(reg, workload, n, seed):
    rec = flowgen.records_for(workload, reg=reg, n=min(n, 1 << 20))
    while rec.n < n:
        rec = flowgen.concat([rec, rec.slice(0, min(rec.n, n - rec.n))])
    rec.bytes[:] = np.random.default_rng(seed).permutation(n).astype(np.uint64) * np.uint64(977) + np.uint64(1)
    return rec


@pytest.fixture(scope="module")
def table():
    import torch
    assert torch.cuda.is_available()
    r = flowgen.registry_for(flowgen.LARGE_TABLE)
    reg = gnm.Registry.from_generated(r)
    assert not reg.info()["acc_in_lds"] and reg.info()["n_nodes"] > 0
    return reg, oracle.Registry.from_generated(r), _records(r, flowgen.LARGE_TABLE, 40_000, 1)


@pytest.mark.parametrize("n", [4, 8, 124, 128, 132, 252, 256, 260, 384, 3968, 4096, 4100, 8191, 39_997])
def test_table_beyond_lds(table, n):
    print("case: byte counts by whole lines,", n, "records", flush=True)
    reg, orc, rec = table
    part = rec.slice(0, n)
    exp = orc.classify_aggregate(part)
    for shift in (0, 1, 2, 3):
        for grid in (0, 1, 3):
            ws = gnm.make_workspace(reg, grid, n_records=n)
            got = run(reg, part, workspace=ws, shift=shift, grid_blocks=grid)
            assert (got == exp).all(), (shift, grid, diff(got, exp))
    off = np.array([0, n // 3, n // 3, n - n // 4, n], dtype=np.uint64)
    got = run(reg, part, window_offsets=off, workspace=gnm.make_workspace(reg, n_records=n, n_windows=4))
    assert (got == orc.classify_aggregate(part, window_offsets=off)).all()


def test_long_arrays():
    n = 1 << 24
    r = flowgen.registry_for(flowgen.PLAIN_LARGE)
    reg, orc = gnm.Registry.from_generated(r), oracle.Registry.from_generated(r)
    assert reg.info()["acc_in_lds"] and reg.info()["n_nodes"] > 0
    rec = _records(r, flowgen.PLAIN_LARGE, n + 5, 2)
    cuts = np.sort(np.random.default_rng(3).integers(0, n, 200))
    for m, shift in ((n - 1, 0), (n, 0), (n + 5, 0), (n + 1, 3)):
        print("case: long arrays,", m, "records, shift", shift, flush=True)
        part = rec.slice(0, m)
        got = run(reg, part, workspace=gnm.make_workspace(reg), shift=shift)
        assert (got == orc.classify_aggregate(part)).all(), (m, shift)
    off = np.concatenate([[0], cuts, [n + 5]]).astype(np.uint64)
    got = run(reg, rec, window_offsets=off, workspace=gnm.make_workspace(reg))
    assert (got == orc.classify_aggregate(rec, window_offsets=off)).all()
