"""Automatic launches about the lines of their rule: half-tile workgroups on a
small table (1 to 256 workgroups, the last full of a tile), a workgroup per
tile on a larger one, and work areas that hold one workgroup per tile only,
sized for an explicit count, or sized automatically and used with twice the
automatic count.  Whole numbers: tolerance 0 against the oracle."""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from tests._gpu import DEV, diff, run
from tests.test_gpu_hosts import check as check_hosts
from tests.test_gpu_hosts import run as run_hosts

pytestmark = pytest.mark.gpu
TILE = 4096


@pytest.fixture(scope="module")
def small():
    import torch
    assert torch.cuda.is_available()
    r = flowgen.registry_for(flowgen.PLAIN_SMALL)
    rec = flowgen.records_for(flowgen.PLAIN_SMALL, reg=r, n=260 * TILE)
    return gnm.Registry.from_generated(r), oracle.Registry.from_generated(r), rec


@pytest.mark.parametrize("n", [1, 4, 5, 9, TILE - 1, TILE, TILE + 1, 3 * TILE + 2, 127 * TILE + 1, 128 * TILE,
                               128 * TILE + 1, 255 * TILE, 256 * TILE, 256 * TILE + 1])
def test_small_table(small, n):
    print("case: automatic grid,", n, "records", flush=True)
    reg, orc, rec = small
    part = rec.slice(0, n)
    exp = orc.classify_aggregate(part)
    tiles = -(-n // TILE)
    for ws in (None, gnm.make_workspace(reg), gnm.make_workspace(reg, tiles), gnm.make_workspace(reg, 2 * tiles)):
        got = run(reg, part, workspace=ws)
        assert (got == exp).all(), diff(got, exp)
    off = np.array([0, n // 3, n // 3, n // 2, n], dtype=np.uint64)
    got = run(reg, part, window_offsets=off, workspace=gnm.make_workspace(reg))
    assert (got == orc.classify_aggregate(part, window_offsets=off)).all()


@pytest.mark.parametrize("grid", [0, 1, 25, 50, 512])
def test_host_table_sizes(small, grid):
    print("case: host tables sized for", grid, "workgroups", flush=True)
    reg, orc, rec = small
    part = rec.slice(0, 100_000)
    for used in {grid, 0 if grid in (25, 50) else grid, 512 if grid == 0 else grid}:
        t = gnm.HostTable(reg, 1 << 16, part.n, grid, device=DEV)
        t, acc = run_hosts(reg, part, 0, table=t, grid_blocks=used, workspace=gnm.make_workspace(reg))
        assert (acc[0] == orc.classify_aggregate(part)).all()
        check_hosts(t, orc, part)
