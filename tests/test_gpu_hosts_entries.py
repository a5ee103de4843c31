"""Staged per-host entries at the limit of their bytes field: flows just below,
at and far above the bytes that an entry holds beside the row (the launch's
split: fewer bits for more sites), among ordinary ones, through every way a
record reaches the staging (vector tiles, their heads and tails, strided
tiles) and both reduce paths.  Whole numbers: tolerance 0."""
import numpy as np
import pytest

import oracle
import paper_1108_1785_amd as gnm
from tests.test_gpu_hosts import _host_records, check, offsets_to_device, run, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def _row_bits(n_sites):
    return max(1, (2 * n_sites - 1).bit_length())


# rows: 2, 256 and 257 or more of a power of two, 40,000
@pytest.mark.parametrize("n_sites", [1, 128, 129, 20_000])
@pytest.mark.parametrize("n,hosts,rpt,grid", [(9_001, 700, 0, 0), (4_099, 60, 1, 2), (5_003, 300, 2, 3),
                                              (12_000, 2, 4, 1), (7, 3, 0, 0)])
def test_bytes_limit(torch_cuda, n_sites, n, hosts, rpt, grid):  # noqa: F811
    say("case: host entries,", n_sites, "sites", n, "flows", hosts, "hosts", rpt, grid)
    rng = np.random.default_rng(n + n_sites)
    args = ([0x0B000000, 0x0C000000], [8, 8], [0, n_sites - 1], n_sites, [0x0A000000], [16])
    remote = (np.where(rng.random(hosts) < 0.5, 0x0B000000, 0x0C000000) | rng.permutation(1 << 16)[:hosts])
    rec = _host_records(n, remote[rng.integers(0, hosts, n)].astype(np.uint32), rng)
    lim = 1 << (63 - _row_bits(n_sites))
    edge = np.array([lim - 1, lim, lim + 1, 2**64 - 1, 2**63, 2**63 - 1, 1_000_001], dtype=np.uint64)
    i = rng.permutation(n)[: max(3, n // 5)]
    i[:2] = 0, n - 1
    rec.bytes[i] = edge[rng.integers(0, edge.size, i.size)]
    rec.last_ms[i[::7]] = rec.first_ms[i[::7]] - np.uint32(1)  # the longest duration
    off = np.array([0, n // 3 + 1, n // 3 + 1, n], np.uint64) if n > 1_000 and grid == 0 else None
    reg, orc = gnm.Registry(*args), oracle.Registry(*args)
    t, _ = run(reg, rec, 1 << 14, off=off, records_per_thread=rpt, grid_blocks=grid)
    check(t, orc, rec)


@pytest.mark.parametrize("grid", [1, 7, 8, 9, 31, 64, 250, 1023])
def test_workgroup_orders(torch_cuda, grid):  # noqa: F811
    # shares of a partition ordered by workgroup modulo 8: grids below, at and
    # beside multiples of 8, and with more workgroups per wave than it keeps
    say("case: host entries on", grid, "workgroups")
    rng = np.random.default_rng(grid)
    args = ([0x0B000000, 0x0C000000], [8, 8], [0, 1], 2, [0x0A000000], [16])
    remote = (0x0B000000 | rng.integers(0, 4_000, 30_000)).astype(np.uint32)
    rec = _host_records(remote.size, remote, rng)
    t, _ = run(gnm.Registry(*args), rec, 1 << 14, grid_blocks=grid)
    check(t, oracle.Registry(*args), rec)
