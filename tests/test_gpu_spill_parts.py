"""GPU parity of the spilled table where its parts run full and its entries
reach their limits: a cache of a few rows whose misses all fall in one tile
(the rest of its part's entries go to the device table with atomics), byte
counts around the entries' 38-bit field, many windows per workgroup, and tables
whose last tile is short.  Every value is a whole number: tolerance 0 against
the oracle."""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from tests.test_gpu_spill import call, expect, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def registry(n_sites, **kw):
    """Site s owns 11.x.y.0/24 number s; the local network is 10.0.0.0/16."""
    args = (0x0B000000 + 256 * np.arange(n_sites), [24] * n_sites, np.arange(n_sites), n_sites, [0x0A000000], [16])
    reg = gnm.Registry(*args, **kw)
    assert not reg.info()["acc_in_lds"]
    return reg, oracle.Registry(*args)


def records(rng, site, edge=0.0):
    n = site.size
    remote = (0x0B000000 + 256 * site + rng.integers(0, 256, n)).astype(np.uint32)
    local = (0x0A000000 + rng.integers(0, 1 << 16, n)).astype(np.uint32)
    inbound = rng.random(n) < 0.5
    b = np.clip(np.floor(rng.lognormal(13, 3, n)), 1, 2.0 ** 40).astype(np.uint64)
    e = rng.random(n) < edge
    b[e] = rng.choice(np.array([2 ** 38 - 1, 2 ** 38, 2 ** 38 + 1, 2 ** 40, 2 ** 63, 2 ** 64 - 1], np.uint64), int(e.sum()))
    first = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    return flowgen.Records(src_ip=np.where(inbound, remote, local), dst_ip=np.where(inbound, local, remote),
                           src_port=np.zeros(n, np.uint16), dst_port=np.zeros(n, np.uint16), proto=np.zeros(n, np.uint8),
                           bytes=b, packets=rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32), first_ms=first,
                           last_ms=(first + rng.integers(0, 300_000, n)).astype(np.uint32))


@pytest.mark.parametrize("n_sites,hot,windows,edge,grid,lds",
                         [(2400, 128, 1, 0.0, 0, 33_200), (2400, 128, 3, 0.1, 5, 33_200), (2400, 2400, 700, 0.02, 7, 36_000),
                          (2400, 2400, 1, 0.5, 0, 0), (2431, 2431, 40, 0.0, 64, 0), (3000, 1, 2, 1.0, 1, 33_000)])
def test_parts(torch_cuda, n_sites, hot, windows, edge, grid, lds):  # noqa: F811
    say("case: spilled parts,", n_sites, "sites,", hot, "in use,", windows, "windows, grid", grid, "lds", lds)
    rng = np.random.default_rng(n_sites + hot + windows)
    reg, orc = registry(n_sites, lds_bytes=lds)
    rec = records(rng, rng.integers(0, hot, 150_000), edge)
    off = None
    if windows > 1:
        off = np.concatenate([[0], np.sort(rng.integers(0, rec.n + 1, windows - 1)), [rec.n]]).astype(np.uint64)
    for filters in (None, {"min_avg_packet_bytes": 100, "min_packets": 4, "min_duration_ms": 1000}):
        exp = expect(orc, rec, off, filters=filters)
        _, got, fl = call(reg, rec, off, grid_blocks=grid, filters=filters)
        assert (got == exp).all(), np.argwhere(got != exp)[:5]
        assert (fl == oracle.flags(exp, n_sites)).all()
