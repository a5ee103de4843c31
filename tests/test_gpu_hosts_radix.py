"""GPU parity of the per-host reduce's radix selection (partitions beyond 2,048
entries): more hosts than its map of 256, so that entries wait for a second and
third batch beside entries already marked with their slot, a host with most of
the flows, and byte counts that entries do not hold.  Whole numbers: tolerance
0 against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1108_1785_amd as gnm
from tests.test_gpu_hosts import _host_records, check, run, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu
REG = ([0x0B000000, 0x0C000000], [8, 8], [0, 1], 2, [0x0A000000], [16])


# 64 partitions up to 185,000 records: hosts of each below, about and far above the map's 256 slots
@pytest.mark.parametrize("hosts,hot", [(64 * 200, 0.0), (64 * 256, 0.0), (64 * 420, 0.0), (64 * 700, 0.3), (900, 0.6),
                                       (3, 0.0)])
def test_batches(torch_cuda, hosts, hot):  # noqa: F811
    say("case: radix selection,", hosts, "hosts, share of one", hot)
    n = 180_000
    rng = np.random.default_rng(hosts)
    remote = (np.where(rng.random(hosts) < 0.5, 0x0B000000, 0x0C000000) | rng.permutation(1 << 18)[:hosts]).astype(np.uint32)
    at = rng.integers(0, hosts, n)
    at[rng.random(n) < hot] = 0
    rec = _host_records(n, remote[at], rng)
    big = rng.random(n) < 0.01
    rec.bytes[big] = rng.choice(np.array([2 ** 61 - 1, 2 ** 61, 2 ** 62, 2 ** 64 - 1], np.uint64), int(big.sum()))
    rec.bytes[rng.random(n) < 0.2] = rec.bytes[0]  # many equal buckets
    reg, orc = gnm.Registry(*REG), oracle.Registry(*REG)
    t, _ = run(reg, rec, 1 << 17)
    check(t, orc, rec)
