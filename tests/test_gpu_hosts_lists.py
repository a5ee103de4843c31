"""GPU parity of the per-host reduce at the edges of its paths: hosts whose
flow count sits at the ranked lists' limit (256), around their words' place
field (512) and around the largest partition kept in LDS (2,048 entries), and
partitions at the map's 512 hosts.  Every value is a whole number: tolerance
0 against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1108_1785_amd as gnm
from tests.test_gpu_hosts import _host_records, check, run, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu
REG = ([0x0B000000, 0x0C000000], [8, 8], [0, 1], 2, [0x0A000000], [16])


@pytest.mark.parametrize("flows", [1, 2, 3, 4, 5, 255, 256, 257, 511, 512, 513, 1023, 1025, 2046, 2048, 2049, 4100])
def test_flows_per_host(torch_cuda, flows):  # noqa: F811
    say("case: hosts of", flows, "flows each")
    rng = np.random.default_rng(flows)
    hosts = max(2, min(300, 12_000 // flows))
    remote = 0x0B000000 | rng.permutation(1 << 16)[:hosts]
    remote = rng.permutation(np.concatenate([np.repeat(remote, flows), 0x0C000000 | rng.integers(0, 1 << 24, 700)]))
    rec = _host_records(remote.size, remote.astype(np.uint32), rng)
    rec.bytes[: remote.size // 2] = rec.bytes[0]  # many equal buckets
    reg, orc = gnm.Registry(*REG), oracle.Registry(*REG)
    t, _ = run(reg, rec, 1 << 14)
    check(t, orc, rec)


@pytest.mark.parametrize("hosts", [64 * 505, 64 * 512, 64 * 530])
def test_hosts_per_partition(torch_cuda, hosts):  # noqa: F811
    # 64 partitions up to 185,000 records: on average at the map's 512 slots
    say("case:", hosts, "hosts in 64 partitions")
    rng = np.random.default_rng(hosts)
    remote = (0x0C000000 | rng.permutation(1 << 22)[:hosts]).astype(np.uint32)
    rec = _host_records(hosts, remote, rng)
    reg, orc = gnm.Registry(*REG), oracle.Registry(*REG)
    t, _ = run(reg, rec, 1 << 16)
    check(t, orc, rec)
