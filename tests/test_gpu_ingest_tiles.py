"""GPU parity of the NetFlow v5 decode at the edges of its launch shapes: tiles
of 32 datagrams, the single-launch form (up to 2,048 datagrams), blocks of
1,024 datagrams, and more blocks than a decode workgroup sums itself (4,096).
Every value is a whole number: tolerance 0."""
import numpy as np
import pytest

import flowgen
from oracle import netflow
from tests.test_gpu_ingest import check, gpu_decode, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def datagrams(n, seed):
    """n datagrams, about a tenth malformed, some spans running backwards."""
    rng = np.random.default_rng(seed)
    bad = n // 10
    rec = flowgen.v5_records(flowgen.PLAIN_SMALL, 31 * n + 31, stream=seed)
    buf, off = flowgen.encode_netflow_v5(rec, rng, partial_frac=0.5, malformed=bad)
    off = off[:n + 1].copy()
    if n > 8:
        for d in rng.integers(1, n, size=n // 50 + 1):  # a start before its predecessor's: both spans change
            off[d] = off[int(rng.integers(0, d))]
    return buf, off


@pytest.mark.parametrize("n", [1, 31, 32, 33, 1023, 1024, 1025, 2047, 2048, 2049, 2080, 3073, 5000])
def test_datagram_counts_around_tiles_and_blocks(torch_cuda, n):  # noqa: F811
    say("case: ingest,", n, "datagrams")
    buf, off = datagrams(n, n)
    exp, rej = netflow.decode_netflow_v5(buf, off)
    host, n_rec, n_rej, _ = gpu_decode(buf, off)
    assert (n_rec, n_rej) == (exp["src_ip"].size, rej)
    check(host, exp, n_rec)
    assert all((v[n_rec:] == v.dtype.type(-1 & ((1 << 8 * v.itemsize) - 1))).all() for v in host.values())


@pytest.mark.parametrize("n", [4096 * 1024, 4096 * 1024 + 1, 4096 * 1024 + 2049])
def test_more_blocks_than_a_workgroup_sums(torch_cuda, n):  # noqa: F811
    say("case: ingest,", n, "datagrams of one record")
    rng = np.random.default_rng(n)
    hdr = np.zeros(n, dtype=flowgen.V5_HEADER)
    rec = np.zeros(n, dtype=flowgen.V5_RECORD)
    ok = rng.random(n) < 0.9
    hdr["version"], hdr["count"] = np.where(ok, 5, 9), 1
    names = {"src_ip": "srcaddr", "dst_ip": "dstaddr", "packets": "dPkts", "bytes": "dOctets", "first_ms": "First",
             "last_ms": "Last", "src_port": "srcport", "dst_port": "dstport", "proto": "prot"}
    for f in names.values():
        rec[f] = rng.integers(0, 1 << (8 * rec[f].itemsize), size=n, dtype=np.uint64).astype(rec[f].dtype)
    buf = np.concatenate([hdr.view(np.uint8).reshape(n, 24), rec.view(np.uint8).reshape(n, 48)], axis=1).reshape(-1)
    off = 72 * np.arange(n + 1, dtype=np.uint64)
    host, n_rec, n_rej, _ = gpu_decode(buf, off, capacity=n)
    assert (n_rec, n_rej) == (int(ok.sum()), int((~ok).sum()))
    check(host, {k: rec[f][ok].astype(host[k].dtype) for k, f in names.items()}, n_rec)
