"""GPU parity of the spilled table where tiles run out of their parts and take
chunks: neighbouring sites of a wide table (one, several and many tiles of every
width, the last one short), windows that share chunks, workgroups with many
windows, a range whose chunks are used up as well, histograms and hosts in the
same pass.  Whole numbers: tolerance 0 against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1108_1785_amd as gnm
from tests.test_gpu_spill import call, expect, say, torch_cuda  # noqa: F401
from tests.test_gpu_spill_parts import records, registry

pytestmark = pytest.mark.gpu
_R = {}


def cached(n_sites, **kw):
    key = (n_sites,) + tuple(sorted(kw.items()))
    if key not in _R:
        _R.clear()
        _R[key] = registry(n_sites, **kw)
    return _R[key]


def check(reg, orc, rec, off, **kw):
    exp = expect(orc, rec, off)
    _, got, fl = call(reg, rec, off, **kw)
    assert (got == exp).all(), np.argwhere(got != exp)[:5]
    assert (fl == oracle.flags(exp, reg.n_sites)).all()


def cut(rng, n, windows):
    if windows == 1:
        return None
    return np.concatenate([[0], np.sort(rng.integers(0, n + 1, windows - 1)), [n]]).astype(np.uint64)


# (sites, first site in use, sites in use, windows, workgroups)
@pytest.mark.parametrize("n_sites,first,hot,windows,grid", [
    (20_000, 3_000, 500, 1, 0), (20_000, 3_000, 2_000, 1, 7), (20_000, 19_400, 600, 20, 3), (20_000, 100, 1_500, 100, 1),
    (20_000, 0, 20_000, 1, 2),
    (140_000, 255, 2, 1, 0), (140_000, 138_000, 2_000, 1, 11), (140_000, 70_000, 3_000, 12, 2),  # tiles of 512 rows
    (400_000, 398_976, 1_024, 1, 9), (400_000, 1_000, 4_000, 5, 3),                              # of 1,024
    (1_100_000, 1_098_000, 2_000, 1, 5), (1_100_000, 0, 1_100_000, 1, 0)])                       # of 2,048
def test_neighbours(torch_cuda, n_sites, first, hot, windows, grid):  # noqa: F811
    say("case: spilled chunks,", n_sites, "sites,", hot, "in use from", first, ",", windows, "windows, grid", grid)
    rng = np.random.default_rng(n_sites + hot + windows + grid)
    reg, orc = cached(n_sites)
    rec = records(rng, first + rng.integers(0, hot, 120_000), 0.01)
    check(reg, orc, rec, cut(rng, rec.n, windows), grid_blocks=grid)


# a cache of 8 rows, so that nearly every record is an entry; a plan without room beside the cache; flushes
# after every 16 records, whose 7 words a row use up the chunks as well
@pytest.mark.parametrize("hot,windows,grid,lds,flush", [
    (130, 1, 4, 33_400, 0), (3_000, 3, 2, 33_400, 0), (3_000, 60, 1, 33_400, 0), (130, 1, 0, 33_400, 500),
    (40, 1, 64, 163_840, 0), (3_000, 1, 1, 163_840, 16), (1_000, 3, 2, 163_840, 16)])
def test_small_cache(torch_cuda, hot, windows, grid, lds, flush):  # noqa: F811
    say("case: spilled chunks,", hot, "in use,", windows, "windows, grid", grid, "lds", lds, "flush", flush)
    rng = np.random.default_rng(hot + windows + grid)
    reg, orc = cached(3_000, lds_bytes=lds)
    rec = records(rng, rng.integers(0, hot, 100_000), 0.02)
    off = cut(rng, rec.n, windows)
    check(reg, orc, rec, off, grid_blocks=grid, flush_records=flush)
    acc0 = expect(orc, rec, off)
    import torch
    acc = torch.from_numpy(acc0.view(np.int64).copy()).to("cuda:0").reshape(-1, reg.rows, 8)
    _, got, _ = call(reg, rec, off, grid_blocks=grid, acc=acc, accumulate=True, flush_records=flush)
    two = np.concatenate([acc0[..., :6] * np.uint64(2), acc0[..., 6:]], axis=-1)
    assert (got == two).all(), np.argwhere(got != two)[:5]


def test_with_histograms_and_hosts(torch_cuda):  # noqa: F811
    import torch
    from tests._gpu import DEV, to_device
    from tests.test_gpu_hosts import check as check_hosts
    rng = np.random.default_rng(5)
    reg, orc = cached(3_000)
    rec = records(rng, 1_000 + rng.integers(0, 700, 60_000))
    say("case: spilled chunks with histograms and hosts")
    hist = gnm.make_rate_hist(reg, 1)
    table = gnm.HostTable(reg, 2 * rec.n, rec.n, 3, device=DEV)
    acc = torch.empty((1, reg.rows, 8), dtype=torch.int64, device=DEV)
    gnm.classify_aggregate(reg, to_device(rec), acc, grid_blocks=3, rate_hist=hist, hosts=table,
                           workspace=gnm.make_workspace(reg, 3, n_records=rec.n, hist=True))
    torch.cuda.synchronize()
    assert (gnm.acc_to_numpy(acc)[0] == orc.classify_aggregate(rec)).all()
    exp = oracle.rate_histograms(orc, rec)[0, :2 * reg.n_sites]
    assert (hist.cpu().numpy().view(np.uint32).reshape(exp.shape) == exp).all()
    check_hosts(table, orc, rec)
