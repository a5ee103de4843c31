"""The median kernel's two shapes and the two-window rule it applies itself.

A wave per batch of buckets up to one (window, site) item per CU, four waves
beyond; one window's warning bits come from the median kernel, several
windows' (or a previous window held in an array the call writes) from the
second kernel.  Whole numbers throughout: every median and flag byte must
equal the oracle's (tolerance 0), from histograms drawn here: empty rows, one
count in the first or the last bucket, counts on both sides of a batch's
edge, and counts beyond 32 bits in sum.
"""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from tests._gpu import DEV

pytestmark = pytest.mark.gpu


def _hist(rng, items):
    """Histogram rows [2 * items, BUCKETS] with the medians on chosen edges."""
    B = gnm.RATE_BUCKETS
    h = np.zeros((2 * items, B), np.uint32)
    for r in range(2 * items):
        kind = r % 7
        if kind == 1:
            h[r, 0] = 1
        elif kind == 2:
            h[r, B - 1] = 1
        elif kind == 3:  # the two sides of a batch's edge, and of a lane's run
            e = 1024 * int(rng.integers(1, (B - 1) // 1024 + 1))
            h[r, e - 1], h[r, e] = rng.integers(1, 4, 2)
        elif kind == 4:
            h[r, rng.integers(0, B, 300)] = 0xFFFFFFFF
        elif kind == 5:
            h[r] = rng.integers(0, 3, B)
        elif kind == 6:
            h[r, rng.integers(0, B, 5)] = rng.integers(1, 1 << 20, 5)
    return h


def _expect(h, nw, S, threshold, need, prev):
    cum = np.cumsum(h.astype(np.uint64), axis=1)
    n = cum[:, -1]
    med = np.where(n == 0, 0xFFFFFFFF, (cum < (n - n // 2)[:, None]).sum(axis=1)).astype(np.uint32)
    return med, oracle.median_flags(med.reshape(nw, 2 * S), n.reshape(nw, 2 * S), S, threshold, need, prev)


# 64 sites: 64 items; 256 and 320, about the line; 1,000 sites: one window of
# 1,000 items, and 4, whose histograms are larger than the memory cache
@pytest.mark.parametrize("sites,nw", [(64, 1), (64, 4), (64, 5), (1000, 1), (1000, 4)])
@pytest.mark.parametrize("prev_kind", ["none", "apart", "in flags", "in medians"])
def test_median_shapes(sites, nw, prev_kind):
    import torch
    print("case: median shapes", sites, nw, prev_kind, flush=True)
    rng = np.random.default_rng(sites + nw)
    w = flowgen.PLAIN_SMALL if sites == 64 else flowgen.PLAIN_LARGE
    reg = gnm.Registry.from_generated(flowgen.registry_for(w))
    S = reg.n_sites
    assert S == sites
    h = _hist(rng, nw * S)
    threshold, need = 10_240_000, 2  # bucket 1024: a batch's edge
    prev = rng.integers(0, 16, S).astype(np.uint8)
    d = torch.from_numpy(h.view(np.int32)).to(DEV)
    med = torch.full((nw * 2 * S,), 7, dtype=torch.int32, device=DEV)
    flg = torch.full((nw * S,), 0xAA, dtype=torch.uint8, device=DEV)
    pt = torch.from_numpy(prev).to(DEV)
    em, ef = _expect(h, nw, S, threshold, need, prev if prev_kind == "apart" else None)
    if prev_kind == "none":
        pt = None
    elif prev_kind == "in flags":
        # written before the rule reads it: the previous window is this call's first
        pt = flg[:S]
        first = ef[0] & 3
        ef = _expect(h, nw, S, threshold, need, first)[1]
    elif prev_kind == "in medians":
        pt = med.view(torch.uint8)[:S]
        ef = _expect(h, nw, S, threshold, need, em.view(np.uint8)[:S])[1]
    gnm.median_flags(reg, d, nw, flg, threshold, need, prev_flags=pt, median_bucket=med)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(med.cpu().numpy().view(np.uint32), em)
    np.testing.assert_array_equal(flg.cpu().numpy().reshape(nw, S), ef)
