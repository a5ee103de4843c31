"""The merge of the partial tables over every number of row tiles about the 8
XCDs (fewer tiles than XCDs, multiples of 8 and beside them), for one window
and for several, with the flags it applies.  Whole numbers: tolerance 0
against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1108_1785_amd as gnm
from tests._gpu import DEV, offsets_to_device, to_device
from tests._helpers import soa

pytestmark = pytest.mark.gpu


# rows = 2 * sites + 3, 8 a tile: 1, 2, 3, 7, 8, 9, 15, 16, 17 and 33 tiles
@pytest.mark.parametrize("n_sites", [1, 3, 7, 25, 30, 31, 57, 62, 63, 130])
@pytest.mark.parametrize("nw", [1, 3])
def test_tiles(n_sites, nw):
    import torch
    print("case: merge,", n_sites, "sites", nw, "windows", flush=True)
    rng = np.random.default_rng(n_sites)
    args = ([0x0B000000 + (s << 12) for s in range(n_sites)], [20] * n_sites, list(range(n_sites)), n_sites,
            [0x0A000000], [16])
    n = 6_000
    remote = 0x0B000000 + (rng.integers(0, n_sites + 1, n) << 12) + rng.integers(0, 4096, n)
    local = 0x0A000000 + rng.integers(0, 1 << 16, n)
    out = rng.random(n) < 0.5
    dur = rng.integers(0, 600_000, n)
    rec = soa([(int(l) if o else int(r), int(r) if o else int(l), int(b), int(p), 7, 7 + int(d))
               for r, l, o, b, p, d in zip(remote, local, out, rng.integers(0, 4_000_000, n),
                                           rng.integers(0, 5000, n), dur)])
    off = None if nw == 1 else np.array([0, n // 5, n // 2, n], dtype=np.uint64)
    reg, orc = gnm.Registry(*args), oracle.Registry(*args)
    exp = np.atleast_3d(orc.classify_aggregate(rec, window_offsets=off)).reshape(nw, reg.rows, 8)
    acc = torch.full((nw, reg.rows, 8), 5, dtype=torch.int64, device=DEV)
    flg = torch.full((nw * n_sites,), 0xAA, dtype=torch.uint8, device=DEV)
    gnm.classify_flag(reg, to_device(rec), acc, flg, threshold_bps=100_000, window_offsets=None if off is None
                      else offsets_to_device(off), n_windows=nw, n=n, workspace=gnm.make_workspace(reg, 9), grid_blocks=9)
    torch.cuda.synchronize()
    assert (gnm.acc_to_numpy(acc).reshape(exp.shape) == exp).all()
    nb, rate = exp[:, :2 * n_sites, 4], exp[:, :2 * n_sites, 5]
    low = (nb >= 1) & (rate // np.maximum(nb, 1) < 100_000)
    assert (flg.cpu().numpy().reshape(nw, n_sites) == (low[:, 0::2] | (low[:, 1::2] << 1))).all()
