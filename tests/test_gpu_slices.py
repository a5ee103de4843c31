"""GPU parity at the edges of the workgroups' slices (an even split of the
records cut at multiples of 4): fewer records than workgroups, slices that
differ by a few records, arrays cut at any element, and a flush limit at the
length of the even split.  Every value is a whole number: tolerance 0."""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from tests._gpu import diff, run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    assert torch.cuda.is_available()
    r = flowgen.registry_for(flowgen.PLAIN_SMALL)
    rec = flowgen.records_for(flowgen.PLAIN_SMALL, reg=r, n=9000)
    return gnm.Registry.from_generated(r), oracle.Registry.from_generated(r), rec


@pytest.mark.parametrize("n", [1, 3, 4, 5, 7, 13, 1023, 4095, 4097, 8190])
@pytest.mark.parametrize("grid", [1, 2, 3, 7, 64])
def test_slices(setup, n, grid):
    print("case: slices,", n, "records on", grid, "workgroups", flush=True)
    reg, orc, rec = setup
    for shift in (0, 1, 2, 3):
        part = rec.slice(0, n)
        if shift > n:
            continue
        exp = orc.classify_aggregate(part)
        ws = gnm.make_workspace(reg, grid)
        for flush in (0, -(-n // grid), -(-n // grid) + 3):
            for rpt in (4, 1):
                got = run(reg, part, grid_blocks=grid, records_per_thread=rpt, workspace=ws, shift=shift,
                          flush_records=flush)
                assert (got == exp).all(), (shift, flush, rpt, diff(got, exp))
    off = np.array([0, n // 3, n // 3, n // 2, n], dtype=np.uint64)
    got = run(reg, part, window_offsets=off, grid_blocks=grid, workspace=ws)
    assert (got == orc.classify_aggregate(part, window_offsets=off)).all()
