"""Launch shapes that the tuner times: every workgroup count once for each number
of records per lane, the automatic launch among them (one workgroup per CU at 4
records per lane on a small registry, two otherwise), and the counts that LDS
allows, half, twice and four times.  Every candidate must leave the oracle's
table."""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from paper_1108_1785_amd import tune
from tests._gpu import DEV, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workload,n", [(flowgen.PLAIN_SMALL, 1_200_000), (flowgen.PLAIN_LARGE, 1_200_000),
                                        (flowgen.PLAIN_SMALL, 100_000)])
def test_each_shape_once(workload, n):
    import torch
    print("case: tuner shapes", workload, n, flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    r = flowgen.registry_for(workload)
    reg, orc = gnm.Registry.from_generated(r), oracle.Registry.from_generated(r)
    per_cu = 2 if reg.info()["lds_bytes"] <= 80 * 1024 else 1
    rec = flowgen.records_for(workload, reg=r, n=n)
    ws = tune.tuning_workspace(reg, device=DEV)
    acc = torch.empty((1, reg.rows, 8), dtype=torch.int64, device=DEV)
    res = gnm.autotune(reg, to_device(rec), acc, reps=1, n=n, workspace=ws)
    torch.cuda.synchronize()
    assert (gnm.acc_to_numpy(acc)[0] == orc.classify_aggregate(rec)).all()
    shapes = {}
    for rpt, grid, _ in res["tried"]:
        shapes.setdefault(rpt, []).append(grid)
    assert sorted(shapes) == [1, 2, 4]
    explicit = [cus * per_cu * k // 2 for k in (1, 2, 4, 8)]
    for rpt, grids in shapes.items():
        tiles = -(-n // (1024 * rpt))
        auto = min(tiles, cus * (1 if rpt == 4 else per_cu))
        if rpt == 4 and per_cu == 2 and tiles < cus:
            auto = min(2 * tiles, cus)  # two workgroups per tile
        assert grids[0] == 0 and sorted(grids[1:]) == [g for g in explicit if g != auto], (rpt, grids, auto)
    if workload == flowgen.PLAIN_SMALL and n > cus * 4096:
        assert [cus if g == 0 else g for g in shapes[4]].count(cus) == 1 and shapes[4].count(2 * cus) == 1
