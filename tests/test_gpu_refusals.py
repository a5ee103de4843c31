"""Work areas that a call refuses: sized against the most workgroups that an
automatic launch is documented to use (as many per CU as LDS allows), however
many the present launch starts.  A host table's buffer and the static scratch
that are too small for those are refused with GNM_E_INVAL, those that hold them
are accepted; nothing is enqueued by a refused call."""
import numpy as np
import pytest

import flowgen
import oracle
import paper_1108_1785_amd as gnm
from tests._gpu import DEV, to_device

pytestmark = pytest.mark.gpu


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def test_host_buffer_of_a_long_run():
    import torch
    r = flowgen.registry_for(flowgen.PLAIN_SMALL)
    reg = gnm.Registry.from_generated(r)
    assert reg.info()["lds_bytes"] <= 80 * 1024  # two workgroups per CU
    cus = _cus()
    n = (cus + 44) * 4096  # a tile each for more workgroups than CUs
    rec = flowgen.records_for(flowgen.PLAIN_SMALL, reg=r, n=100_000)
    d = {f: t.repeat(-(-n // rec.n))[:n].contiguous() for f, t in to_device(rec).items()}
    acc = torch.full((1, reg.rows, 8), 7, dtype=torch.int64, device=DEV)
    small = gnm.HostTable(reg, 1 << 18, n, cus, device=DEV)
    small.keys.fill_(5)
    with pytest.raises(gnm.GnmError) as e:
        gnm.classify_aggregate(reg, d, acc, n=n, hosts=small)
    assert e.value.code == gnm.GNM_E_INVAL and "host table" in str(e.value)
    torch.cuda.synchronize()
    assert (acc == 7).all() and (small.keys == 5).all()
    for table, grid in ((gnm.HostTable(reg, 1 << 18, n, cus + 44, device=DEV), 0), (small, cus)):
        gnm.classify_aggregate(reg, d, acc, n=n, hosts=table, grid_blocks=grid)
        torch.cuda.synchronize()
        assert int(acc[0, :, 0].sum()) == n


def test_static_scratch_of_a_long_run():
    import torch
    sites = 640  # 512 tables of 1,283 rows pass 32 MiB, 256 do not
    args = (0x0B000000 + 256 * np.arange(sites), [24] * sites, np.arange(sites), sites, [0x0A000000], [16])
    reg = gnm.Registry(*args, root_bits=8)
    cus = _cus()
    assert reg.info()["acc_in_lds"] and reg.info()["lds_bytes"] <= 80 * 1024
    assert gnm.workspace_bytes(reg, 2 * cus) > gnm.static_scratch_bytes() > gnm.workspace_bytes(reg, cus)
    n = 2 * cus * 4096
    rng = np.random.default_rng(3)
    part = flowgen.Records(*(np.zeros(4096, t) for t in (np.uint32, np.uint32, np.uint16, np.uint16, np.uint8, np.uint64,
                                                         np.uint32, np.uint32, np.uint32)))
    part.src_ip[:] = 0x0B000000 + 256 * rng.integers(0, sites, 4096)
    part.dst_ip[:] = 0x0A000001
    part.bytes[:] = rng.integers(1, 1 << 30, 4096)
    part.last_ms[:] = 100
    d = {f: t.repeat(2 * cus) for f, t in to_device(part).items()}
    acc = torch.full((1, reg.rows, 8), 7, dtype=torch.int64, device=DEV)
    fl = torch.full((sites,), 9, dtype=torch.uint8, device=DEV)
    with pytest.raises(gnm.GnmError) as e:
        gnm.classify_flag_static(reg, d, acc, fl, n=n)
    assert e.value.code == gnm.GNM_E_INVAL and "static scratch" in str(e.value)
    torch.cuda.synchronize()
    assert (acc == 7).all() and (fl == 9).all()
    gnm.classify_flag_static(reg, d, acc, fl, n=n, grid_blocks=cus)
    torch.cuda.synchronize()
    exp = oracle.Registry(*args).classify_aggregate(part)
    got = gnm.acc_to_numpy(acc)[0]
    assert (got[:, :6] == exp[:, :6] * np.uint64(2 * cus)).all() and (got[:, 6:] == exp[:, 6:]).all()
