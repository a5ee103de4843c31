"""CPU-only: a tuning cache written before the launch rules changed is not
believed.  Its keys lack the launch revision, so the workload is timed again and
stored under a key of its own, which the next call then finds."""
import json

import numpy as np

import paper_1108_1785_amd as gnm
from paper_1108_1785_amd import tune


def test_older_winners_are_timed_again(tmp_path, monkeypatch):
    reg = gnm.Registry([0x0B000000], [24], [0], 1, [0x0A000000], [16], host_only=True)
    monkeypatch.setattr(tune, "_device_name", lambda: "card/gfx950/256")
    timed = []

    def autotune(reg, rec, acc, **kw):
        timed.append(kw["n"])
        return {"records_per_thread": 4, "grid_blocks": 0, "best_ms": 1.0, "tried": []}

    monkeypatch.setattr(tune, "autotune", autotune)
    i = reg.info()
    shape = "p%d-s%d-r%d-l%d-li%d-ai%d" % (i["n_prefixes"], i["n_sites"], i["root_bits"], i["list_max"],
                                          i["lines_in_lds"], i["acc_in_lds"])
    old = "card/gfx950/256|%s|%s|n2^10|w2^0|atomic" % (gnm.version(), shape)
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({old: {"records_per_thread": 1, "grid_blocks": 2048, "best_ms": 0.5, "tried": []}}))
    rec = {"src_ip": np.zeros(1024)}
    first = tune.tuned_params(reg, rec, None, n=1024, cache_path=str(path))
    assert timed == [1024] and not first["cached"] and first["records_per_thread"] == 4
    again = tune.tuned_params(reg, rec, None, n=1024, cache_path=str(path))
    assert timed == [1024] and again["cached"] and again["records_per_thread"] == 4
    assert old in json.loads(path.read_text())  # an older library may still use its own
