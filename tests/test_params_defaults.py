"""CPU-only: what no argument of make_params names is the library's default, as
gnm_params_default() gives it, not a copy of it in the binding; the filters, the
flush and the launch shape are as given, or off and automatic."""
import ctypes

import paper_1108_1785_amd as gnm


def test_defaults_come_from_the_library(monkeypatch):
    real = ctypes.CDLL(gnm.LIB_PATH)

    class Other:
        """The library with other defaults."""

        def __init__(self, path, *a, **kw):
            pass

        def __getattr__(self, name):
            if name != "gnm_params_default":
                return getattr(real, name)

            class Default:
                restype = argtypes = None

                def __call__(self):
                    p = gnm.Params()
                    p.bulk_bytes, p.records_per_thread, p.min_packets, p.reserved2 = 5, 2, 7, 11
                    return p

            f = Default()
            object.__setattr__(self, name, f)
            return f

    monkeypatch.setattr(ctypes, "CDLL", Other)
    monkeypatch.setattr(gnm, "_lib", None)
    monkeypatch.setattr(gnm, "_defaults", b"", raising=False)
    p = gnm.make_params()
    assert p.reserved2 == 11  # no argument names it
    assert (p.bulk_bytes, p.records_per_thread, p.min_packets) == (1_000_000, 0, 0)
    p = gnm.make_params(filters={"min_packets": 3}, grid_blocks=9)
    assert (p.reserved2, p.min_packets, p.grid_blocks, p.bulk_bytes) == (11, 3, 9, 1_000_000)


def test_given_parameters():
    d = gnm.lib().gnm_params_default()
    p = gnm.make_params()
    assert bytes(p) == bytes(d)
    p = gnm.make_params(bulk_bytes=2**63, accumulate=True, records_per_thread=2, grid_blocks=5, flush_records=9,
                        filters={"min_duration_ms": 4})
    assert (p.bulk_bytes, p.flags, p.records_per_thread, p.grid_blocks, p.flush_records, p.min_duration_ms) == \
        (2**63, 1, 2, 5, 9, 4)
    assert (p.workspace, p.rate_hist, p.min_packets, p.min_avg_packet_bytes) == (None, None, 0, 0)
