"""The binding's own decisions, with the library replaced by a recorder (no GPU)."""
import ctypes
import json

import numpy as np
import pytest

import paper_2607_12074_amd as m4


class Recorder:
    """Stands for libm4: every entry point succeeds and keeps its arguments."""

    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append((name, args))
            return m4.M4_OK
        return call


@pytest.fixture
def ctx(monkeypatch):
    rec = Recorder()
    monkeypatch.setattr(m4, "lib", lambda: rec)
    c = m4.Context.__new__(m4.Context)
    c.h, c.device, c.arch = ctypes.c_void_p(1), 0, "gfx950 256 CU"
    c.rec = rec
    yield c
    c.h = None


GRAPH = (np.array([0, 2, 4, 6], np.int64), np.array([1, 2, 0, 2, 0, 1], np.int32))


def test_tunings_of_other_kernels_are_not_reused(ctx, tmp_path):
    # an entry as it was stored before thresholds were keyed by the kernels
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({"gfx950 256 CU/g1.2": {"hub_min": 32, "probe_w": 4}}))
    assert not ctx.autotune(graph=GRAPH, cache=str(cache))["cached"]
    assert "m4_autotune" in [name for name, _ in ctx.rec.calls]
    again = ctx.autotune(graph=GRAPH, cache=str(cache))
    assert again["cached"] and again["hub_min"] != 32
    assert len(json.loads(cache.read_text())) == 2


@pytest.mark.parametrize("asked", [{}, {"stats": True}, {"timing": True}])
def test_statistics_are_computed_when_asked_for(ctx, asked):
    got = ctx.count(*GRAPH, **asked)
    (name, args), = ctx.rec.calls
    assert name == "m4_count_motifs4_ex"
    assert (args[4] is not None) == bool(asked)
    assert got[:1] == ((0,) if not asked else ((0,) * 6,))
