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


def on_device(events, handle):
    """A stand-in for a CUDA tensor, and a torch whose current stream has that
    handle; both write what happens to events."""
    class Tensor:
        is_cuda, device = True, "cuda:0"

        def __init__(self, values):
            self.values = np.asarray(values)

        def to(self, dtype):
            events.append("converted")
            return self

        def contiguous(self):
            return self

        def get_device(self):
            return 0

        def numel(self):
            return self.values.size

        def data_ptr(self):
            return self.values.ctypes.data

        def __getitem__(self, at):
            return self

        def __len__(self):
            return self.values.size

    Tensor.__module__ = "torch.stand_in"

    class Stream:
        cuda_stream = handle

        def synchronize(self):
            events.append("waited")
    return Tensor, Stream


@pytest.mark.parametrize("entry", ["count", "count_noalloc", "edge_triangles", "orbits",
                                   "count_batch", "autotune"])
# torch's default stream; a side stream, current; a stream that is not current
@pytest.mark.parametrize("current,given,waits", [(0, None, True), (64, None, False),
                                                 (64, 64, False), (64, 128, True),
                                                 (0, 128, True)])
def test_device_arrays_are_complete_before_the_call(ctx, monkeypatch, entry, current, given,
                                                    waits):
    import torch
    events = []
    Tensor, Stream = on_device(events, current)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream())

    def empty(*shape, **kw):
        events.append("allocated")
        return Tensor(np.zeros(64, np.int64))
    monkeypatch.setattr(torch, "empty", empty)
    lib = m4.lib()
    monkeypatch.setattr(m4, "lib", lambda: lib)
    lib.calls = type("Calls", (list,), {"append": lambda self, x: events.append(x[0])})()
    arrays = [Tensor(a) for a in GRAPH]
    if entry == "count_batch":
        voff, eoff = np.array([0, 3]), np.array([0, 6])
        arrays = [Tensor(voff), Tensor(eoff)] + arrays
    if entry == "autotune":
        if given is not None:
            pytest.skip("takes no stream")
        waits = True  # it runs on the context's stream
        ctx.autotune(graph=arrays)
    else:
        getattr(ctx, entry)(*arrays, stream=given)
    call = events.index({"count": "m4_count_motifs4_ex", "count_noalloc":
                         "m4_count_motifs4_noalloc", "edge_triangles": "m4_edge_triangles",
                         "orbits": "m4_count_orbits4", "count_batch": "m4_count_batch",
                         "autotune": "m4_autotune"}[entry])
    before = events[:call]
    assert ("waited" in before) == waits
    if waits:  # after everything that torch does for the call
        assert before[-1] == "waited"
