"""A graph that torch's default stream is still writing when it is passed: the call
has to wait for it, though its own stream does not.  Until the writes the arrays
hold another graph of the same size."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu
N, M = 3000, 20000


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_12074_amd as m4
    c = m4.Context(0)
    yield c
    c.close()


def late(first, then):
    """Device arrays of `first`, overwritten with `then` after some 50 ms of work."""
    import torch
    arrays = [torch.from_numpy(a.copy()).cuda() for a in first]
    after = [torch.from_numpy(a.copy()).cuda() for a in then]
    x = torch.ones(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    for _ in range(40):
        x = x @ x * 1e-4
    for a, b in zip(arrays, after):
        a.copy_(b)
    return arrays


@pytest.mark.parametrize("entry", ["count", "count_noalloc", "edge_triangles", "orbits",
                                   "count_batch"])
@pytest.mark.parametrize("convert", [False, True])
def test_arrays_written_on_the_default_stream(ctx, entry, convert):
    import torch
    import paper_2607_12074_amd as m4
    first, then = gg.gnm(N, M, 1), gg.gnm(N, M, 2)
    if entry == "count_batch":
        first, then = m4.pack_batch([first] * 3), m4.pack_batch([then] * 3)
    want = oracle.closure(*gg.gnm(N, M, 2))
    if convert:  # types that the binding converts, on the same stream
        first = [a.astype(np.int32 if a.dtype == np.int64 else np.int64) for a in first]
        then = [a.astype(np.int32 if a.dtype == np.int64 else np.int64) for a in then]
    else:
        first, then = list(first), list(then)
    got = getattr(ctx, entry)(*late(first, then))
    if entry in ("count", "count_noalloc"):
        assert got == want
    elif entry == "count_batch":
        assert [tuple(int(x) for x in row) for row in got] == [want] * 3
    elif entry == "orbits":
        assert int(got[:, 10].sum()) == 4 * want[5] and int(got[:, 4].sum()) == 4 * want[3]
    else:
        ref = ctx.edge_triangles(*gg.gnm(N, M, 2))
        assert np.array_equal(got.cpu().numpy().view(np.uint32), ref)
    torch.cuda.synchronize()


def test_a_stream_that_is_not_current(ctx):
    import torch
    side = torch.cuda.Stream()
    want = oracle.closure(*gg.gnm(N, M, 2))
    arrays = late(gg.gnm(N, M, 1), gg.gnm(N, M, 2))
    assert ctx.count(*arrays, stream=side.cuda_stream) == want
    side.synchronize()
