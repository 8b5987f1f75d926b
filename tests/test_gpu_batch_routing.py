"""Arenas with graphs that the fused kernel passes over (no edges, fewer than
four vertices, degrees or work beyond its LDS structures), alone, in runs and
between others, in both variants, replayed with other contents, and through the
server."""
from math import comb

import numpy as np
import pytest

import graphgen as gg
import oracle
from tests import graphs as G
from tests.test_gpu_serve import _collect
from tests.test_oracle_pins import CLOSED, cf_wheel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_12074_amd as m4
    c = m4.Context(0)
    yield c
    c.close()


def rows(out):
    return [tuple(int(x) for x in row) for row in out]


EMPTY = lambda: (G.csr(5, []), (0,) * 6)
TINY = lambda: (G.complete(3), (0,) * 6)
STAR = lambda: (G.star(999), (comb(999, 3), 0, 0, 0, 0, 0))  # degree beyond both variants
K40 = lambda: (G.complete(40), (0, 0, 0, 0, 0, comb(40, 4)))


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("kinds", [[EMPTY], [TINY], [STAR], [EMPTY, K40], [K40, STAR, TINY],
                                   [STAR] * 3 + [K40]],
                         ids=["empty", "tiny", "star", "empty,K40", "K40,star,tiny", "stars,K40"])
@pytest.mark.parametrize("times", [1, 700])
def test_passed_over(ctx, variant, kinds, times):
    import paper_2607_12074_amd as m4
    if times > 1 and STAR in kinds:
        times = 40  # each star is a call of its own
    made = [k() for k in kinds] * times
    ctx.set_tuning(batch_variant=variant)
    try:
        out = ctx.count_batch(*m4.pack_batch([g for g, _ in made]))
    finally:
        ctx.set_tuning(batch_variant=0)
    assert rows(out) == [want for _, want in made]


def test_closed_forms(ctx):
    import paper_2607_12074_amd as m4
    graphs = [make() for _, make, _ in CLOSED]
    want = [tuple(e) for _, _, e in CLOSED]
    graphs += [G.wheel(3000), G.complete(900), G.complete_bipartite(4, 2000), G.csr(5, [])]
    want += [cf_wheel(3000), (0, 0, 0, 0, 0, comb(900, 4)),
             (4 * comb(2000, 3) + 2000 * comb(4, 3), 0, 0, comb(4, 2) * comb(2000, 2), 0, 0),
             (0,) * 6]
    assert rows(ctx.count_batch(*m4.pack_batch(graphs))) == want


def test_replayed_with_other_contents(ctx):
    # the same offsets: a graph becomes too large for the kernel and back
    import paper_2607_12074_amd as m4
    rest = [gg.batch_graph(i, seed=21) for i in range(30)]
    first = [gg.gnm(1000, 999, 3), gg.gnm(40, 780, 4)] + rest
    second = [G.star(999), G.complete(40)] + rest
    arena, other = m4.pack_batch(first), m4.pack_batch(second)
    assert np.array_equal(arena[0], other[0]) and np.array_equal(arena[1], other[1])
    ref = [oracle.closure(*g) for g in first]
    ref2 = [STAR()[1], K40()[1]] + ref[2:]
    rp, col = arena[2].copy(), arena[3].copy()
    for contents, want in ((arena, ref), (other, ref2), (arena, ref), (other, ref2)):
        rp[:], col[:] = contents[2], contents[3]
        assert rows(ctx.count_batch(arena[0], arena[1], rp, col)) == want
        assert ctx.count(*first[2]) == ref[2]  # eager work between the replays


def test_server_of_small_and_empty_requests(ctx):
    import paper_2607_12074_amd as m4
    made = [k() for k in (EMPTY, TINY, K40, STAR)] * 20
    srv = m4.Server(ctx, 256 << 20)
    ids = {srv.submit(*g, tag=i): i for i, (g, _) in enumerate(made)}
    res = _collect(srv, len(made), timeout=60.0)
    srv.close()
    for rid, r in res.items():
        assert r["status"] == 0 and r["counts"] == made[ids[rid]][1], ids[rid]
