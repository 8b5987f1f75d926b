"""Small graphs (up to 8192 vertices) are prepared and planned by fused kernels;
the same graph with isolated vertices beyond that takes the general path, and
everything it returns must be equal, at the edges of both: one vertex more,
rows around 256 entries and over the whole graph, out-degrees beyond the LDS
classes, hub tables, isolated vertices, checked input."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from tests import graphs as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_12074_amd as m4
    c = m4.Context(0)
    yield c
    c.close()


def pad(g, n):
    rp = np.asarray(g[0], dtype=np.int64)
    return np.concatenate([rp, np.full(n + 1 - len(rp), rp[-1], np.int64)]), g[1]


def hubs(n, m, seed, rows):
    """A random graph with vertices of exactly the given degrees joined in."""
    rng = np.random.default_rng(seed)
    e = [rng.integers(0, n, (m, 2))]
    for i, d in enumerate(rows):
        to = rng.choice(n, d, replace=False)
        e.append(np.stack([np.full(d, n + i), to], 1))
    e = np.concatenate(e)
    return gg.from_edges(n + len(rows), e[:, 0].astype(np.int32), e[:, 1].astype(np.int32))


CASES = [
    ("n=4", lambda: G.cycle(4)),
    ("n=63", lambda: gg.gnm(63, 300, 1)),
    ("n=64", lambda: gg.gnm(64, 300, 2)),
    ("n=65", lambda: gg.gnm(65, 300, 3)),
    ("n=1024", lambda: gg.gnm(1024, 9000, 4)),
    ("n=1025", lambda: gg.gnm(1025, 9000, 5)),
    ("n=8191", lambda: gg.gnm(8191, 30000, 6)),
    ("n=8192", lambda: gg.gnm(8192, 60000, 7)),
    ("long rows", lambda: hubs(3000, 9000, 8, [127, 128, 255, 256, 257, 300, 2999])),
    ("star", lambda: G.star(8191)),
    ("wheel", lambda: G.wheel(8000)),
    ("hub tables", lambda: gg.gnm(700, 150000, 9)),
    ("power law", lambda: gg.rmat(12, 12, 0.57, 0.19, 0.19, 10)),
    ("path and isolated", lambda: pad(G.path(50), 4000)),
    ("beyond the LDS classes", lambda: G.complete_bipartite(1030, 1040)),
    ("bipartite", lambda: G.complete_bipartite(300, 700)),
]


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_equals_the_general_path(ctx, name, make):
    import paper_2607_12074_amd as m4
    g = make()
    n = len(g[0]) - 1
    big = pad(g, 9000)
    want = oracle.closure(*g)
    got, st = ctx.count(*g, stats=True)
    gen, sg = ctx.count(*big, stats=True)
    assert got == gen == want
    for k in ("cost_wedge", "wedges", "cache_hits"):
        if k == "cost_wedge" or st["basis_used"] == sg["basis_used"]:
            assert st[k] == sg[k], k
    for flags in (m4.M4_BASIS_WEDGE, m4.M4_VALIDATE, m4.M4_NO_CACHE):
        assert ctx.count(*g, flags=flags) == want
    assert np.array_equal(ctx.edge_triangles(*g), ctx.edge_triangles(*big))
    assert (ctx.orbits(*g) == ctx.orbits(*big)[:n]).all()


@pytest.mark.parametrize("n", [8192, 8193])
def test_edge_basis_on_both_sides(ctx, n):
    import paper_2607_12074_amd as m4
    g = gg.gnm(n, 12000, 3)
    assert ctx.count(*g, flags=m4.M4_BASIS_EDGE) == oracle.closure(*g)


def test_checked_input_is_refused(ctx):
    import paper_2607_12074_amd as m4
    rp, col = gg.gnm(500, 2000, 1)
    bad = np.array(col)
    bad[0], bad[1] = bad[1], bad[0]  # unsorted row
    with pytest.raises(m4.M4Error):
        ctx.count(rp, bad, flags=m4.M4_VALIDATE)
    with pytest.raises(m4.M4Error):
        ctx.orbits(rp, bad, flags=m4.M4_VALIDATE)
    assert ctx.count(rp, col, flags=m4.M4_VALIDATE) == oracle.closure(rp, col)
