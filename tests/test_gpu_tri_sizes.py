"""Triangle owners at the edges of the out-degree classes (16, 64, 128, 256, 512):
a clique has one owner of every out-degree below its size, and beside it a
random graph gives owners whose lists hold other vertices too.  Counts against
the oracle, per-vertex orbits and per-edge triangles against closed forms, with
the lists read, with every list probed through hub tables, and in between."""
from math import comb

import numpy as np
import pytest

import graphgen as gg
import oracle
from tests import graphs as G
from tests.test_oracle_orbits import cf_complete

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_12074_amd as m4
    c = m4.Context(0)
    yield c
    c.close()


HUBS = [dict(hub_min=0), dict(hub_min=4, probe_w=1, probe_w_far=1), dict(hub_min=4, probe_w=8)]


@pytest.mark.parametrize("n", [3, 16, 17, 18, 65, 66, 129, 130, 257, 258, 513, 514])
def test_cliques_beside_a_random_graph(ctx, n):
    rnd = gg.gnm(400, 9000, n)  # out-degrees around 25 in lists of about 45
    ref = oracle.closure(*rnd)
    ref_orb = oracle.orbits_esu(*rnd)
    g = G.disjoint_union(G.complete(n), rnd)
    base = ctx.get_tuning()
    try:
        for hubs in HUBS:
            ctx.set_tuning(**hubs)
            got = ctx.count(*g)
            assert got == ref[:5] + (ref[5] + comb(n, 4),), hubs
            t = ctx.edge_triangles(*g)
            assert (t[:n * (n - 1)] == n - 2).all(), hubs
            orb = ctx.orbits(*g)
            assert (orb[:n] == cf_complete(n)).all(), hubs
            assert (orb[n:] == ref_orb).all(), hubs
    finally:
        ctx.set_tuning(**base)


# sparse owners among long lists: most elements read belong to no triangle
@pytest.mark.parametrize("n,m", [(3000, 30000), (2000, 100000), (900, 150000)])
@pytest.mark.parametrize("hubs", HUBS, ids=["scan", "probe", "mixed"])
def test_random_graphs(ctx, n, m, hubs):
    g = gg.gnm(n, m, n + m)
    src = np.repeat(np.arange(n), np.diff(g[0]))
    A = G.adjacency(g)
    base = ctx.get_tuning()
    try:
        ctx.set_tuning(**hubs)
        assert ctx.count(*g) == oracle.closure(*g)
        assert np.array_equal(ctx.edge_triangles(*g), (A @ A)[src, g[1]])
    finally:
        ctx.set_tuning(**base)


# owners of one wavefront dealt in turn, and in runs from the work counter (from
# 262144 owners on); without the cache none of them takes the register kernel
@pytest.mark.parametrize("n", [150000, 300001])
def test_dealing(ctx, n):
    import paper_2607_12074_amd as m4
    g = gg.gnm(n, 4 * n, 5)
    ref = oracle.closure(*g)
    assert ctx.count(*g, flags=m4.M4_NO_CACHE) == ref
    assert ctx.count(*g) == ref
    # halo partitions: the register kernel on the separate arrays
    got, st = ctx.count(*g, flags=m4.M4_FORCE_PARTITION, budget=96 * n + 40 * n, stats=True)
    assert got == ref and st["partitions"] > 1
