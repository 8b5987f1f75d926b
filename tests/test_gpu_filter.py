"""4-cycle owners counted through the LDS bitmap filters, at the edges of their
wedge bounds and tables.

The graph joins k middle vertices to each of m leaves and to a hub that also
has enough pendant vertices to rank highest: the hub's wedge endpoints are the
m leaves, each met k times, so its wedge bound is k m, every endpoint is a
candidate and the number of distinct ones is chosen exactly.  Without its
pendants the graph is K_{k, m+1}: C(k, 2) C(m + 1, 2) induced 4-cycles."""
from math import comb

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_12074_amd as m4
    c = m4.Context(0)
    yield c
    c.close()


def hub_graph(k, m):
    mid, leaf, hub = np.arange(k), k + np.arange(m), k + m
    pend = hub + 1 + np.arange(m + k)
    src = np.concatenate([np.repeat(mid, m), mid, np.full(m + k, hub)])
    dst = np.concatenate([np.tile(leaf, k), np.full(k, hub), pend])
    return gg.from_edges(hub + 1 + m + k, src, dst)


# wedge bounds 2 m around the tiny (256), light (2048), medium (12288) limits
# and the rank ranges of the large filter (131072); tables of 768, 3072 and
# 24576 planned candidates are exceeded from m = 769, 3073 and 24577 on
@pytest.mark.parametrize("m", [2, 127, 128, 129, 768, 769, 1024, 1025, 3072, 3073, 6144, 6145,
                               24577, 60000, 65537, 140001])
def test_candidates_around_the_bounds(ctx, m):
    import paper_2607_12074_amd as m4
    g = hub_graph(2, m)
    ref = oracle.closure(*g)
    assert ref[3] == comb(2, 2) * comb(m + 1, 2)
    base = ctx.get_tuning()
    try:
        for bin_win in (0, 1):
            ctx.set_tuning(c4_bin_win=bin_win, c4_bin_dense=0)
            got, st = ctx.count(*g, flags=m4.M4_BASIS_WEDGE, stats=True)
            assert got == ref, bin_win
            if bin_win and 2 * m > 12288:
                assert st["k_rows"][m4.KERNELS.index("c4_bin")] > 0
    finally:
        ctx.set_tuning(**base)


# a class planned for 64 candidates (many classes), for exactly as many as
# there are, and for 2^24 (one class: the table overflows and the classes are
# split until they fit)
@pytest.mark.parametrize("k,m", [(2, 40000), (3, 33333), (2, 65537)])
@pytest.mark.parametrize("cap", [64, 40000, 1 << 24])
def test_classes_of_the_large_filter(ctx, k, m, cap):
    import paper_2607_12074_amd as m4
    g = hub_graph(k, m)
    base = ctx.get_tuning()
    try:
        ctx.set_tuning(c4_bin_win=1, c4_bin_dense=0, c4_bin_cap=cap)
        got, st = ctx.count(*g, flags=m4.M4_BASIS_WEDGE, stats=True)
    finally:
        ctx.set_tuning(**base)
    assert got == oracle.closure(*g)
    assert got[3] == comb(k, 2) * comb(m + 1, 2)
    assert st["k_rows"][m4.KERNELS.index("c4_bin")] > 0


# the same edges with per-vertex credits: leaves and hub lie on C(k, 2) m
# cycles, middles on (k - 1) C(m + 1, 2), pendants on none
@pytest.mark.parametrize("k,m", [(2, 2), (2, 128), (2, 129), (3, 700), (2, 1024), (2, 1025),
                                 (2, 3073), (2, 6145), (2, 24577), (3, 60000), (2, 140001)])
def test_cycle_credits_around_the_bounds(ctx, k, m):
    got = ctx.orbits(*hub_graph(k, m))[:, 4]
    assert (got[:k] == (k - 1) * comb(m + 1, 2)).all()
    assert (got[k:k + m + 1] == comb(k, 2) * m).all()
    assert not got[k + m + 1:].any()


def test_credits_with_counts_beyond_the_packed_slots(ctx):
    # above 2^24 vertices a 32-bit slot keeps counts below 65536: K_{2, 70000},
    # thin among the ranks of a 400000-cycle, takes the 64-bit slots
    import torch
    from tests import graphs as G
    from tests.test_oracle_orbits import cf_bipartite
    k = 70002
    rp, col = G.disjoint_union(G.complete_bipartite(2, 70000), G.cycle(400000))
    n = (1 << 24) + 10
    full = torch.full((n + 1,), int(rp[-1]), dtype=torch.int64, device="cuda")
    full[:len(rp)] = torch.from_numpy(rp).cuda()
    cold = torch.from_numpy(col).cuda()
    torch.cuda.synchronize()
    got = ctx.orbits(full, cold)
    torch.cuda.synchronize()
    assert (got[:k].cpu().numpy().view(np.uint64) == cf_bipartite(2, 70000)).all()
    # on a long cycle every vertex ends two paths and is inside two
    ring = torch.zeros(11, dtype=torch.int64, device="cuda")
    ring[:2] = 2
    assert bool((got[k:k + 400000] == ring).all())
    assert not bool(got[k + 400000:].any())


# graphs of up to 8192 vertices count every owner above 256 wedges directly:
# around that size, and around the tiny bound
@pytest.mark.parametrize("n,m", [(8191, 90000), (8192, 90000), (8193, 90000), (300, 4000),
                                 (64, 900)])
def test_direct_counters_around_their_size(ctx, n, m):
    import paper_2607_12074_amd as m4
    g = gg.gnm(n, m, 7)
    got, st = ctx.count(*g, flags=m4.M4_BASIS_WEDGE, stats=True)
    assert got == oracle.closure(*g)
    orb = ctx.orbits(*g)
    assert int(orb[:, 4].sum()) == 4 * got[3] and int(orb[:, 10].sum()) == 4 * got[5]
    if n <= 300:
        assert (orb == oracle.orbits_esu(*g)).all()
