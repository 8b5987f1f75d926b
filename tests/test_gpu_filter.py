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
