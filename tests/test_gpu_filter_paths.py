"""The bitmap filters themselves, with and without per-vertex credits: owners
whose endpoints are thin over many ranks, so that no part of them is counted
directly.

m vertices stand at chosen places among T of degree 2 (the rest a ring), each
joined to two middles; a hub is joined to the middles and has pendants enough to
rank highest.  The hub's endpoints are the m vertices, each met twice: wedge
bound 2 m, m candidates.  Without pendants and ring the graph is K_{2, m+1}."""
from math import comb

import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu
DIRECT_SPAN = 262144  # ranks of a part that is counted directly
BITS = 131072  # of the large filter's second bitmap


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_12074_amd as m4
    c = m4.Context(0)
    yield c
    c.close()


def thin(places, total):
    """(graph, middles, hub): ids 0 .. total - 1 have degree 2, in rank order."""
    m = len(places)
    ring = np.setdiff1d(np.arange(total), places)
    mid, hub = total + np.arange(2), total + 2
    pend = hub + 1 + np.arange(m + 2)
    src = np.concatenate([np.tile(places, 2), mid, np.full(m + 2, hub), ring])
    dst = np.concatenate([np.repeat(mid, m), np.full(2, hub), pend, np.roll(ring, 1)])
    return gg.from_edges(hub + m + 3, src.astype(np.int32), dst.astype(np.int32)), mid, hub


def spread(m, total, seed=1):
    return np.sort(np.random.default_rng(seed).choice(total, m, replace=False))


def stacked(m, total):
    """Places that share few bits of the second bitmap: 1 / 8 of them."""
    at = np.arange(m)
    return np.sort(at % (m // 8) + at // (m // 8) * BITS)


def check(ctx, places, total, walks=None, **tuning):
    import paper_2607_12074_amd as m4
    m = len(places)
    g, mid, hub = thin(places, total)
    n = len(g[0]) - 1
    base = ctx.get_tuning()
    slots = [m4.KERNELS.index(k) for k in ("c4_hash", "c4_med", "c4_bin")]
    try:
        ctx.set_tuning(**tuning)
        got, st = ctx.count(*g, flags=m4.M4_BASIS_WEDGE, stats=True)
        orb = ctx.orbits(*g)[:, 4]
    finally:
        ctx.set_tuning(**base)
    assert got[3] == comb(m + 1, 2)
    want = np.zeros(n, np.uint64)
    want[places] = want[hub] = m
    want[mid] = comb(m + 1, 2)
    assert (orb == want).all()
    return {k: (st["k_rows"][i], st["k_elems"][i], st["k_aux2"][i])
            for k, i in zip(("hash", "med", "bin"), slots)}


# the hub's wedge bound is above 12288, its range above DIRECT_SPAN ranks; the
# parts of the last two (131072 endpoints each) are still above it
@pytest.mark.parametrize("m,total", [(6145, 300000), (12000, 300000), (24000, 500000),
                                     (30000, 500000), (65000, 300000), (100001, 900000),
                                     (140001, 1400000)])
def test_large_filter(ctx, m, total):
    parts = -(-2 * m // 131072)
    assert total // parts > DIRECT_SPAN
    rows, elems, walks = check(ctx, spread(m, total), total, c4_bin_win=1, c4_bin_dense=0)["bin"]
    assert rows >= 1 and elems >= 2 * m
    assert walks >= 2 * parts  # a bitmap walk and a counting walk


# one class, a class for every 64 candidates, and the classes between
@pytest.mark.parametrize("m,total", [(12000, 300000), (30000, 500000), (140001, 1400000)])
def test_classes(ctx, m, total):
    seen = {}
    for cap in (64, 1000, 24576):
        seen[cap] = check(ctx, spread(m, total, 2), total, c4_bin_win=1, c4_bin_dense=0,
                          c4_bin_cap=cap)["bin"][2]
    assert seen[64] > m // 64 and seen[1000] > m // 1000 and seen[64] > seen[1000] > seen[24576]


# The later middle meets one rank m times: two walks; the earlier has no endpoint:
# one.  The hub's two parts meet 50000 ranks each, twice: four classes planned, five
# walks.
def test_few_ranks_met_often(ctx):
    walks = check(ctx, spread(100001, 900000), 900000, c4_bin_win=1, c4_bin_dense=0)["bin"][2]
    assert 2 <= walks - 2 * 5 <= 4


# Eight candidates to a bit of the second bitmap: 8191 bits plan two classes of
# 65528 candidates, more than the table holds.  They are dropped and walked in
# four: six walks of the hub (seven if six classes were planned), five of the later
# middle (98286 expected) and one of the earlier, which has no endpoint.
def test_an_overflowing_class_is_split(ctx):
    walks = check(ctx, stacked(65528, 8 * BITS), 8 * BITS, c4_bin_win=1, c4_bin_dense=0)["bin"][2]
    assert walks == 6 + 5 + 1


# the smaller filters beyond the small graphs' kernels: wedge bounds around
# theirs, tables of 768 and 3072 planned candidates
@pytest.mark.parametrize("m", [129, 700, 769, 1024, 1025, 3000, 3073, 6144])
def test_light_and_medium_filters(ctx, m):
    got = check(ctx, spread(m, 20000), 20000)
    rows, elems, walks = got["hash" if m <= 1024 else "med"]
    assert rows >= 1 and elems >= 2 * m and walks >= 2


# the ranged medium bucket (up to 65536 wedges, thin over many windows)
@pytest.mark.parametrize("m", [6145, 20000, 32768])
def test_ranged_medium_filter(ctx, m):
    total = 1500000
    rows, elems, walks = check(ctx, spread(m, total), total, c4_bin_win=0, c4_med_win=1)["med"]
    assert rows >= 1 and elems >= 2 * m and walks >= 2


# A hub whose endpoints lie in two rows: cut in pieces, so that all groups of lanes
# walk.  Whole, the filter took 18 times the time of the windows (which count both
# owners), in pieces 1.4 times; the line is drawn at 8.
def test_two_long_rows(ctx):
    import paper_2607_12074_amd as m4
    m, total = 140001, 2140001
    g, mid, hub = thin(np.arange(m), total)  # all in the first of the parts
    base = ctx.get_tuning()
    ms = {}
    try:
        for name, win in (("c4_window", 0), ("c4_bin", 1)):
            ctx.set_tuning(c4_bin_win=win, c4_bin_dense=0, c4_med_win=0)
            took = []
            for _ in range(5):
                got, st = ctx.count(*g, flags=m4.M4_BASIS_WEDGE | m4.M4_SERIAL, timing=True)
                took.append(st["ms_kernel"][m4.KERNELS.index(name)])
            assert got[3] == comb(m + 1, 2)
            ms[name] = min(took)
    finally:
        ctx.set_tuning(**base)
    print(ms)
    assert ms["c4_bin"] < 8 * ms["c4_window"]


# an owner's lower neighbours are counted once, whatever its parts: two of the hub
# (three parts), m of each middle (two)
def test_parts_count_lower_neighbours_once(ctx):
    import paper_2607_12074_amd as m4
    m, total = 140001, 1400000
    base = ctx.get_tuning()
    try:
        ctx.set_tuning(c4_bin_win=1, c4_bin_dense=0)
        _, st = ctx.count(*thin(spread(m, total), total)[0], flags=m4.M4_BASIS_WEDGE, stats=True)
    finally:
        ctx.set_tuning(**base)
    i = m4.KERNELS.index("c4_bin")
    assert (st["k_rows"][i], st["k_aux"][i]) == (3, 2 + 2 * m)


# tunings saved when c4_bin_cap was the scratch of a workgroup (2^20 endpoints by
# default) plan no class that the table cannot hold
def test_plans_beyond_the_table(ctx):
    walks = [check(ctx, spread(60000, 600000), 600000, c4_bin_win=1, c4_bin_dense=0,
                   c4_bin_cap=cap)["bin"][2] for cap in (0, 32769, 1 << 20, 1 << 24)]
    assert len(set(walks)) == 1
