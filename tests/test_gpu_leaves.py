"""Hubs with many neighbours of degree 1: these hold no wedge endpoint, so the
4-cycle kernels read an owner's other lower neighbours only, in every bucket."""
from math import comb

import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_12074_amd as m4
    c = m4.Context(0)
    yield c
    c.close()


def leafy(m, leaves, ring=0):
    """K_{2, m+1} with `leaves` pendants on one of the m + 1, beside a cycle."""
    mid, other, hub = np.arange(2), 2 + np.arange(m), 2 + m
    pend = hub + 1 + np.arange(leaves)
    cyc = hub + 1 + leaves + np.arange(ring)
    src = np.concatenate([np.repeat(mid, m), mid, np.full(leaves, hub), cyc])
    dst = np.concatenate([np.tile(other, 2), np.full(2, hub), pend, np.roll(cyc, 1)])
    return gg.from_edges(hub + 1 + leaves + ring, src.astype(np.int32), dst.astype(np.int32))


# hub's wedge bound 2 m: tiny, light, medium and large buckets; with few leaves
# the graph is small, with many the hub's lower neighbours exceed the filters'
# packed counts (when the leaves are among them)
@pytest.mark.parametrize("m,ring", [(3, 0), (60, 0), (600, 0), (3000, 0), (70001, 400000)])
@pytest.mark.parametrize("leaves", [5000, 90000])
def test_leaves_are_not_read(ctx, m, ring, leaves):
    import paper_2607_12074_amd as m4
    g = leafy(m, leaves, ring)
    cycles = comb(m + 1, 2)
    base = ctx.get_tuning()
    try:
        ctx.set_tuning(c4_bin_win=1, c4_bin_dense=0)
        got, st = ctx.count(*g, flags=m4.M4_BASIS_WEDGE, stats=True)
        n = len(g[0]) - 1
        part, sp = ctx.count(*g, flags=m4.M4_FORCE_PARTITION, budget=96 * n + 40 * n, stats=True)
    finally:
        ctx.set_tuning(**base)
    assert got[3] == cycles and part == got
    filters = [m4.KERNELS.index(k) for k in ("c4_hash", "c4_med", "c4_bin")]
    # lower neighbours of degree 2 and more: m + 2 for the hub and at most
    # m + 1 for either middle, one for a ring vertex (two for its last)
    assert sum(st["k_aux"][i] for i in filters) <= 3 * (m + 2) + ring + 1
    # middles and others of K_{2, m+1}: C(m + 1, 2) and m cycles each
    orb = ctx.orbits(*g)[:, 4]
    assert (orb[:2] == cycles).all() and (orb[2:m + 3] == m).all() and not orb[m + 3:].any()
