"""The anchor-selection objective: the serial parts of the edge stage (its owner
counter, its longest row) against the fixed part of the wedge stage, and graphs
beyond 8192 vertices, where the choice is settled without its inputs."""
import pytest

import graphgen as gg
import oracle
from tests import graphs as G

pytestmark = pytest.mark.gpu

CASES = [
    ("short rows, few owners", G.cycle(300), 1),
    ("short rows, few enough owners", G.cycle(1000), 1),
    ("short rows, too many owners", G.cycle(4000), 0),
    ("one vertex below settled", G.cycle(8192), 0),
    ("settled", G.cycle(8193), 0),
    ("settled, hubs", gg.ba(9000, 3, 6), 0),
    ("a long row among few owners", G.wheel(60), 0),
    ("empty rows", G.disjoint_union(G.csr(100, []), G.complete(5)), 1),
]


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_12074_amd as m4
    c = m4.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("name,g,used", CASES, ids=[c[0] for c in CASES])
def test_choice_and_counts(ctx, name, g, used):
    import paper_2607_12074_amd as m4
    got, st = ctx.count(*g, stats=True)
    assert got == oracle.closure(*g)
    assert st["basis_used"] == used == (1 if st["cost_edge"] < st["cost_wedge"] else 0)
    # the estimates of a settled choice are those of an unsettled one, up to
    # the edge basis' lower bound
    forced, sf = ctx.count(*g, flags=m4.M4_BASIS_WEDGE, stats=True)
    assert forced == got and sf["cost_wedge"] == st["cost_wedge"]
    assert st["cost_edge"] <= sf["cost_edge"]
