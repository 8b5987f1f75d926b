"""The basis chosen for small graphs, whose plans are shared by both: uniform graphs
on which the wedge basis was measured faster by 15 us and more, of which the
objective took the edge basis while it priced a plan of the wedge stage's own."""
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,degree", [(60, 16), (100, 16), (200, 8), (200, 16), (400, 4), (400, 8),
                                      (700, 4), (700, 8), (1000, 4), (1000, 8), (2000, 4)])
def test_wedges_are_chosen(n, degree):
    import paper_2607_12074_amd as m4
    ctx = m4.Context(0)
    g = gg.gnm(n, n * degree // 2, 1)
    got, st = ctx.count(*g, stats=True)
    assert got == oracle.closure(*g)
    assert st["basis_used"] == 0 and st["cost_wedge"] <= st["cost_edge"]
    ctx.close()
