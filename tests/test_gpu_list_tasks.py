"""4-cycle listing where one apex holds most pairs: its tasks' pairs are
shared out through the arena, smaller tasks are listed where they are
grouped, with small and large id ranges per task."""
import pytest

import graphgen
import oracle
from oracle import canonical_csr
from gpu_util import build
from test_gpu_sl import edge_sets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


# K_{12,100}: the apexes are the twelve vertices of degree 100, the i-th with
# 4,950 i pairs, so the ids 7 .. 11 are above the 32,768 pairs a task is
# shared out from and the others below.  Isolated vertices set the id range:
# one id above 65,536 takes the larger parts.
@pytest.mark.parametrize("n", [112, 2049, 65536, 65537])
def test_list_large_and_small_tasks(gpm, n):
    e = graphgen.complete_bipartite(12, 100)
    e = graphgen.EdgeList(n, e.u, e.v, name=f"K12,100 in {n}")
    g = build(gpm, e)
    off, adj = canonical_csr(e.n, e.u, e.v)
    total, chk, rows = oracle.list_c4(off, adj, cap=400000)
    assert total == 66 * 4950
    pat = gpm.cycle4(gpm.EDGE_INDUCED | gpm.LIST)
    t, w, c, got = gpm.list_embeddings(g, pat, 400000)
    assert (t, w, c) == (total, total, chk)
    assert edge_sets("4-cycle", got.cpu().tolist()) == edge_sets("4-cycle", rows.tolist())


def test_list_truncated_large_task(gpm):
    """A buffer that the large tasks fill: the total and the checksum still
    cover every embedding."""
    e = graphgen.complete_bipartite(12, 100)
    g = build(gpm, e)
    off, adj = canonical_csr(e.n, e.u, e.v)
    total, chk, rows = oracle.list_c4(off, adj, cap=400000)
    pat = gpm.cycle4(gpm.EDGE_INDUCED | gpm.LIST)
    t, w, c, got = gpm.list_embeddings(g, pat, 1000)
    assert (t, w, c) == (total, 1000, chk)
    sets = edge_sets("4-cycle", got.cpu().tolist())
    assert len(sets) == 1000 and sets <= edge_sets("4-cycle", rows.tolist())
