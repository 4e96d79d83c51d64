"""Counts of 4- and 5-vertex patterns whose last two steps are taken together:
every connected pattern, vertex- and edge-induced, on a graph with rows of
several 64-candidate chunks and one with short rows, against the oracle."""
import pytest

import graphgen
import oracle
from gpu_util import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


@pytest.fixture(scope="module")
def graphs(gpm):
    es = [graphgen.disjoint_union([graphgen.star_graph(150), graphgen.erdos_renyi(90, 0.25, seed=3),
                                   graphgen.complete_bipartite(3, 70)]),
          graphgen.erdos_renyi(400, 0.02, seed=4)]
    return [(build(gpm, e), *oracle.canonical_csr(e.n, e.u, e.v)) for e in es]


@pytest.mark.parametrize("k,index", [(4, i) for i in range(6)] + [(5, i) for i in range(21)])
def test_connected_patterns(gpm, graphs, k, index):
    edges = gpm.motif_class_pattern(k, index)
    for g, off, adj in graphs:
        for induced, flags in ((True, gpm.VERTEX_INDUCED), (False, gpm.EDGE_INDUCED)):
            got = gpm.count(g, gpm.pattern(k, edges, flags))
            want = oracle.pattern_count(off, adj, k, edges, induced)
            assert got == (want[0] if isinstance(want, tuple) else want)
