"""5-clique counts of local graphs on the matrix cores: out-degrees around the
edges of row words, tiles of 32 members and the classes' bounds, in complete
graphs (closed form) and dense random ones (the oracle)."""
from math import comb

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


@pytest.mark.parametrize("n", [66, 97, 129, 130, 193, 257, 258, 289, 321, 513, 514, 577, 705, 1001,
                               1025])
def test_complete_graphs(gpm, n):
    g = build(gpm, graphgen.complete_graph(n))
    assert gpm.count(g, gpm.clique(5)) == comb(n, 5)
    assert gpm.clique_counts(g, 5) == [comb(n, k) for k in (3, 4, 5)]


@pytest.mark.parametrize("n,p", [(300, 0.6), (420, 0.7), (700, 0.25)])
def test_dense_random(gpm, n, p):
    e = graphgen.erdos_renyi(n, p, seed=n)
    off, adj = oracle.canonical_csr(e.n, e.u, e.v)
    g = build(gpm, e)
    for k in (4, 5):
        assert gpm.count(g, gpm.clique(k)) == oracle.clique_count(off, adj, k)
