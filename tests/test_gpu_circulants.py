"""Circulant graphs, where neighbours share most of their neighbours: arcs of
many triangles whose rows cross the waves that merge them (counted per arc,
through the diamonds, sum over edges of C(T_e, 2)), and 4-cycles that lie in
few of an apex's id ranges."""
from math import comb

import numpy as np
import pytest

import graphgen
import oracle
from oracle import canonical_csr
from gpu_util import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


def circulant(n, s, stride=1):
    """n vertices, ids stride apart, each joined to the s next."""
    v = np.repeat(np.arange(n), s)
    w = (v + np.tile(np.arange(1, s + 1), n)) % n
    return graphgen.EdgeList(n * stride, (v * stride).astype(np.int32),
                             (w * stride).astype(np.int32), f"circulant {n} {s}")


def triangles_on(s):
    """Triangles on an edge of each length 1 .. s (n > 3 s)."""
    near = set(range(-s, s + 1)) - {0}
    return [sum(1 for x in near if x - d in near) for d in range(1, s + 1)]


# out-degrees s, and up to 2 s at the lowest ids: 16 is the merged rows' whole
# range, 17 and 20 cross its end, 32 is the longest merged row, 33 beyond it
@pytest.mark.parametrize("s", [2, 5, 16, 17, 20, 31, 32, 33])
@pytest.mark.parametrize("n", [101, 1000])
@pytest.mark.parametrize("shuffled", [False, True])
def test_triangles_per_arc(gpm, s, n, shuffled):
    e = circulant(n, s)
    g = build(gpm, graphgen.relabel(e, 5) if shuffled else e)
    t = triangles_on(s)
    assert gpm.count(g, gpm.clique(3)) == n * sum(t) // 3
    assert gpm.count(g, gpm.diamond()) == n * sum(comb(x, 2) for x in t)


# 64 ids in one row, rows of 1 to 32 hits: 3 hits and 4 take different routes
@pytest.mark.parametrize("k", [3, 4, 5, 6, 7, 20, 33])
def test_disjoint_cliques(gpm, k):
    g = build(gpm, graphgen.disjoint_union([graphgen.complete_graph(k)] * 50))
    assert gpm.count(g, gpm.clique(3)) == 50 * comb(k, 3)
    assert gpm.count(g, gpm.diamond()) == 50 * comb(k, 2) * comb(k - 2, 2)


# ids below and above 65,536 (ranges of 2,048 and of 8,192 ids), neighbours
# side by side or ranges apart
@pytest.mark.parametrize("n,stride", [(200, 1), (200, 300), (200, 350), (400, 170)])
def test_list_4cycles(gpm, n, stride):
    e = circulant(n, 20, stride)
    g = build(gpm, e)
    total, chk, _ = oracle.list_c4(*canonical_csr(e.n, e.u, e.v), cap=0)
    t, w, c, _ = gpm.list_embeddings(g, gpm.cycle4(gpm.EDGE_INDUCED | gpm.LIST), 1000)
    assert (t, w, c) == (total, 1000, chk)
