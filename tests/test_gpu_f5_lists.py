"""The 5-motif formulas with and without the common-neighbour lists: dense
graphs whose lists exceed their arena (counted without them), edges of 512
triangles and more, vertices split into several tasks; closed forms and the
enumeration route."""
from math import comb

import numpy as np
import pytest

import graphgen
from gpu_util import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


# K_n has n - 2 triangles an edge: up to 192 fit
@pytest.mark.parametrize("n", [5, 150, 194, 195, 300])
def test_complete_graphs(gpm, n):
    want = [0] * 21
    want[20] = comb(n, 5)
    assert gpm.motif_count_formula(build(gpm, graphgen.complete_graph(n)), 5) == want


def test_big_arcs_and_split_vertices(gpm):
    """K_514 beside K_{300,800}: 512 triangles on an edge (a workgroup per
    arc), 131,328 at a vertex (many tasks), and room for the lists.  K_{a,b}
    alone has 4-stars and K_{2,3} copies, two classes."""
    a, b = 300, 800
    e = graphgen.disjoint_union([graphgen.complete_graph(514), graphgen.complete_bipartite(a, b)])
    want = [0] * 21
    want[20] = comb(514, 5)
    want[0] = a * comb(b, 4) + b * comb(a, 4)
    want[10] = comb(a, 2) * comb(b, 3) + comb(a, 3) * comb(b, 2)
    assert gpm.motif_count_formula(build(gpm, graphgen.relabel(e, 5)), 5) == want


def test_multipartite(gpm):
    """Many classes at once, by the enumeration route: a complete multipartite
    graph joined to a random one by a few edges."""
    a = graphgen.complete_multipartite([3, 5, 8])
    b = graphgen.erdos_renyi(70, 0.15, 9)
    e = graphgen.disjoint_union([a, b])
    u = np.concatenate([e.u, np.arange(8, dtype=np.int32)])
    v = np.concatenate([e.v, np.arange(20, 28, dtype=np.int32)])
    g = build(gpm, graphgen.EdgeList(e.n, u, v, "joined"))
    assert gpm.motif_count_formula(g, 5) == gpm.motif_count_enum(g, 5)
