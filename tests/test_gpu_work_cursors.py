"""Kernels whose workers take their tasks from the spread work cursors: numbers
of tasks from one to several times the workers, with remainders of the number
of cursors, on disjoint unions whose counts are closed forms."""
from math import comb

import pytest

import graphgen
from gpu_util import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


@pytest.mark.parametrize("times", [1, 2, 15, 17, 2047, 2049, 8193, 40001])
def test_path_chunks(gpm, times):
    """One induced 4-path a copy: a task or two a copy."""
    g = build(gpm, graphgen.disjoint_union([graphgen.path_graph(4)] * times))
    path = gpm.pattern(4, [(0, 1), (1, 2), (2, 3)], gpm.VERTEX_INDUCED)
    assert gpm.count(g, path) == times
    assert sum(gpm.motif_count_enum(g, 4)) == times


@pytest.mark.parametrize("times", [1, 16, 33, 250])
def test_clique_tasks(gpm, times):
    """Out-degrees of 69 (segment tasks; the class of 65..256) and, in one copy
    of K_300, 299 (the class of 257..512)."""
    g = build(gpm, graphgen.disjoint_union([graphgen.complete_graph(70)] * times +
                                           [graphgen.complete_graph(300)]))
    want = [times * comb(70, k) + comb(300, k) for k in (3, 4, 5)]
    assert gpm.clique_counts(g, 5) == want
    for k in (3, 4, 5):
        assert gpm.count(g, gpm.clique(k)) == want[k - 3]


@pytest.mark.parametrize("times", [1, 5, 17, 700, 1500])
def test_five_motif_arcs(gpm, times):
    """K_6: six 5-cliques a copy and no other connected 5-set."""
    g = build(gpm, graphgen.disjoint_union([graphgen.complete_graph(6)] * times))
    assert gpm.motif_count_formula(g, 5) == [0] * 20 + [6 * times]
