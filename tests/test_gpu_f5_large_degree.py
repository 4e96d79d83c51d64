"""The 5-motif formulas on graphs with a vertex of up to 64,000 neighbours: a
vertex joined to every vertex of t disjoint 4-cycles, in closed form.  The
wheel kernel's counters, as many as the largest degree, fit four waves a
workgroup up to about 19,200, then one, and one workgroup a CU at the top."""
from itertools import permutations
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


def code(edges):
    return min(sorted(tuple(sorted((p[a], p[b]))) for a, b in edges)
               for p in permutations(range(5)))


def cone(t):
    base = 4 * np.arange(t)[:, None]
    u = np.concatenate([(base + [0, 1, 2, 3]).ravel(), np.full(4 * t, 4 * t)])
    v = np.concatenate([(base + [1, 2, 3, 0]).ravel(), np.arange(4 * t)])
    return graphgen.EdgeList(4 * t + 1, u.astype(np.int32), v.astype(np.int32), f"cone{t}")


def cone_counts(gpm, t):
    """Every connected set of five holds the joined vertex (number 4 below) and
    four others, by how many 4-cycles they meet: a 4-cycle gives one vertex in
    4 ways, an edge in 4, two apart in 2, a path of three in 4."""
    spokes = [(4, i) for i in range(4)]
    kinds = {
        (): t * 2 * comb(t - 1, 2) * 16 + comb(t, 2) * 4 + comb(t, 4) * 256,
        ((0, 1),): t * 4 * ((t - 1) * 2 + comb(t - 1, 2) * 16),
        ((0, 1), (2, 3)): comb(t, 2) * 16,
        ((0, 1), (1, 2)): t * 4 * (t - 1) * 4,
        ((0, 1), (1, 2), (2, 3), (3, 0)): t,
    }
    want = [0] * 21
    classes = [code(gpm.motif_class_pattern(5, i)) for i in range(21)]
    for edges, n in kinds.items():
        want[classes.index(code(spokes + list(edges)))] += n
    assert sum(want) == comb(4 * t, 4)
    return want


@pytest.mark.parametrize("t", [2, 4700, 4900, 6000, 9900, 16000])
def test_cone_over_4_cycles(gpm, t):
    print(f"5-motif formula, degree {4 * t}", flush=True)
    g = build(gpm, graphgen.relabel(cone(t), t))
    assert g.max_degree == 4 * t
    assert gpm.motif_count_formula(g, 5) == cone_counts(gpm, t)
