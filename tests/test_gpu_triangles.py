"""Triangle kernels at the edges of their dispatch: arcs merged a lane each
(out-degrees up to 32), roots staged in LDS (33 to 1024) in runs of
neighbours, roots searched in global memory (above 1024); counts, per-arc
counts (through the diamonds, sum over edges of C(T_e, 2)) and listing."""
from math import comb

import numpy as np
import pytest

import graphgen
import oracle
from gpu_util import build

pytestmark = pytest.mark.gpu
FINE = {"tc_tau": [2048] * 3, "tc_blocks_per_cu": [1] * 3}


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


# K_n's out-degrees are 0 .. n - 1: the ends of the classes (32, 33; 64, 65;
# 256, 257; 1024, 1025) and of the units of 16 entries, and with the smallest
# chunks a root's neighbours in one task (256) or two (257)
@pytest.mark.parametrize("n", [3, 17, 18, 33, 34, 65, 66, 257, 258, 1025, 1026])
@pytest.mark.parametrize("fine", [False, True])
def test_complete_graphs(gpm, n, fine):
    g = build(gpm, graphgen.relabel(graphgen.complete_graph(n), n))
    if fine:
        g.set_tuning(**FINE)
    assert gpm.count(g, gpm.clique(3)) == comb(n, 3)
    assert gpm.count(g, gpm.diamond()) == comb(n, 2) * comb(n - 2, 2)
    cap = min(comb(n, 3), 10000)
    total, written, _, rows = gpm.list_embeddings(
        g, gpm.clique(3, gpm.VERTEX_INDUCED | gpm.LIST), cap)
    assert (total, written) == (comb(n, 3), cap)
    got = {tuple(sorted(r)) for r in rows.cpu().tolist()}
    assert len(got) == cap and all(len(set(r)) == 3 and r[2] < n for r in got)


def mixed():
    """Cliques of 20 to 60 vertices (both kernels), each vertex with pendant
    and short-list neighbours (empty and one-entry segments), a random part
    and a relabelling."""
    parts = [graphgen.complete_graph(k) for k in (20, 33, 34, 60)]
    parts.append(graphgen.erdos_renyi(400, 0.2, 5))
    e = graphgen.disjoint_union(parts)
    rng = np.random.default_rng(7)
    hang = np.arange(e.n, e.n + 3000)
    u = np.concatenate([e.u, hang, rng.integers(0, e.n, 3000)])
    v = np.concatenate([e.v, rng.integers(0, e.n, 3000), hang[rng.integers(0, 3000, 3000)]])
    return graphgen.relabel(graphgen.EdgeList(e.n + 3000, u.astype(np.int32),
                                              v.astype(np.int32), "mixed"), 3)


@pytest.mark.parametrize("order", ["degree", "core"])
@pytest.mark.parametrize("fine", [False, True])
def test_mixed_lists(gpm, order, fine):
    e = mixed()
    g = build(gpm, e)
    if order == "core":
        g.orient(gpm.ORIENT_CORE)
    if fine:
        g.set_tuning(**FINE)
    off, adj = oracle.canonical_csr(e.n, e.u, e.v)
    tri = oracle.clique_count(off, adj, 3)
    assert gpm.count(g, gpm.clique(3)) == tri
    assert gpm.motif_count(g, 4) == oracle.motif4(off, adj)
    total, written, chk, rows = gpm.list_embeddings(
        g, gpm.clique(3, gpm.VERTEX_INDUCED | gpm.LIST), tri)
    got = {tuple(sorted(r)) for r in rows.cpu().tolist()}
    assert total == written == tri == len(got)
    codes = set((np.repeat(np.arange(e.n), np.diff(off)) * e.n + adj).tolist())
    assert all(a * e.n + b in codes and a * e.n + c in codes and b * e.n + c in codes
               for a, b, c in got)
