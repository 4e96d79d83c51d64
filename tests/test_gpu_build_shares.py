"""Graph build at the edges of its work split: shares of 1,024 items (row
starts and arcs), rows longer than a share, runs of empty rows longer than
one, and the row lengths where the sorters change, with duplicates and loops
in the stream; CSR and DAG against the oracle, from the stream and from the
CSR."""
import numpy as np
import pytest
import torch

import graphgen
from oracle import canonical_csr
from gpu_util import build, degree_rank_dag

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


def star(n, centre, length, seed):
    """A vertex joined to `length` others of n, a tenth of the edges twice and
    some loops: its raw row is longer than its final one."""
    rng = np.random.default_rng(seed)
    others = rng.permutation(n - 1)[:length]
    others = others + (others >= centre)
    u = np.concatenate([np.full(length, centre), others[:length // 10], others[:20]])
    v = np.concatenate([others, np.full(length // 10, centre), others[:20]])
    return graphgen.EdgeList(n, u.astype(np.int32), v.astype(np.int32), f"star{length} in {n}")


CASES = {
    # items = n + arcs + 1: one share less one item, exactly one, one more
    "cycle_1021": lambda: graphgen.cycle_graph(340),
    "cycle_1024": lambda: graphgen.cycle_graph(341),
    "path_1025": lambda: graphgen.path_graph(342),
    "one_vertex": lambda: graphgen.EdgeList(1, np.zeros(1, np.int32), np.zeros(1, np.int32), ""),
    # empty rows before, between and after the only edges
    "sparse": lambda: graphgen.EdgeList(9000, np.array([3000, 3000, 8000], np.int32),
                                        np.array([3001, 6500, 8999], np.int32), ""),
    "all_empty": lambda: graphgen.EdgeList(5000, np.zeros(0, np.int32), np.zeros(0, np.int32), ""),
    # sorters: 16 and 512 entries, then the bitmap (few ids)
    "row16": lambda: star(3000, 7, 16, 1),
    "row17": lambda: star(3000, 7, 17, 2),
    "row470": lambda: star(3000, 0, 465, 3),
    "row600": lambda: star(3000, 2999, 600, 4),
    "hub": lambda: star(100000, 50000, 70000, 5),
    # many ids: registers up to 2048 raw entries, the bitmap above
    "wide_row1800": lambda: star(140000, 139999, 1800, 6),
    "wide_row2000": lambda: star(140000, 0, 2000, 7),
    "rmat": lambda: graphgen.rmat(11, seed=5),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_build_and_from_csr(gpm, name):
    e = CASES[name]()
    off, adj = canonical_csr(e.n, e.u, e.v)
    src, dst = degree_rank_dag(off, adj)
    dag_off = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=e.n))])
    g = build(gpm, e)
    h = gpm.Graph.from_csr(e.n, torch.from_numpy(np.asarray(off, np.int32)).cuda(),
                           torch.from_numpy(np.asarray(adj, np.int32)).cuda())
    for x in (g, h):
        assert (x.m, x.max_degree) == (adj.shape[0] // 2, int(np.diff(off).max()))
        assert x.max_out_degree == (int(np.diff(dag_off).max()))
        got = [t.cpu().numpy() for t in (*x.csr(), *x.dag())]
        for a, b in zip(got, (off, adj, dag_off, dst, src)):
            assert np.array_equal(a, b)
