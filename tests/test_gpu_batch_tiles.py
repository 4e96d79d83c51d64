"""Batched 4-motif counts at the edges of the 32 x 32 codegree tiles, of row
words and of the tiers, on empty, sparse, dense and complete graphs, and with
numbers of graphs around the work cursors' and the workgroups' numbers."""
from math import comb

import numpy as np
import pytest
import torch

import graphgen
import oracle
from gpu_util import build

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 192, 193, 204, 205, 224, 225, 255, 256,
         257, 320]


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


def counts(gpm, parts, k, config=None):
    voff = np.cumsum([0] + [p.n for p in parts]).astype(np.int32)
    g = build(gpm, graphgen.disjoint_union(parts))
    return gpm.batch_motif_count(g, torch.from_numpy(voff).cuda(), k, config=config).cpu().tolist()


@pytest.mark.parametrize("threads,tiers", [(64, 3), (128, 2), (256, 1)])
def test_sizes_and_densities(gpm, threads, tiers):
    parts = [graphgen.erdos_renyi(n, p, seed=7 * n + i) for n in SIZES
             for i, p in enumerate((0.0, 0.03, 0.5))]
    config = gpm.batch_default_config()
    config.team_threads, config.tiers = threads, tiers
    got = counts(gpm, parts, 4, config)
    for row, p in zip(got, parts):
        off, adj = oracle.canonical_csr(p.n, p.u, p.v)
        assert row == oracle.motif4(off, adj) + [0], p.n


@pytest.mark.parametrize("n", [63, 256, 257, 1000, 1023, 1024])
def test_complete_and_bipartite(gpm, n):
    a, b = n // 2, n - n // 2
    got = counts(gpm, [graphgen.complete_graph(n), graphgen.complete_bipartite(a, b)], 4)
    assert got[0] == [0, 0, 0, 0, 0, comb(n, 4), 0]
    claw = a * comb(b, 3) + b * comb(a, 3)
    assert got[1] == [claw, 0, comb(a, 2) * comb(b, 2), 0, 0, 0, 0]


@pytest.mark.parametrize("graphs", [1, 7, 4095, 4097, 9001])
@pytest.mark.parametrize("k", [3, 4])
def test_numbers_of_graphs(gpm, graphs, k):
    parts = [graphgen.complete_graph(5), graphgen.path_graph(4), graphgen.star_graph(3)]
    want = {3: [[0, 10, 0], [2, 0, 0], [3, 0, 0]],
            4: [[0, 0, 0, 0, 0, 5, 0], [0, 1, 0, 0, 0, 0, 0], [1, 0, 0, 0, 0, 0, 0]]}[k]
    got = counts(gpm, [parts[i % 3] for i in range(graphs)], k)
    assert got == [want[i % 3] for i in range(graphs)]
