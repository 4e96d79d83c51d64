"""5-clique listing at roots of out-degree 513 to 1024, every number of 64-bit
words a row: total, checksum and rows against the oracle."""
import numpy as np
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


def wide(d, p, seed):
    """A vertex joined to d others, which are joined at random (p) and each to
    d + 50 of 4 d leaves, so that their degrees are above d: the vertex is a
    root of out-degree d."""
    rng = np.random.default_rng(seed)
    iu, ju = np.triu_indices(d, 1)
    keep = rng.random(iu.shape[0]) < p
    us, vs = [np.full(d, d), iu[keep]], [np.arange(d), ju[keep]]
    for h in range(d):
        us.append(np.full(d + 50, h))
        vs.append(d + 1 + rng.choice(4 * d, d + 50, replace=False))
    return graphgen.EdgeList(5 * d + 1, np.concatenate(us).astype(np.int32),
                             np.concatenate(vs).astype(np.int32), f"wide{d}")


@pytest.mark.parametrize("d", [513, 577, 640, 700, 768, 832, 833, 880, 896, 897, 960, 1023, 1024])
def test_rows_of_9_to_16_words(gpm, d):
    e = wide(d, 40.0 / d, d)
    print(f"5-clique listing, root of out-degree {d}", flush=True)
    g = build(gpm, e)
    assert g.max_out_degree == d
    off, adj = oracle.canonical_csr(e.n, e.u, e.v)
    total, chk, rows = oracle.clique_list(off, adj, 5, cap=1 << 20)
    assert 0 < total < 1 << 20
    t, w, c, got = gpm.list_embeddings(g, gpm.clique(5, gpm.VERTEX_INDUCED | gpm.LIST), 1 << 20)
    assert (t, w, c) == (total, total, chk)
    assert {tuple(sorted(r)) for r in got.cpu().tolist()} == {tuple(sorted(r)) for r in rows.tolist()}
