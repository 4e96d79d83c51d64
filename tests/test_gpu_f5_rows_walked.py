"""The 5-motif formulas without the common-neighbour lists, up to 65,536
vertices: a graph of several motif classes beside one whose lists exceed their
arena (K_300: 298 triangles an edge), padded to the sizes where the row kernels
change (a bitmap of N(a) per wave up to about 39,700 vertices, one for the
workgroup above)."""
from math import comb

import pytest

import graphgen
import oracle
from gpu_util import build
from test_gpu_motif5_formula import big_hub, padded

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


@pytest.fixture(scope="module")
def joined(gpm):
    hub = big_hub()
    off, adj = oracle.canonical_csr(hub.n, hub.u, hub.v)
    want = [oracle.pattern_count(off, adj, 5, gpm.motif_class_pattern(5, i), True)[0]
            for i in range(21)]
    want[20] += comb(300, 5)
    return graphgen.disjoint_union([hub, graphgen.complete_graph(300)]), want


@pytest.mark.parametrize("n", [451, 32768, 39000, 40000, 60000, 65536])
def test_lists_that_do_not_fit(gpm, joined, n):
    e, want = joined
    assert want[18] > 0 and want[19] > 0 and sum(w > 0 for w in want) > 12
    print(f"5-motif formula without lists, {n} vertices", flush=True)
    gpm.timing_read()
    gpm.timing_enable(True)
    got = gpm.motif_count_formula(build(gpm, e if n == e.n else padded(e, n, n)), 5)
    gpm.timing_enable(False)
    assert {"k_f5_trace5", "k_f5_wheel"} <= {name for name, _, _ in gpm.timing_read()}
    assert got == want
