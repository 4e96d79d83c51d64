"""gpm_timing_read's work units of the triangle kernels: the shorter out-list of
each arc's two, by the kernel that takes the arc."""
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


def timed(gpm, call):
    gpm.timing_read()
    gpm.timing_enable(True)
    try:
        call()
    finally:
        gpm.timing_enable(False)
    units = {}
    for name, _, n in gpm.timing_read():
        units[name] = units.get(name, 0) + n
    return units


@pytest.mark.parametrize("name", ["k20", "k60", "k1100", "rmat12"])
def test_triangle_units(gpm, name):
    e = graphgen.rmat(12, seed=8) if name == "rmat12" else graphgen.complete_graph(int(name[1:]))
    g = build(gpm, e)
    off, adj, src = (x.cpu().numpy() for x in g.dag())
    d = np.diff(off).astype(np.int64)
    du, dv = d[src], d[adj]
    most, least = np.maximum(du, dv), np.minimum(du, dv)
    want = {"k_tc_arcs": int(least[(most <= 32) & (du >= 2)].sum()),
            "k_tc_seg": int(least[(most > 32) & (most <= 1024)].sum()),
            "k_tc_seg<hub>": int(least[most > 1024].sum())}
    counting = timed(gpm, lambda: gpm.count(g, gpm.clique(3)))
    assert {k: counting.get(k, 0) for k in want} == want
    arcs = timed(gpm, lambda: gpm.count(g, gpm.diamond()))
    assert (arcs["k_tc_arcs<arcs>"], arcs.get("k_tc_seg<arcs>", 0)) == \
        (want["k_tc_arcs"], want["k_tc_seg"])
