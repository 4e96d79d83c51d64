"""Calls in less device memory than their preferred workspace: any size from
the smallest on gives the same counts, below it the call is refused with its
outputs untouched, and the Python call falls back to it where the device has
no room."""
import ctypes
from math import comb

import pytest
import torch

import graphgen
from gpu_util import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


def sizes(least, most):
    """From the smallest to the preferred size, with odd ones between."""
    step = (most - least) // 7
    return [least, least + 256, least + 5000] + [least + i * step + i for i in range(1, 7)] + [most]


class limited_memory:
    """At most `free` bytes beyond what is in use, for torch's allocator."""

    def __init__(self, free):
        self.free = free

    def __enter__(self):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        total = torch.cuda.get_device_properties(0).total_memory
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + self.free) / total)

    def __exit__(self, *args):
        torch.cuda.set_per_process_memory_fraction(1.0)


def ptr(t):
    return ctypes.c_void_p(t.data_ptr())


@pytest.mark.parametrize("name", ["rmat11", "k194", "k195", "edges0"])
def test_formulas(gpm, name):
    e = {"rmat11": lambda: graphgen.rmat(11, seed=4), "k194": lambda: graphgen.complete_graph(194),
         "k195": lambda: graphgen.complete_graph(195),
         "edges0": lambda: graphgen.disjoint_union([graphgen.path_graph(2)])}[name]()
    g = build(gpm, e)
    want = gpm.motif_count_formula(g, 5)
    if name[0] == "k":
        assert want == [0] * 20 + [comb(e.n, 5)]
    least, most = gpm.motif_formula_compact_bytes(g, 5), gpm.motif_formula_workspace_bytes(g, 5)
    assert least <= most
    lib, ws = gpm.load(), torch.empty(most, dtype=torch.uint8, device="cuda")
    for n in sizes(least, most):
        print(f"5-motif formulas of {name} in {n} of {most} bytes", flush=True)
        ws.fill_(0xA5)
        out = torch.full((22,), -1, dtype=torch.int64, device="cuda")
        assert lib.gpm_motif_count_formula_compact(g.handle, 5, ptr(ws), n, ptr(out), None) == 0
        torch.cuda.synchronize()
        assert out.tolist() == want + [0], n
        assert bool((ws[n:] == 0xA5).all()), n
    out = torch.full((22,), -1, dtype=torch.int64, device="cuda")
    rc = lib.gpm_motif_count_formula_compact(g.handle, 5, ptr(ws), least - 256, ptr(out), None)
    assert rc == 2 and bool((out == -1).all())


def test_formulas_where_the_lists_have_no_room(gpm):
    g = build(gpm, graphgen.rmat(14, seed=5))
    want = gpm.motif_count_formula(g, 5)
    least, most = gpm.motif_formula_compact_bytes(g, 5), gpm.motif_formula_workspace_bytes(g, 5)
    assert most > least + (256 << 20)
    with limited_memory(least + (64 << 20)):
        assert gpm.motif_count_formula(g, 5) == want


# K_{12,100}: the five largest tasks have 32,768 pairs and more, the line from
# which a task's pairs are shared out through the arena; with 65,537 vertices
# the ids of a task are cut otherwise.  RMAT-12 has hundreds of such tasks.
@pytest.mark.parametrize("name", ["k12_100", "k12_100 wide", "rmat12"])
def test_4_cycle_listing(gpm, name):
    e = graphgen.rmat(12, seed=3) if name == "rmat12" else graphgen.complete_bipartite(12, 100)
    if name[-4:] == "wide":
        e = graphgen.EdgeList(65537, e.u, e.v, name)
    g = build(gpm, e)
    p = gpm.cycle4(gpm.EDGE_INDUCED | gpm.LIST)
    want = list(gpm.list_embeddings(g, p, 1000)[:3])
    if name != "rmat12":
        assert want[:2] == [comb(12, 2) * comb(100, 2), 1000]
    least, most = gpm.list_compact_bytes(g, p), gpm.workspace_bytes(g, p)
    assert least < most
    lib, ws = gpm.load(), torch.empty(most, dtype=torch.uint8, device="cuda")
    buf = torch.empty((1000, 4), dtype=torch.int32, device="cuda")
    arena = [least + (2 << 20) + x for x in (0, 20000, 300000, 3000000)]   # past the task list
    for n in sizes(least, most) + [x for x in arena if x < most]:
        print(f"4-cycles of {name} in {n} of {most} bytes", flush=True)
        ws[least:] = 0xA5
        out = torch.full((3,), -1, dtype=torch.int64, device="cuda")
        assert lib.gpm_list_compact(g.handle, ctypes.byref(p), ptr(ws), n, ptr(buf), 1000,
                                    ptr(out), None) == 0
        torch.cuda.synchronize()
        assert [x % (1 << 64) for x in out.tolist()] == want, n
        assert bool((ws[n:] == 0xA5).all()), n
    out = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    rc = lib.gpm_list_compact(g.handle, ctypes.byref(p), ptr(ws), least - 256, ptr(buf), 1000,
                              ptr(out), None)
    assert rc == 2 and bool((out == -1).all())


def test_4_cycle_listing_where_the_arena_has_no_room(gpm):
    g = build(gpm, graphgen.rmat(13, seed=6))
    p = gpm.cycle4(gpm.EDGE_INDUCED | gpm.LIST)
    want = gpm.list_embeddings(g, p, 100)[:3]
    least, most = gpm.list_compact_bytes(g, p), gpm.workspace_bytes(g, p)
    assert most > least + (400 << 20)
    with limited_memory(least + (64 << 20)):
        assert gpm.list_embeddings(g, p, 100)[:3] == want
