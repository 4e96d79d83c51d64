"""Graph build at the largest sizes the header accepts, where an index that
steps past the last arc or row leaves 32 signed bits: 2^31 - 2 arcs, and
2^31 - 2 vertices.  Closed forms (70 GB of the device's memory at most)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
I32 = dict(dtype=torch.int32, device="cuda")


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    yield m
    torch.cuda.empty_cache()


# n * k = 2^30 - 1: every vertex joined to the k after it, cyclically
N, K = 1549411, 693


@pytest.fixture(scope="module")
def circulant():
    ids = torch.arange(N, **I32)
    u = ids.repeat(K)
    v = torch.empty_like(u)
    for d in range(1, K + 1):
        v[(d - 1) * N:d * N] = (ids + d) % N
    return u, v


def check_circulant(g):
    assert (g.m, g.max_degree) == (N * K, 2 * K) and 2 * g.m == 2**31 - 2
    off, adj = g.csr()
    assert torch.equal(off, torch.arange(N + 1, dtype=torch.int64, device="cuda").mul(2 * K).int())
    step = torch.cat([torch.arange(-K, 0, **I32), torch.arange(1, K + 1, **I32)])
    rows = adj.view(N, 2 * K)
    dag_off, dag_adj, dag_src = g.dag()
    deg = dag_off[1:] - dag_off[:-1]
    assert int(dag_off[-1]) == N * K
    for a in range(0, N, 100000):
        z = min(N, a + 100000)
        want = torch.sort((torch.arange(a, z, **I32)[:, None] + step) % N, dim=1).values
        assert torch.equal(rows[a:z], want), a
        # degrees are equal, so an arc points to the larger id
        up = want > torch.arange(a, z, **I32)[:, None]
        assert torch.equal(deg[a:z], up.sum(1, dtype=torch.int32)), a
        lo, hi = int(dag_off[a]), int(dag_off[z])
        assert torch.equal(dag_adj[lo:hi], want[up]), a
        assert torch.equal(dag_src[lo:hi], torch.arange(a, z, **I32).repeat_interleave(deg[a:z])), a


def test_most_arcs(gpm, circulant):
    print("build of 2^31 - 2 arcs", flush=True)
    check_circulant(gpm.Graph.build(N, *circulant))


def test_most_vertices(gpm):
    """Edges at both ends of the id range: the rows of the last share."""
    print("build of 2^31 - 2 vertices", flush=True)
    torch.cuda.empty_cache()
    n = 2**31 - 2
    u = torch.tensor([n - 1, n - 2, n - 1, 0, n - 65], **I32)
    v = torch.tensor([n - 2, n - 70, 0, 1, n - 70], **I32)
    g = gpm.Graph.build(n, u, v)
    assert (g.n, g.m, g.max_degree, g.max_out_degree) == (n, 5, 2, 1)
    off, adj = g.csr()
    assert adj.tolist() == [1, n - 1, 0, n - 65, n - 2, n - 70, n - 70, n - 1, 0, n - 2]
    dag_off, dag_adj, dag_src = g.dag()
    arcs = sorted(zip(dag_src.tolist(), dag_adj.tolist()))
    # degrees: 1 and n - 65 have one, the others two
    assert arcs == [(0, n - 1), (1, 0), (n - 70, n - 2), (n - 65, n - 70), (n - 2, n - 1)]
    for offs, steps in ((off, {0: 2, 1: 1, n - 70: 2, n - 65: 1, n - 2: 2, n - 1: 2}),
                        (dag_off, {0: 1, 1: 1, n - 70: 1, n - 65: 1, n - 2: 1})):
        at, total = 0, 0
        for r, d in sorted(steps.items()):
            part = offs[at:r + 1]
            assert int(part.min()) == int(part.max()) == total
            at, total = r + 1, total + d
        assert int(offs[at:].min()) == int(offs[at:].max()) == total


def test_most_arcs_from_csr(gpm, circulant):
    """The checked adoption of the same CSR: its search in rows that begin
    beyond 2^30."""
    g = gpm.Graph.build(N, *circulant)
    off, adj = (t.clone() for t in g.csr())
    del g
    print("adoption of 2^31 - 2 arcs", flush=True)
    check_circulant(gpm.Graph.from_csr(N, off, adj))
    last = adj[-1].clone()
    adj[-1] = adj[-2]                    # not ascending
    with pytest.raises(gpm.GpmError) as err:
        gpm.Graph.from_csr(N, off, adj)
    assert err.value.status == 6
    adj[-1] = last


def test_searches_beyond_half_the_arcs(gpm):
    """A cycle of 600,000,000 vertices: the searches in its rows add up arc
    numbers above 2^31.  It has as many induced 4-paths and wedges as vertices."""
    torch.cuda.empty_cache()
    n = 600_000_000
    u = torch.arange(n, **I32)
    v = torch.roll(u, -1)
    g = gpm.Graph.build(n, u, v)
    del u, v
    torch.cuda.empty_cache()
    print("patterns of a cycle of 600,000,000 vertices", flush=True)
    assert gpm.count(g, gpm.pattern(4, [(0, 1), (1, 2), (2, 3)], gpm.VERTEX_INDUCED)) == n
    torch.cuda.empty_cache()
    assert gpm.motif_count_enum(g, 3) == [n, 0]
