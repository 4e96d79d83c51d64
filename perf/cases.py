"""The library's work as a user's program has it done, case by case.

A case is one call of the public entry points on a seeded synthetic graph:

  build     raw edge stream -> canonical CSR and degree-ordered DAG
  cliques   k-cliques of one size (k = 3: triangles)
  fused     the 3-, 4- .. kmax-cliques in one pass
  motifs    induced 3- or 4-motif counts by local counting
  motifs5   the 21 induced 5-motif counts by formulas
  batch     3- or 4-motif counts of many small graphs at once
  list      listing of diamonds, 4-cycles, triangles or 4-cliques
  pattern   a vertex-induced pattern on the general plan

Graphs are power-law ("rmat": a, b, c, d = 0.57, 0.19, 0.19, 0.05, the ids
permuted) or uniform ("er"): `n` vertices, not always a power of two, and a
raw stream of random pairs, repeats and self-loops among them, up to the one
that completes `edges` distinct edges.  Graphs are drawn on the GPU from the
seed alone.
"""
import math

import torch

import paper_2011_03135_amd as gpm

_PATTERNS = {
    "4-path": (4, [(0, 1), (1, 2), (2, 3)]),
    "4-cycle": (4, [(0, 1), (1, 2), (2, 3), (3, 0)]),
}


def listed():
    return [
        # loading: the largest graph of the benchmark, its raw stream to a graph handle
        {"name": "build rmat20", "op": "build", "graph": "rmat", "n": 1 << 20, "edges": 1 << 24},
        # the headline counts on a large power-law graph
        {"name": "triangles rmat20", "op": "cliques", "k": 3, "graph": "rmat", "n": 1 << 20,
         "edges": 1 << 24, "kept": True},
        {"name": "3-4-5-cliques rmat20", "op": "fused", "k": 5, "graph": "rmat", "n": 1 << 20,
         "edges": 1 << 24, "kept": True},
        # the same counts on an ordinary graph, and its size is no power of two
        {"name": "4-cliques rmat 100003", "op": "cliques", "k": 4, "graph": "rmat", "n": 100003,
         "edges": 1600003, "kept": True},
        # a sparse graph without hubs: many short rows instead of a few long ones
        {"name": "triangles er 3000001", "op": "cliques", "k": 3, "graph": "er", "n": 3000001,
         "edges": 24000000, "kept": True},
        # the smallest calls: one request's counts, the answer on the host
        {"name": "3-motifs er4096", "op": "motifs", "k": 3, "graph": "er", "n": 4096,
         "edges": 33767, "kept": False},
        {"name": "4-motifs rmat12", "op": "motifs", "k": 4, "graph": "rmat", "n": 1 << 12,
         "edges": 1 << 16, "kept": False},
        # motif counts of a larger resident graph
        {"name": "4-motifs rmat18", "op": "motifs", "k": 4, "graph": "rmat", "n": 1 << 18,
         "edges": 1 << 22, "kept": True},
        {"name": "5-motifs rmat13", "op": "motifs5", "graph": "rmat", "n": 1 << 13,
         "edges": 1 << 17, "kept": True},
        # a data set of small graphs, the whole of it in one call
        {"name": "batch 20000 4-motifs", "op": "batch", "k": 4, "graphs": 20000},
        # listing into a bounded buffer, with the total and the checksum of all of them
        {"name": "list 4-cycles rmat15", "op": "list", "pattern": "4-cycle", "graph": "rmat",
         "n": 1 << 15, "edges": 1 << 19, "cap": 1 << 20},
        # a pattern that no specialised plan covers
        {"name": "induced 4-path rmat12", "op": "pattern", "pattern": "4-path", "graph": "rmat",
         "n": 1 << 12, "edges": 1 << 16, "kept": True},
    ]


def _between(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _drawn_graph(rng, lo, hi, per_vertex=(6.0, 16.0)):
    n = _between(rng, lo, hi)
    return {"graph": rng.choice(["rmat", "rmat", "er"]), "n": n,
            "edges": int(n * rng.uniform(*per_vertex))}


def draw(rng):
    op = rng.choice(["build", "cliques", "fused", "motifs", "motifs", "motifs5", "batch", "list",
                     "pattern"])
    if op == "build":
        return {"op": op, **_drawn_graph(rng, 1000, 1 << 20)}
    if op == "cliques":
        return {"op": op, "k": rng.choice([3, 4, 5]), **_drawn_graph(rng, 1000, 1 << 20),
                "kept": rng.random() < 0.5}
    if op == "fused":
        return {"op": op, "k": rng.choice([4, 5]), **_drawn_graph(rng, 1000, 1 << 20),
                "kept": rng.random() < 0.5}
    if op == "motifs":
        return {"op": op, "k": rng.choice([3, 4]), **_drawn_graph(rng, 500, 1 << 18),
                "kept": rng.random() < 0.5}
    if op == "motifs5":
        return {"op": op, **_drawn_graph(rng, 500, 1 << 13), "kept": rng.random() < 0.5}
    if op == "batch":
        return {"op": op, "k": rng.choice([3, 4]), "graphs": _between(rng, 100, 20000)}
    if op == "list":
        return {"op": op, "pattern": rng.choice(["diamond", "4-cycle", "3-clique", "4-clique"]),
                **_drawn_graph(rng, 1000, 1 << 15), "cap": _between(rng, 1 << 12, 1 << 20)}
    return {"op": op, "pattern": rng.choice(sorted(_PATTERNS)), **_drawn_graph(rng, 500, 1 << 12),
            "kept": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs ---

def _pairs(case, gen, count):
    """`count` random vertex pairs (int64)."""
    n = case["n"]
    if case["graph"] == "er":
        return (torch.randint(0, n, (count,), generator=gen, device="cuda"),
                torch.randint(0, n, (count,), generator=gen, device="cuda"))
    scale = max(1, (n - 1).bit_length())
    u = torch.zeros(count, dtype=torch.int64, device="cuda")
    v = torch.zeros(count, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        r = torch.rand(count, generator=gen, device="cuda")
        bu = r >= 0.76                                   # quadrants c, d
        bv = ((r >= 0.57) & (r < 0.76)) | (r >= 0.95)    # quadrants b, d
        u = (u << 1) | bu
        v = (v << 1) | bv
    return (u * n) >> scale, (v * n) >> scale


def _stream(case, seed):
    """The raw edge stream (u, v), int32 on the GPU."""
    n, want = case["n"], case["edges"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    perm = torch.randperm(n, generator=gen, device="cuda")
    u = v = torch.empty(0, dtype=torch.int64, device="cuda")
    while True:
        more = _pairs(case, gen, want // 4 + 64 if u.numel() else int(1.1 * want) + 64)
        u, v = torch.cat([u, more[0]]), torch.cat([v, more[1]])
        key, at = torch.sort(torch.minimum(u, v) * n + torch.maximum(u, v), stable=True)
        first = torch.ones_like(key, dtype=torch.bool)
        first[1:] = key[1:] != key[:-1]
        at = at[first & (key // n != key % n)]           # first entry of each distinct edge
        if at.numel() >= want:
            cut = int(torch.sort(at).values[want - 1].item()) + 1
            return perm[u[:cut]].int(), perm[v[:cut]].int()


def _small_graphs(count, seed):
    """Random geometric graphs in the unit square, 10 to 200 vertices and a
    mean degree of 3 to 8 each, plus a tenth as many random edges: the raw
    stream of their union and each graph's first vertex."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    size = torch.randint(10, 201, (count,), generator=gen, device="cuda")
    voff = torch.zeros(count + 1, dtype=torch.int64, device="cuda")
    voff[1:] = torch.cumsum(size, 0)
    degree = 3.0 + 5.0 * torch.rand(count, generator=gen, device="cuda")
    r2 = degree / (math.pi * (size - 1))
    us, vs = [], []
    ids = torch.arange(200, device="cuda")
    upper = ids[:, None] < ids[None, :]
    for g0 in range(0, count, 1000):
        g1 = min(count, g0 + 1000)
        at = torch.rand(g1 - g0, 200, 2, generator=gen, device="cuda")
        dx = at[:, :, None, 0] - at[:, None, :, 0]
        dy = at[:, :, None, 1] - at[:, None, :, 1]
        near = (dx * dx + dy * dy < r2[g0:g1, None, None]) & upper
        near &= (ids < size[g0:g1, None])[:, None, :]
        g, a, b = near.nonzero(as_tuple=True)
        more = torch.randint(0, max(1, g.numel()), (g.numel() // 10,), generator=gen, device="cuda")
        ga = g[more]
        span = size[g0:g1][ga]
        ea = (torch.rand(ga.numel(), generator=gen, device="cuda") * span).long()
        eb = (torch.rand(ga.numel(), generator=gen, device="cuda") * span).long()
        base = voff[g0:g1]
        us += [a + base[g], torch.minimum(ea, span - 1) + base[ga]]
        vs += [b + base[g], torch.minimum(eb, span - 1) + base[ga]]
    return (int(voff[-1].item()), torch.cat(us).int(), torch.cat(vs).int(),
            voff.to(torch.int32))


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    op = case["op"]
    s = {"op": op, "k": case.get("k", 0)}
    if op == "batch":
        n, u, v, s["voff"] = _small_graphs(case["graphs"], seed)
        s["graph"] = gpm.Graph.build(n, u, v)
        return s
    u, v = _stream(case, seed)
    if op == "build":
        # a loader keeps its buffers
        gb, sb = gpm.Graph.build_bytes(case["n"], u.numel())
        s.update(n=case["n"], u=u, v=v, storage=_bytes(gb), scratch=_bytes(sb))
        return s
    g = s["graph"] = gpm.Graph.build(case["n"], u, v)
    if op == "list":
        s["cap"] = case["cap"]
        name = case["pattern"]
        s["pattern"] = (gpm.diamond(gpm.EDGE_INDUCED | gpm.LIST) if name == "diamond"
                        else gpm.cycle4(gpm.EDGE_INDUCED | gpm.LIST) if name == "4-cycle"
                        else gpm.clique(int(name[0]), gpm.VERTEX_INDUCED | gpm.LIST))
        return s
    if op == "cliques":
        s["pattern"] = gpm.clique(case["k"])
    if op == "pattern":
        k, edges = _PATTERNS[case["pattern"]]
        s["pattern"] = gpm.pattern(k, edges, gpm.VERTEX_INDUCED)
    s["ws"] = s["out"] = None
    if case["kept"]:
        # a program that counts again and again keeps its workspace and its
        # result on the device; the others take the answer on the host
        need, width = {
            "cliques": lambda: (gpm.workspace_bytes(g, s["pattern"]), 1),
            "pattern": lambda: (gpm.workspace_bytes(g, s["pattern"]), 1),
            "fused": lambda: (gpm.binding.clique_counts_workspace_bytes(g, case["k"]),
                              case["k"] - 2),
            "motifs": lambda: (gpm.motif_workspace_bytes(g, case["k"]),
                               3 if case["k"] == 3 else 7),
            "motifs5": lambda: (gpm.motif_formula_workspace_bytes(g, 5), 22),
        }[op]()
        s["ws"] = _bytes(need)
        s["out"] = torch.zeros(width, dtype=torch.int64, device="cuda")
    return s


# --------------------------------------------------------------------- run ---

def _low(x):
    """Host counts as 64-bit words (a count may fill all 64 bits)."""
    return x - (1 << 64) if x >= 1 << 63 else x


def run(s):
    op = s["op"]
    if op == "build":
        g = gpm.Graph.build(s["n"], s["u"], s["v"], scratch=s["scratch"], storage=s["storage"])
        return [*g.csr(), *g.dag()]
    g = s["graph"]
    if op == "batch":
        return gpm.batch_motif_count(g, s["voff"], s["k"])
    if op == "list":
        # the rows come in any order, so the order-free checksum over every
        # embedding stands for them
        total, written, checksum, _ = gpm.list_embeddings(g, s["pattern"], s["cap"])
        return [_low(total), written, _low(checksum)]
    if op in ("cliques", "pattern"):
        got = gpm.count(g, s["pattern"], ws=s["ws"], out=s["out"])
    elif op == "fused":
        got = gpm.clique_counts(g, s["k"], ws=s["ws"], out=s["out"])
    elif op == "motifs":
        got = gpm.motif_count(g, s["k"], ws=s["ws"], out=s["out"])
    else:
        got = gpm.motif_count_formula(g, 5, ws=s["ws"], out=s["out"])
    if isinstance(got, torch.Tensor):
        return got
    return [_low(x) for x in got] if isinstance(got, list) else _low(got)


# -------------------------------------------------------------------- work ---

def work(case):
    """Bytes of the inputs read once and the outputs written once (of a raw
    stream its distinct edges).  Counting is whole numbers and bits: no
    floating-point operations."""
    if case["op"] == "batch":
        # 105 vertices and 290 edges a graph on average
        arcs, width = 580 * case["graphs"], 3 if case["k"] == 3 else 7
        return {"bytes": 4 * arcs + 4 * 106 * case["graphs"] + 8 * width * case["graphs"],
                "flops": 0}
    n, m = case["n"], case["edges"]
    if case["op"] == "build":
        return {"bytes": 8 * m + 16 * m + 8 * (n + 1), "flops": 0}
    if case["op"] in ("cliques", "fused"):
        return {"bytes": 4 * m + 4 * (n + 1) + 24, "flops": 0}
    rows = 16 * case["cap"] if case["op"] == "list" else 0
    return {"bytes": 8 * m + 4 * (n + 1) + 176 + rows, "flops": 0}


# ------------------------------------------------------------------- exact ---

def _canonical(n, u, v):
    """Canonical CSR and degree-ordered DAG of a raw stream, in 64 bits."""
    u, v = u.long(), v.long()
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    a, b = key // n, key % n
    deg = torch.bincount(a, minlength=n)
    up = (deg[a] < deg[b]) | ((deg[a] == deg[b]) & (a < b))

    def offsets(src):
        off = torch.zeros(n + 1, dtype=torch.int64, device=src.device)
        off[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
        return off

    return [offsets(a), b, offsets(a[up]), b[up], a[up]]


def exact(case, seed):
    if case["op"] == "build":
        return _canonical(case["n"], *_stream(case, seed))
    if case["op"] == "motifs" and case["k"] == 3 and case["n"] <= 1 << 13:
        off, adj = _canonical(case["n"], *_stream(case, seed))[:2]
        deg = off[1:] - off[:-1]
        a = torch.zeros(case["n"], case["n"], dtype=torch.float64, device="cuda")
        a[torch.repeat_interleave(torch.arange(case["n"], device="cuda"), deg), adj] = 1.0
        tri = int(((a @ a) * a).sum().item()) // 6
        counts = [int((deg * (deg - 1) // 2).sum().item()) - 3 * tri, tri]
        return torch.tensor(counts + [0]) if case["kept"] else counts
    return None
