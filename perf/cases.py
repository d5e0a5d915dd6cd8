"""The traversal work that a program using this framework has it do, as cases that can be timed.

Each case is one call of a public entry point on a resident graph.  Graphs are drawn on the GPU from the seed with the
distributions of `paper_1701_01170_amd.graphgen` (R-MAT a = 0.57, b = c = 0.19, vertices relabelled, symmetrised, no loops
or duplicates; uniform random graphs; 4-neighbour grids; unions of small R-MAT graphs; weights 1..64, one per undirected
edge), since the host generator takes seconds at the larger sizes.

Keys of a case: `kind` (the entry point), `family` with its sizes, `k` (sources), `symmetric` / `renumber` (ingest options)
and `tuned` (the stored knobs of the autotuner, as the benchmark runs, or the library's defaults, as the README's example).
"""
import math

import numpy as np
import torch

import paper_1701_01170_amd as gr
from paper_1701_01170_amd import autotune

RMAT_A, RMAT_B, RMAT_C = 0.57, 0.19, 0.19
_context = None


def _case(name, kind, family, *, k=1, symmetric=True, renumber=False, tuned=False, **sizes):
    return dict({"name": name} if name else {}, kind=kind, family=family, k=k, symmetric=symmetric, renumber=renumber,
                tuned=tuned, **sizes)


def listed():
    return [
        # the smallest call: launches and host round trips count (the smoke test's graph)
        _case("bfs_rmat12", "bfs", "rmat", scale=12, edge_factor=16),
        # ordinary graphs with the defaults: a social-network-like one, and a directed one, where only push steps may run
        _case("bfs_rmat18", "bfs", "rmat", scale=18, edge_factor=16),
        _case("sssp_er_directed", "sssp", "er", n=300007, degree=8, symmetric=False),
        # the benchmark's step: BFS and SSSP on R-MAT 22, degree-renumbered, tuned knobs
        _case("bfs_rmat22", "bfs", "rmat", scale=22, edge_factor=16, renumber=True, tuned=True),
        _case("sssp_rmat22", "sssp", "rmat", scale=22, edge_factor=16, renumber=True, tuned=True),
        # road-like graphs: thousands of levels with small frontiers
        _case("bfs_grid2048", "bfs", "grid", rows=2048, cols=2048, tuned=True),
        _case("sssp_grid768", "sssp", "grid", rows=768, cols=768, tuned=True),
        # many sources on one graph (all-pairs samples, centralities), and many small graphs in one call
        _case("bfs_multi_rmat20", "bfs_multi", "rmat", scale=20, edge_factor=16, k=64, renumber=True, tuned=True),
        _case("sssp_multi_rmat20", "sssp_multi", "rmat", scale=20, edge_factor=16, k=16, renumber=True, tuned=True),
        _case("sssp_union256", "sssp", "union", graphs=256, scale_lo=10, scale_hi=16, ef_lo=8, ef_hi=32, k=256, tuned=True),
        _case("bc_rmat22", "bc", "rmat", scale=22, edge_factor=16, k=4, renumber=True, tuned=True),
        # the largest graph of the benchmark
        _case("sssp_rmat25", "sssp", "rmat", scale=25, edge_factor=16, renumber=True, tuned=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: any kind, family, size and option that a call may have."""
    kind = rng.choice(["bfs", "bfs", "bfs", "sssp", "sssp", "sssp", "bfs_multi", "sssp_multi", "bc"])
    many = kind in ("bfs_multi", "sssp_multi", "bc")
    family = rng.choice(["rmat", "rmat", "er", "grid"] + (["union"] if kind == "sssp" else []))
    tuned, renumber, symmetric = rng.random() < 0.5, rng.random() < 0.5, True
    k = 1
    if kind == "bfs_multi":
        k = _log_int(rng, 2, 64)
    elif kind == "sssp_multi":
        k = _log_int(rng, 2, 16)
    elif kind == "bc":
        k = rng.randint(1, 4)
    if family == "rmat":
        sizes = dict(scale=rng.randint(10, 20 if many else 22), edge_factor=rng.randint(4, 32))
    elif family == "er":
        sizes = dict(n=_log_int(rng, 1000, 1 << (19 if many else 21)), degree=rng.randint(3, 32))
        symmetric = many or rng.random() < 0.5
    elif family == "grid":
        side = 400 if many else 1500
        sizes = dict(rows=_log_int(rng, 20, side), cols=_log_int(rng, 20, side))
        renumber = False
    else:
        graphs = _log_int(rng, 4, 256)
        sizes = dict(graphs=graphs, scale_lo=rng.randint(6, 10), scale_hi=rng.randint(11, 15), ef_lo=rng.randint(4, 8),
                     ef_hi=rng.randint(9, 32))
        k = graphs
    return _case(None, kind, family, k=k, symmetric=symmetric, renumber=renumber, tuned=tuned, **sizes)


# ---- inputs ----------------------------------------------------------------

def _rmat_ends(n_edges, scale, gen):
    """R-MAT end points: one quadrant per bit.  `scale` is a number, or a tensor with each edge's own scale."""
    top = int(scale) if not torch.is_tensor(scale) else int(scale.max())
    u = torch.zeros(n_edges, dtype=torch.int32, device="cuda")
    v = torch.zeros_like(u)
    for bit in range(top):
        r = torch.rand(n_edges, device="cuda", generator=gen)
        down = r >= RMAT_A + RMAT_B
        right = ((r >= RMAT_A) & ~down) | (r >= RMAT_A + RMAT_B + RMAT_C)
        if torch.is_tensor(scale):
            down, right = down & (bit < scale), right & (bit < scale)
        u |= down.int() << bit
        v |= right.int() << bit
    return u, v


def _pairs(case, gen):
    """(number of vertices, sorted int64 keys u * V + v of the directed edges, first vertex of each part)."""
    family, parts = case["family"], None
    if family == "rmat":
        V = 1 << case["scale"]
        n, step, ends = case["edge_factor"] * V, 1 << 26, []
        relabel = torch.randperm(V, device="cuda", generator=gen)
        for at in range(0, n, step):  # in pieces: the temporaries of a large graph stay small
            u, v = _rmat_ends(min(step, n - at), case["scale"], gen)
            ends.append(relabel[u] * V + relabel[v])
        keys = torch.cat(ends)
        del ends
    elif family == "er":
        V = case["n"]
        n = int(V * case["degree"] / (2 if case["symmetric"] else 1))
        keys = torch.randint(V * V, (n,), device="cuda", generator=gen)
    elif family == "grid":
        V = case["rows"] * case["cols"]
        ids = torch.arange(V, device="cuda").view(case["rows"], case["cols"])
        keys = torch.cat([(ids[:, :-1] * V + ids[:, 1:]).reshape(-1), (ids[:-1] * V + ids[1:]).reshape(-1)])
    else:
        pick = np.random.RandomState(7)  # the parts' sizes belong to the case, their edges to the seed
        scales = pick.randint(case["scale_lo"], case["scale_hi"] + 1, case["graphs"])
        factors = pick.randint(case["ef_lo"], case["ef_hi"] + 1, case["graphs"])
        parts = np.concatenate([[0], np.cumsum(1 << scales)])
        V = int(parts[-1])
        part = torch.repeat_interleave(torch.arange(case["graphs"], device="cuda"),
                                       torch.from_numpy(factors * (1 << scales)).cuda())
        u, v = _rmat_ends(part.numel(), torch.from_numpy(scales).cuda()[part].int(), gen)
        first = torch.from_numpy(parts[:-1]).cuda()[part]
        keys = (u + first) * V + (v + first)
    u, v = keys // V, keys % V
    keys = keys[u != v]
    if case["symmetric"]:
        del u, v
        keys = torch.cat([keys, (keys % V) * V + keys // V])
    return V, torch.unique(keys), parts


def _weights(u, v, seed):
    """1 + hash(seed, {u, v}) mod 64: the same for both directions of an edge."""
    h = torch.minimum(u, v) * 0x1E3779B97F4A7C15 + torch.maximum(u, v) * 0x3F58476D1CE4E5B9 + seed
    h = (h ^ (h >> 31)) * 0x14D049BB133111EB
    return (1 + ((h ^ (h >> 29)) & 63)).int()


def prepare(case, seed):
    """The resident graph, its options, the sources and the output buffers."""
    global _context
    if _context is None:
        _context = gr.Context(0)  # one for the process, as a program keeps it
    gen = torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + 17)
    V, keys, parts = _pairs(case, gen)
    kind, k, E = case["kind"], case["k"], keys.numel()
    R = torch.searchsorted(keys, torch.arange(V + 1, device="cuda") * V).int()
    u, v = keys // V, keys % V
    del keys
    C = v.int()
    W = _weights(u, v, int(seed)) if kind in ("sssp", "sssp_multi") else None
    # sources have neighbours: the row of a random edge (of each part's edges, in a union)
    if parts is None:
        at = torch.randint(E, (k,), device="cuda", generator=gen)
    else:
        bounds = R[torch.from_numpy(parts).cuda()].double()
        x = torch.rand(k, device="cuda", generator=gen, dtype=torch.float64)
        at = (bounds[:-1] + x * (bounds[1:] - bounds[:-1])).long()
    sources = u[at].cpu().numpy().astype(np.int32)
    del u, v
    graph = gr.Graph.from_csr(_context, R, C, W, symmetric=case["symmetric"], renumber=case["renumber"])
    opts = autotune.tuned_opts(graph, kind) if case["tuned"] else None
    if kind == "bc":
        out = (torch.empty(V, dtype=torch.float64, device="cuda"), None)
    else:
        shape = (k, V) if kind in ("bfs_multi", "sssp_multi") else (V,)
        out = tuple(torch.empty(shape, dtype=torch.int32, device="cuda") for _ in range(2))
    return {"kind": kind, "graph": graph, "opts": opts, "sources": sources, "out": out}


def run(state):
    """One call.  BFS: depths and parents; SSSP: distances and predecessors; BC: the centralities."""
    graph, sources, opts, out = state["graph"], state["sources"], state["opts"], state["out"]
    if state["kind"] == "bfs":
        gr.bfs(graph, int(sources[0]), opts=opts, out=out)
    elif state["kind"] == "sssp":
        gr.sssp(graph, sources, opts=opts, out=out)
    elif state["kind"] == "bfs_multi":
        gr.bfs_multi(graph, sources, opts=opts, out=out)
    elif state["kind"] == "sssp_multi":
        gr.sssp_multi(graph, sources, opts=opts, out=out)
    else:
        gr.bc(graph, sources, opts=opts, out=out)
        return out[0]
    return out


def _sizes(case):
    """Vertices and (expected) directed edges."""
    if case["family"] == "rmat":
        scales, factors = [case["scale"]], [case["edge_factor"]]
    elif case["family"] == "er":
        return case["n"], case["n"] * case["degree"]
    elif case["family"] == "grid":
        return case["rows"] * case["cols"], 4 * case["rows"] * case["cols"] - 2 * (case["rows"] + case["cols"])
    else:  # every scale alike, the mean edge factor
        scales = list(range(case["scale_lo"], case["scale_hi"] + 1))
        factors = [(case["ef_lo"] + case["ef_hi"]) / 2] * len(scales)
    # the share of generated pairs that are duplicates or loops: 0.186 at scale 14 and factor 16, falling by 2^-0.26 a scale
    E = [2 * f * (1 << s) * (1 - min(0.9, 0.186 * 2 ** (-0.26 * (s - 14)) * (f / 16) ** 0.75)) for s, f in zip(scales, factors)]
    many = case["graphs"] / len(scales) if case["family"] == "union" else 1
    return int(many * sum(1 << s for s in scales)), int(many * sum(E))


def work(case):
    """The graph read once and every output written once; an addition and a comparison per edge and source, and for
    centralities a multiplication and an addition in each of the two passes."""
    V, E = _sizes(case)
    kind, k = case["kind"], case["k"]
    rows = k if kind in ("bfs_multi", "sssp_multi") else 1
    read = 4 * V + (8 if kind in ("sssp", "sssp_multi") else 4) * E
    return {"bytes": read + 8 * V * rows, "flops": {"bc": 4 * k, "bfs": 1, "sssp": 2}.get(kind, 2 * rows) * E}


def exact(case, seed):
    """Centralities in 64 bits, level by level over the edge list; the other kinds return whole numbers."""
    if case["kind"] != "bc":
        return None
    state = prepare(case, seed)
    R, C, _ = state["graph"].export()
    V = R.numel() - 1
    u = torch.repeat_interleave(torch.arange(V, device="cuda"), (R[1:] - R[:-1]).long())
    v = C.long()
    total = torch.zeros(V, dtype=torch.float64, device="cuda")
    for s in state["sources"].tolist():
        depth = torch.full((V,), -1, dtype=torch.int32, device="cuda")
        sigma = torch.zeros(V, dtype=torch.float64, device="cuda")
        depth[s], sigma[s] = 0, 1.0
        steps = []
        while True:
            here = depth[u] == len(steps)
            a, b = u[here], v[here]
            depth[b[depth[b] < 0]] = len(steps) + 1
            on = depth[b] == len(steps) + 1
            a, b = a[on], b[on]
            if not a.numel():
                break
            sigma.index_add_(0, b, sigma[a])
            steps.append((a, b))
        delta = torch.zeros(V, dtype=torch.float64, device="cuda")
        for a, b in reversed(steps):
            delta.index_add_(0, a, sigma[a] / sigma[b] * (1 + delta[b]))
        delta[s] = 0
        total += delta
    return total
