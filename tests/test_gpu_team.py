"""Blocks of small levels on one XCD's workgroups (k_team): graphs at the edges of its forms (longest row 2, 4, 5, 8: edge
slots per vertex; 9 and more: staged frontier), frontiers and levels at its bounds (2048 staged vertices, 32768 edges,
more than one vertex per workgroup), queue refills, caps inside a block, tracing, two contexts at once."""
import threading

import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return gr.Context(0)


def lattice(rows, cols, steps):
    ids = np.arange(rows * cols).reshape(rows, cols)
    e = []
    for dr, dc in steps:
        a = ids[:rows - dr, max(0, -dc):cols - max(0, dc)]
        e.append(np.stack([a.ravel(), (ids[dr:, max(0, dc):cols + min(0, dc)]).ravel()], 1))
    return gg.add_weights(gg.sort_adjacency(gg.from_edges(rows * cols, np.concatenate(e), symmetric=True)), seed=5)


def tree(fan, n):
    """A root with `fan` children, each with children of its own up to n vertices."""
    e = [((i - 1) // fan, i) for i in range(1, n)]
    return gg.add_weights(gg.sort_adjacency(gg.from_edges(n, e, symmetric=True)), seed=6)


GRAPHS = {
    "path": lambda: lattice(1, 5000, [(0, 1)]),
    "grid": lambda: lattice(150, 97, [(0, 1), (1, 0)]),
    "hex": lambda: lattice(90, 80, [(0, 1), (1, 0), (1, 1)]),
    "king": lambda: lattice(120, 70, [(0, 1), (1, 0), (1, 1), (1, -1)]),
    "knight": lambda: lattice(60, 70, [(0, 1), (1, 0), (1, 1), (1, -1), (2, 1)]),
    "tree9": lambda: tree(9, 20000),      # levels of 1, 9, 81, 729, 6561, ... vertices
    "tree2047": lambda: tree(2047, 40000),
    "tree2049": lambda: tree(2049, 40000),
    "star_edges": lambda: tree(16, 16 + 16 * 16 * 16 * 9),
}


def same(hg, g, srcs, **kw):
    for s in srcs:
        ed, ep = oracle.bfs(hg.row_offsets, hg.col_indices, s)
        d, p, _ = gr.bfs(g, s, opts=gr.default_opts(**kw))
        np.testing.assert_array_equal(d.cpu().numpy(), ed, err_msg=f"{kw} {s}")
        np.testing.assert_array_equal(p.cpu().numpy(), ep, err_msg=f"{kw} {s}")
        edist, epred = oracle.sssp(hg.row_offsets, hg.col_indices, hg.weights, [s])
        for delta in (0, 16, 100):
            t, r, _ = gr.sssp(g, [s], opts=gr.default_opts(sssp_delta=delta, **kw))
            np.testing.assert_array_equal(t.cpu().numpy().view(np.uint32), edist, err_msg=f"{kw} {s} {delta}")
            np.testing.assert_array_equal(r.cpu().numpy(), epred, err_msg=f"{kw} {s} {delta}")


@pytest.mark.parametrize("name", list(GRAPHS))
def test_forms(ctx, name):
    hg = GRAPHS[name]()
    for symmetric, renumber in ((True, False), (True, True), (False, False)):
        g = gr.Graph.from_host(ctx, hg, symmetric=symmetric, renumber=renumber)
        srcs = [0, hg.n_vertices // 2, hg.n_vertices - 1]
        same(hg, g, srcs)
        same(hg, g, srcs[:1], device_max_edges=100)
        same(hg, g, srcs[:1], graph_blocks=1)
        buf = (gr.LevelTrace * 8192)()
        same(hg, g, srcs[:1], trace=buf, trace_capacity=8192)
        g.free()


@pytest.mark.parametrize("cap", [1, 2, 63, 64, 65, 4095, 4096, 4097])
def test_caps(ctx, cap):
    hg = GRAPHS["path"]()
    g = gr.Graph.from_host(ctx, hg, symmetric=True)
    ed, _ = oracle.bfs(hg.row_offsets, hg.col_indices, 0)
    d, _, st = gr.bfs(g, 0, opts=gr.default_opts(max_iterations=cap))
    np.testing.assert_array_equal(d.cpu().numpy(), np.where(ed <= cap, ed, -1))
    assert st["iterations"] == cap
    g.free()


def test_two_contexts_at_once():
    import torch
    hg = GRAPHS["grid"]()
    errors = []

    def work(k):
        try:
            c = gr.Context(0)
            g = gr.Graph.from_host(c, hg, symmetric=True)
            stream = torch.cuda.Stream()
            for i in range(6):
                s = (k * 977 + i * 131) % hg.n_vertices
                with torch.cuda.stream(stream):
                    d, p, _ = gr.bfs(g, s, stream=stream)
                    ed, ep = oracle.bfs(hg.row_offsets, hg.col_indices, s)
                    np.testing.assert_array_equal(d.cpu().numpy(), ed)
                    np.testing.assert_array_equal(p.cpu().numpy(), ep)
            g.free()
            c.close()
        except BaseException as e:  # noqa: BLE001  (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
