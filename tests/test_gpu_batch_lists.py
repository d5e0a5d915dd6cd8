"""Batched calls where their lists are collected and split: a wavefront's list for the far pile or the next frontier over
more than its room (stars and wide trees), the pull's rows of the wavefront tier one and several at a time.  Equal to the
oracle."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return gr.Context(0)


def tree(fan, n):
    i = np.arange(1, n)
    return gg.sort_adjacency(gg.from_edges(n, np.stack([(i - 1) // fan, i], 1), symmetric=True))


@pytest.mark.parametrize("make", [lambda: tree(69999, 70000), lambda: tree(40, 70000), lambda: tree(300, 20000)],
                         ids=["star", "tree40", "tree300"])
def test_sssp_lists(ctx, make):
    h = gg.add_weights(make(), seed=41)
    srcs = [0, 1, h.n_vertices - 1, h.n_vertices // 2, 2, 3, 41, 7, 8, 9, 10, 11, 12, 13, 14, 15]
    exp = [oracle.sssp(h.row_offsets, h.col_indices, h.weights, [s]) for s in srcs]
    g = gr.Graph.from_host(ctx, h, symmetric=True)
    for k in (1, 6, 16):
        for kw in ({}, dict(sssp_delta=1), dict(sssp_delta=33), dict(sssp_delta=33, lb_chunk=2048), dict(lb_chunk=2048)):
            d, p, _ = gr.sssp_multi(g, srcs[:k], opts=gr.default_opts(**{"lb_chunk": 1024, **kw}))
            np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), np.stack([x for x, _ in exp[:k]]))
            np.testing.assert_array_equal(p.cpu().numpy(), np.stack([x for _, x in exp[:k]]))
    g.free()


@pytest.mark.parametrize("n,degree", [(300, 90), (9000, 70), (20000, 100)])  # rows per turn: 1, 1 and 2, 3
def test_bfs_rows_of_the_wavefront_tier(ctx, n, degree):
    rng = np.random.default_rng(n)
    h = gg.sort_adjacency(gg.from_edges(n, rng.integers(0, n, (n * degree // 2, 2)), symmetric=True))
    srcs = [int(s) for s in gg.sources(h, 64, seed=3)]
    exp = [oracle.bfs(h.row_offsets, h.col_indices, s) for s in srcs]
    g = gr.Graph.from_host(ctx, h, symmetric=True)
    for k in (1, 7, 64):
        for kw in ({}, dict(policy=gr.POLICY_FIXED, fixed_action=gr.PULL_TWC),
                   dict(policy=gr.POLICY_FIXED, fixed_action=gr.PUSH_LB, device_max_edges=-1)):
            d, p, _ = gr.bfs_multi(g, srcs[:k], opts=gr.default_opts(**kw))
            np.testing.assert_array_equal(d.cpu().numpy(), np.stack([x for x, _ in exp[:k]]))
            np.testing.assert_array_equal(p.cpu().numpy(), np.stack([x for _, x in exp[:k]]))
    g.free()
