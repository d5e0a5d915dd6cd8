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
