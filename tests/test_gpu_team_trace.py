"""Traced calls run the same teams as untraced ones, and their records say what the levels held: a tree whose fourth level
has more vertices than the staged form takes (2048), meshes of each slot count, against the oracle's levels."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return gr.Context(0)


def tree7():
    n = 1 + 7 + 49 + 343 + 2401
    return gg.sort_adjacency(gg.from_edges(n, [((i - 1) // 7, i) for i in range(1, n)], symmetric=True))


@pytest.mark.parametrize("make", [tree7, lambda: gg.grid(1, 300), lambda: gg.grid(70, 33)], ids=["tree7", "path", "grid"])
def test_records_and_form(ctx, make):
    hg = gg.add_weights(make(), seed=9)
    g = gr.Graph.from_host(ctx, hg, symmetric=True)
    for call in (lambda o: gr.bfs(g, 0, opts=o)[2], lambda o: gr.sssp(g, [0], opts=o)[2]):
        buf = (gr.LevelTrace * 2048)()
        plain = call(gr.default_opts())
        traced = call(gr.default_opts(trace=buf, trace_capacity=2048))
        assert plain["team_levels"] == plain["iterations"] == traced["team_levels"] == traced["iterations"]
    depth, _ = oracle.bfs(hg.row_offsets, hg.col_indices, 0)
    deg = np.diff(hg.row_offsets)
    o = gr.default_opts(trace=buf, trace_capacity=2048)
    gr.bfs(g, 0, opts=o)
    assert o.trace_count == depth.max() + 1
    for t in buf[:o.trace_count]:
        level = deg[depth == t.level]
        assert (t.n_f, t.m_f, t.max_deg_f) == (level.size, level.sum(), level.max()), t.level
    g.free()
