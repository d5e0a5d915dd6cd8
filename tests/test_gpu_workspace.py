"""The arrays that a batched call can do without: refused by a bound on the context's working memory, the call takes the
other path; held by it, they are given back where another call needs the room.  Outputs equal to the oracle."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def context(limit_kb):
    with pytest.MonkeyPatch.context() as m:
        if limit_kb:
            m.setenv("GR_WORKSPACE_LIMIT_KB", str(limit_kb))
        return gr.Context(0)


@pytest.fixture(scope="module")
def cases():
    out = []
    for hg in (gg.rmat(12, 12, seed=5), gg.grid(40, 30)):  # the grid is deeper than the depth planes hold
        hg = gg.add_weights(gg.sort_adjacency(hg), seed=4)
        srcs = [int(s) for s in gg.sources(hg, 64, seed=6)]
        b = [oracle.bfs(hg.row_offsets, hg.col_indices, s) for s in srcs]
        t = [oracle.sssp(hg.row_offsets, hg.col_indices, hg.weights, [s]) for s in srcs[:16]]
        out.append((hg, srcs, [np.stack(x) for x in zip(*b)], [np.stack(x) for x in zip(*t)]))
    return out


def bfs(g, srcs, exp):
    d, p, _ = gr.bfs_multi(g, srcs)
    np.testing.assert_array_equal(d.cpu().numpy(), exp[0])
    np.testing.assert_array_equal(p.cpu().numpy(), exp[1])


def sssp(g, srcs, exp):
    d, p, _ = gr.sssp_multi(g, srcs[:16], opts=gr.default_opts(lb_chunk=1024))
    np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), exp[0])
    np.testing.assert_array_equal(p.cpu().numpy(), exp[1])


@pytest.mark.parametrize("renumber", [False, True])
@pytest.mark.parametrize("i", [0, 1])
def test_every_limit(cases, i, renumber):
    """From too little for any call up to room for everything: GR_ENOMEM up to some limit, right outputs from there on.
    What both calls cannot do without is some 290 bytes per vertex with the head-room; the batched BFS holds 320 more
    where they fit, which the second call then has to get."""
    hg, srcs, eb, es = cases[i]
    V = hg.n_vertices
    fits = set()
    for per_vertex in range(50, 700, 25):
        limit = per_vertex * V >> 10
        for order in ((bfs, eb), (sssp, es)), ((sssp, es), (bfs, eb)):
            ctx = context(limit)
            g = gr.Graph.from_host(ctx, hg, symmetric=True, renumber=renumber)
            for call, exp in order:
                try:
                    for _ in range(2):
                        call(g, srcs, exp)
                except gr.GrError as e:
                    assert e.code == gr.GR_ENOMEM and per_vertex < 350, (call, per_vertex)
                    assert call is not order[0][0] or call not in fits, (call, per_vertex)
                else:
                    if call is order[0][0]:
                        fits.add(call)
            g.free()
            ctx.close()
        assert bfs in fits or per_vertex < 250  # without the parent rows
        assert sssp in fits or per_vertex < 350
    assert fits == {bfs, sssp}


def test_no_limit(cases):
    for hg, srcs, eb, es in cases:
        ctx = context(None)
        g = gr.Graph.from_host(ctx, hg, symmetric=True)
        bfs(g, srcs, eb)
        sssp(g, srcs, es)
        g.free()
        ctx.close()
