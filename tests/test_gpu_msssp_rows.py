"""Batched shortest paths on graphs of more than 65536 vertices, where the next frontier is listed by the relaxation (few
edges) or found in tiles of 1024 vertices (many): each with rows of 4, 8 and 16 slots, with and without the queue's far
pile.  Whole numbers: equal to the oracle."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return gr.Context(0)


@pytest.mark.parametrize("make", [lambda: gg.grid(331, 200), lambda: gg.rmat(17, 10, seed=31)], ids=["grid", "rmat17"])
def test_equals_oracle(ctx, make):
    h = gg.add_weights(gg.sort_adjacency(make()), seed=32)
    assert h.n_vertices > 1 << 16
    srcs = [int(s) for s in gg.sources(h, 16, seed=33)]
    exp = [oracle.sssp(h.row_offsets, h.col_indices, h.weights, [s]) for s in srcs]
    for renumber in (False, True):
        g = gr.Graph.from_host(ctx, h, symmetric=True, renumber=renumber)
        for k in (1, 4, 5, 8, 9, 16):
            for kw in ({}, dict(sssp_delta=40), dict(sssp_opt_off=gr.SSSP_OPT_CULL)):
                d, p, _ = gr.sssp_multi(g, srcs[:k], opts=gr.default_opts(lb_chunk=1024, **kw))
                np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), np.stack([x for x, _ in exp[:k]]))
                np.testing.assert_array_equal(p.cpu().numpy(), np.stack([x for _, x in exp[:k]]))
        g.free()
