"""Batched shortest paths where the one-byte distance bounds and the staging can go wrong: bounds that fit and that run
out of range, quanta of 1 and more, rows of each slot count, chunks of more segments than are staged at a time, lists of
pairs longer than one round.  Whole numbers: equal to the oracle."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return gr.Context(0)


def short_rows_behind_hubs():
    """17 hubs over 6000 vertices that each have one to three more neighbours: a chunk of 2048 edges there is of more
    than 256 segments, and every hub's edge is relaxed for all sources at once."""
    rng = np.random.default_rng(5)
    n, h = 6000, 17
    e = [(i, h + j) for i in range(h) for j in range(n) if rng.random() < (0.9 if i == 0 else 0.05)]
    e += [(h + j, h + n + j % 900) for j in range(n)] + [(h + n + j, h + n + 900 + j) for j in range(900)]
    return gg.sort_adjacency(gg.from_edges(h + n + 1800, np.array(e), symmetric=True))


@pytest.mark.parametrize("lo,hi", [(0, 1), (1, 64), (100, 127), (30000, 140000)])
@pytest.mark.parametrize("make", [short_rows_behind_hubs, lambda: gg.rmat(12, 24, seed=9), lambda: gg.grid(40, 41)])
def test_equals_oracle(ctx, make, lo, hi):
    h = gg.add_weights(make(), seed=21, lo=lo, hi=hi)
    srcs = [int(s) for s in gg.sources(h, 20, seed=8)]
    exp = [oracle.sssp(h.row_offsets, h.col_indices, h.weights, [s]) for s in srcs]
    for renumber in (False, True):
        g = gr.Graph.from_host(ctx, h, symmetric=True, renumber=renumber)
        for k, kw in ((4, {}), (7, {}), (20, {}), (20, dict(lb_chunk=2048)), (16, dict(sssp_delta=2 * hi + 1, lb_chunk=512))):
            d, p, _ = gr.sssp_multi(g, srcs[:k], opts=gr.default_opts(**kw))
            np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), np.stack([x for x, _ in exp[:k]]))
            np.testing.assert_array_equal(p.cpu().numpy(), np.stack([x for _, x in exp[:k]]))
        g.free()
