"""gr_sssp's relaxation with the hubs' mirror in LDS: rows at and around the uniform batches, fewer vertices than the
table has entries and more, ends in it and beyond it, the largest weights that its size allows.  Whole numbers: equal to
the oracle."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return gr.Context(0)


def hubs_and_leaves(n, hub_degrees, per_leaf, seed):
    """Hub h at hub_degrees[h] random ones of n leaves; a few hubs at every leaf, so that the leaves' rows are long."""
    rng = np.random.default_rng(seed)
    e = []
    for h, d in enumerate(hub_degrees):
        e.append(np.stack([np.full(d, h), len(hub_degrees) + rng.permutation(n)[:d]], 1))
    for h in range(per_leaf):
        e.append(np.stack([np.full(n, len(hub_degrees) + n + h), len(hub_degrees) + np.arange(n)], 1))
    g = gg.from_edges(len(hub_degrees) + n + per_leaf, np.concatenate(e), symmetric=True)
    return gg.sort_adjacency(g)


@pytest.mark.parametrize("n,hubs,per_leaf,wmax", [
    (70000, [1, 63, 64, 65, 191, 192, 193, 511, 512, 513, 1024, 1025, 5000], 70, 64),   # all ends in the table
    (131072, [], 66, 200), (200000, [3, 100, 700, 70000], 40, 64),                       # most ends beyond it
    (70000, [200, 2000], 70, 61000)])
def test_equals_oracle(ctx, n, hubs, per_leaf, wmax):
    h = gg.add_weights(hubs_and_leaves(n, hubs, per_leaf, n + per_leaf), seed=3, lo=1, hi=wmax)
    g = gr.Graph.from_host(ctx, h, symmetric=True, renumber=True)
    for src in (len(hubs) + 5, h.n_vertices - 1):
        ed, ep = oracle.sssp(h.row_offsets, h.col_indices, h.weights, [src])
        for delta in (0, wmax // 2):
            d, p, _ = gr.sssp(g, src, opts=gr.default_opts(sssp_delta=delta))
            np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), ed)
            np.testing.assert_array_equal(p.cpu().numpy(), ep)
    g.free()
