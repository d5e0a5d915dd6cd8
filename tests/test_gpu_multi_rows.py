"""gr_bfs_multi at the edges of its row tiers (rows of 64 / 65, 2048 / 2049 and more than 8192 neighbours), of the
depths its bit planes hold (15 / 16 and beyond) and of the row widths (k around powers of two, more than one pass)."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1701_01170_amd as gr
    c = gr.Context(0)
    yield c
    c.close()


def tier_graph(seed=3):
    """Hubs with the row lengths at the tiers' edges over 9000 shared leaves, and a path of 40 vertices at one leaf
    (depths up to some 45)."""
    from paper_1701_01170_amd import graphgen as gg
    rng = np.random.default_rng(seed)
    leaves, path = 9000, 40
    edges, hub = [], leaves + path
    for deg in (64, 65, 511, 512, 513, 2048, 2049, 8192, 8193, 8999):
        for v in rng.choice(leaves, deg, replace=False):
            edges.append((hub, int(v)))
        hub += 1
    for i in range(path):
        edges.append((5 if i == 0 else leaves + i - 1, leaves + i))
    return gg.sort_adjacency(gg.from_edges(hub + 1, edges, symmetric=True))  # the last vertex is isolated


@pytest.mark.parametrize("renumber", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3, 16, 33, 64, 70])
def test_tiers_planes_and_widths(ctx, k, renumber):
    import paper_1701_01170_amd as gr
    hg = tier_graph()
    g = gr.Graph.from_host(ctx, hg, symmetric=True, renumber=renumber)
    V = hg.n_vertices
    rng = np.random.default_rng(k)
    srcs = np.concatenate([[V - 12, V - 1, 9039][:k], rng.integers(0, V, max(k - 3, 0))]).astype(np.int32)
    exp = {int(s): oracle.bfs(hg.row_offsets, hg.col_indices, int(s)) for s in set(srcs.tolist())}
    for kw in (dict(), dict(policy=gr.POLICY_FIXED, fixed_action=gr.PULL_TWC),
               dict(policy=gr.POLICY_FIXED, fixed_action=gr.PUSH_LB, device_max_edges=-1),
               dict(max_iterations=16), dict(max_iterations=15)):
        d, p, _ = gr.bfs_multi(g, srcs, opts=gr.default_opts(**kw))
        d0, _, _ = gr.bfs_multi(g, srcs, want_parent=False, opts=gr.default_opts(**kw))
        cap = kw.get("max_iterations", V)
        for i, s in enumerate(srcs.tolist()):
            ed, ep = exp[s]
            np.testing.assert_array_equal(d[i].cpu().numpy(), np.where(ed <= cap, ed, -1), err_msg=f"{kw} {s}")
            np.testing.assert_array_equal(p[i].cpu().numpy(), np.where(ed <= cap, ep, -1), err_msg=f"{kw} {s}")
            np.testing.assert_array_equal(d0[i].cpu().numpy(), np.where(ed <= cap, ed, -1), err_msg=f"{kw} {s}")
    g.free()


@pytest.mark.parametrize("k", [1, 5, 64])
@pytest.mark.parametrize("action", [gr.PUSH_LB, gr.PUSH_TWC])
def test_parents_of_large_pushed_levels(ctx, k, action):
    """Every level pushed: small ones take parents by atomic minima, large ones search them over rows of each length."""
    rng = np.random.default_rng(k)
    hub = [(0, v) for v in range(1, 5000)] + [(1, v) for v in range(2, 1500)] + [(2, v) for v in range(3, 60)]
    e = np.concatenate([np.array(hub), rng.integers(0, 6000, (40000, 2))])
    for h in (gg.rmat(13, 16, seed=31), gg.sort_adjacency(gg.from_edges(6000, e[e[:, 0] != e[:, 1]], symmetric=True))):
        srcs = [int(s) for s in gg.sources(h, k, seed=17)]
        ed, ep = oracle.bfs_multi(h.row_offsets, h.col_indices, srcs)
        for renumber in (False, True):
            g = gr.Graph.from_host(ctx, h, symmetric=True, renumber=renumber)
            o = gr.default_opts(policy=gr.POLICY_FIXED, fixed_action=action, device_max_edges=-1)
            d, p, _ = gr.bfs_multi(g, srcs, opts=o)
            np.testing.assert_array_equal(d.cpu().numpy(), ed)
            np.testing.assert_array_equal(p.cpu().numpy(), ep)
            g.free()
