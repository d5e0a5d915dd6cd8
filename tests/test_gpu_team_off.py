"""Teams of workgroups (k_team) that are called off: with a poll limit of 0 no team forms, every kernel of a block still
ends, and the block's other kernels run the levels.  Outputs equal to the oracle."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu

GRAPHS = {
    "grid": lambda: gg.grid(60, 71),                 # sliced frontiers
    "rmat": lambda: gg.rmat(11, 8, seed=4),          # staged ones
    "path": lambda: gg.grid(1, 700),                 # many blocks
}


@pytest.fixture(scope="module")
def no_teams():
    with pytest.MonkeyPatch.context() as m:
        m.setenv("GR_TEAM_POLLS", "0")
        return gr.Context(0)


@pytest.mark.parametrize("name", list(GRAPHS))
def test_called_off_equals_oracle(no_teams, name):
    hg = gg.add_weights(gg.sort_adjacency(GRAPHS[name]()), seed=3)
    s = int(gg.sources(hg, 1, seed=2)[0])
    ed, ep = oracle.bfs(hg.row_offsets, hg.col_indices, s)
    edist, epred = oracle.sssp(hg.row_offsets, hg.col_indices, hg.weights, [s])
    for symmetric in (True, False):
        g = gr.Graph.from_host(no_teams, hg, symmetric=symmetric)
        for kw in ({}, dict(graph_blocks=1), dict(max_iterations=4 * hg.n_vertices)):
            d, p, _ = gr.bfs(g, s, opts=gr.default_opts(**kw))
            np.testing.assert_array_equal(d.cpu().numpy(), ed)
            np.testing.assert_array_equal(p.cpu().numpy(), ep)
            for delta in (0, 40):
                t, r, _ = gr.sssp(g, [s], opts=gr.default_opts(sssp_delta=delta, **kw))
                np.testing.assert_array_equal(t.cpu().numpy().view(np.uint32), edist)
                np.testing.assert_array_equal(r.cpu().numpy(), epred)
        g.free()


def test_one_try_per_call(no_teams):
    """The first team that cannot form is the last one that a call waits for; where teams form, they run the levels."""
    hg = gg.add_weights(GRAPHS["path"](), seed=3)
    for ctx, off in ((no_teams, True), (gr.Context(0), False)):
        g = gr.Graph.from_host(ctx, hg, symmetric=True)
        for kw in ({}, dict(graph_blocks=1)):
            stats = [gr.bfs(g, 0, opts=gr.default_opts(**kw))[2]]
            stats += [gr.sssp(g, [0], opts=gr.default_opts(sssp_delta=d, **kw))[2] for d in (0, 40)]
            for st in stats:
                assert st["team_levels"] == -1 if off else st["team_levels"] > st["iterations"] // 2, (kw, st)
        g.free()
