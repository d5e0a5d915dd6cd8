"""The pushed passes of gr_bc at every chunk size and where its LDS table fills up: more target vertices than slots,
collisions, rows across chunk ends.  Tolerance as in test_gpu_bc.py: sums of positive terms in another order, relative
error below (levels + largest degree) * 4 * 2^-53 < 1e-9."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return gr.Context(0)


@pytest.fixture(scope="module")
def graph():
    """A source over 12000 middle vertices (more than the table's slots), each with a few of 30000 leaves, every tenth
    leaf also at one of three hubs of the middle level."""
    rng = np.random.default_rng(11)
    mid, leaves = 12000, 30000
    e = [(0, 1 + i) for i in range(mid)]
    for leaf in range(leaves):
        v = 1 + mid + leaf
        e += [(int(1 + m), v) for m in rng.integers(0, mid, 2)]
        if leaf % 10 == 0:
            e.append((1 + leaf // 10 % 3, v))
    return gg.sort_adjacency(gg.from_edges(1 + mid + leaves, np.array(sorted(set(e))), symmetric=True))


@pytest.mark.parametrize("chunk", [0, 512, 1024, 2048, 4096, 8192, 16384])
def test_pushed_passes(ctx, graph, chunk):
    o = gr.default_opts(bc_dir=gr.BC_DIR_PUSH | gr.BC_DIR_PUSH << 2, lb_chunk=chunk, lb_min_avg_degree=0.0)
    for renumber in (False, True):
        g = gr.Graph.from_host(ctx, graph, symmetric=True, renumber=renumber)
        for s in (0, 5, graph.n_vertices - 1):
            eb, es = oracle.bc(graph.row_offsets, graph.col_indices, [s], want_sigma=True)
            b, sig, _ = gr.bc(g, [s], want_sigma=True, opts=o)
            np.testing.assert_array_equal(sig.cpu().numpy(), es)
            err = np.abs(b.cpu().numpy() - eb) / np.maximum(1.0, np.abs(eb))
            assert err.max() <= 1e-9, (s, renumber, int(err.argmax()))
        g.free()
