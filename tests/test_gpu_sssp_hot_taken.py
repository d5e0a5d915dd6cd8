"""The inputs of the tests of k_sssp_relax_hot do take it: an iteration in LB mode over a degree-ordered graph with at least
4 M frontier edges, 64 per vertex on average and 16 chunks per CU."""
import numpy as np
import pytest
import torch

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg
from test_gpu_sssp_hot import hubs_and_leaves

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,hubs,per_leaf,wmax", [(70000, [1, 64, 192, 512, 5000], 70, 64), (131072, [], 66, 200)])
def test_rule_met(n, hubs, per_leaf, wmax):
    h = gg.add_weights(hubs_and_leaves(n, hubs, per_leaf, n + per_leaf), seed=3, lo=1, hi=wmax)
    ctx = gr.Context(0)
    g = gr.Graph.from_host(ctx, h, symmetric=True, renumber=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    buf = (gr.LevelTrace * 256)()
    o = gr.default_opts(trace=buf, trace_capacity=256)
    src = len(hubs) + 5
    d, p, _ = gr.sssp(g, src, opts=o)
    hot = [t for t in buf[:o.trace_count]
           if t.kernel == 10 and t.m_f >= 1 << 22 and t.m_f >= 64 * t.n_f and t.m_f >= 16 * cus * 1024]
    assert hot
    ed, ep = oracle.sssp(h.row_offsets, h.col_indices, h.weights, [src])
    np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), ed)
    np.testing.assert_array_equal(p.cpu().numpy(), ep)
    g.free()
