"""The distance-ordered frontier of gr_sssp at the edges of its work split: vertices around a thread's and a workgroup's
share, one bin that takes everything and more bins than fit, many binned iterations.  Whole numbers: equal to the oracle."""
import numpy as np
import pytest

import oracle
import paper_1701_01170_amd as gr
from paper_1701_01170_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return gr.Context(0)


@pytest.mark.parametrize("n", [7, 8, 9, 2047, 2048, 2049, 2055, 16384, 50003])
@pytest.mark.parametrize("lo,hi", [(1, 1), (1, 64), (1, 40000)])
def test_equals_oracle(ctx, n, lo, hi):
    h = gg.add_weights(gg.erdos_renyi(n, 6, seed=n), seed=4, lo=lo, hi=hi)
    srcs = [0, n // 2, n - 1]
    for renumber in (False, True):
        g = gr.Graph.from_host(ctx, h, symmetric=True, renumber=renumber)
        for s in (srcs[:1], srcs):
            ed, ep = oracle.sssp(h.row_offsets, h.col_indices, h.weights, s)
            for kw in ({}, dict(device_max_edges=-1), dict(device_max_edges=-1, sssp_opt_off=gr.SSSP_OPT_CULL),
                       dict(device_max_edges=-1, policy=gr.POLICY_FIXED, fixed_action=gr.PUSH_TWC)):
                d, p, _ = gr.sssp(g, s, opts=gr.default_opts(**kw))
                np.testing.assert_array_equal(d.cpu().numpy().view(np.uint32), ed, err_msg=str(kw))
                np.testing.assert_array_equal(p.cpu().numpy(), ep, err_msg=str(kw))
        g.free()
