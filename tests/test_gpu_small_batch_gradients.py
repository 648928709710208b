"""Gradients of small residual steps, whose last stage takes d-input and d-filter in one kernel and adds its partial sums up four images at a time: batches
with every remainder of four, the smallest and the largest.  The gradient protocol and bounds of the other network tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B, inputs       # noqa: E402
from paper_1908_11848_amd.emulation import Emulation        # noqa: E402
from gpu_util import gradient_parity                        # noqa: E402


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 9, 31, 32])
def test_gradient(oracle_nn, batch):
    from oracle import nn
    ncls = 10
    w = inputs.init_weights(B.dssp_model_segments(B.model_id("resnet14"), ncls), 4, jitter=0.1)
    xs, ys = inputs.batches(4, 1, 1, batch, ncls)
    em = Emulation("resnet14", 1, 0, 0, 0.05, w, batch, ncls, xs, ys)
    try:
        B.dssp_pull(em.ctx, 0, em.w_local[0])
        for _ in range(3):                      # as launches, as the graph's capture, as a replay
            em.step(0, 0)
        stats = {}
        err, _ = gradient_parity(nn.make_net("resnet14", ncls), em, 0, w, xs[0][0], ys[0][0], stats)
        assert err < 1e-4 and stats["grad_max_abs"] < 1e-3
    finally:
        em.close()
