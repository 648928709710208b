"""Stride-2 convolutions of small residual steps, whose gradients come from one kernel that also masks the one to the input and leaves its sum records: batches on
either side of where the kernel behind adds up as many records (16 images with 16 channels, 32 with 32), and the smallest.  The gradient protocol and bounds of the
other network tests."""
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B, inputs       # noqa: E402
from paper_1908_11848_amd.emulation import Emulation        # noqa: E402
from gpu_util import gradient_parity                        # noqa: E402


@pytest.mark.parametrize("model,batch", [("resnet8", 1), ("resnet8", 15), ("resnet8", 16), ("resnet14", 16), ("resnet8", 17), ("resnet8", 32), ("resnet8", 33)])
def test_gradient(oracle_nn, model, batch):
    from oracle import nn
    ncls = 10
    w = inputs.init_weights(B.dssp_model_segments(B.model_id(model), ncls), 4, jitter=0.1)
    xs, ys = inputs.batches(4, 1, 1, batch, ncls)
    em = Emulation(model, 1, 0, 0, 0.05, w, batch, ncls, xs, ys)
    try:
        B.dssp_pull(em.ctx, 0, em.w_local[0])
        for _ in range(3):                      # as launches, as the graph's capture, as a replay
            em.step(0, 0)
        stats = {}
        err, _ = gradient_parity(nn.make_net(model, ncls), em, 0, w, xs[0][0], ys[0][0], stats)
        assert err < 1e-4 and stats["grad_max_abs"] < 1e-3
    finally:
        em.close()
