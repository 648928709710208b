"""The end of a residual network's step in one kernel (last batch norm, pooling, last layer, softmax and back): classes at the edges of a wavefront
and of what the kernel holds (129: the layers one by one), shortcuts of the same and of twice the size, batches from one image up.  The gradient protocol and
bounds of the other network tests."""
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B, inputs       # noqa: E402
from paper_1908_11848_amd.emulation import Emulation        # noqa: E402
from gpu_util import gradient_parity                        # noqa: E402


@pytest.mark.parametrize("model,batch,ncls", [("resnet8", 1, 2), ("resnet8", 13, 7), ("resnet14", 5, 64), ("resnet14", 3, 65), ("resnet8", 37, 127),
                                              ("resnet8", 128, 128), ("resnet14", 6, 128), ("resnet14", 5, 129)])
def test_gradient(oracle_nn, model, batch, ncls):
    from oracle import nn
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
