"""AlexNet-style steps where the way their wide filters are converted changes: carried by the first layer's kernel, by a launch of its own where that kernel
fills the chip exactly (104 to 128 images with one wide layer, from 95 with two), carried again beyond.  Saved activations and gradients must have the bits that the raw
launchers give on the step's own tensors."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B, inputs       # noqa: E402
from paper_1908_11848_amd.emulation import Emulation        # noqa: E402
from gpu_util import dev, empty, host, stream_ptr           # noqa: E402


@pytest.mark.parametrize("model", ["alexnet_ds", "alexnet_3c"])
@pytest.mark.parametrize("batch", [1, 97, 104, 128, 129])
def test_second_layer_has_the_bits_of_the_single_layers(model, batch):
    ncls, L, s = 10, B.lib(), stream_ptr()
    w = inputs.init_weights(B.dssp_model_segments(B.model_id(model), ncls), 2, jitter=0.1).astype(np.float32)
    xs, ys = inputs.batches(2, 1, 1, batch, ncls)
    em = Emulation(model, 1, 0, 0, 0.01, w, batch, ncls, xs, ys)
    B.dssp_pull(em.ctx, 0, em.w_local[0])
    em.step(0, 0)
    a2 = em.workspace_tensor(0, 0, 1)
    g, _ = em.worker_grad(0)
    em.close()
    X, w1, b1 = dev(xs[0][0]), dev(w[:4800]), dev(w[4800:4864])
    w2, b2 = dev(w[4864:4864 + 102400]), dev(w[4864 + 102400:4864 + 102464])
    a1, p1, arg = empty((batch, 32, 32, 64)), empty((batch, 15, 15, 64)), empty((batch, 15, 15, 64), dtype=__import__("torch").uint8)
    assert L.dsspk_conv_first_pool_fwd(s, X.data_ptr(), w1.data_ptr(), b1.data_ptr(), a1.data_ptr(), p1.data_ptr(), arg.data_ptr(), batch) == 0
    planes = empty(L.dsspk_conv_split_filter_bytes(64, 64, 5) // 4)
    assert L.dsspk_conv_split_filters(s, w2.data_ptr(), planes.data_ptr(), None, 64, 64, 5) == 0
    y = empty((batch, 15, 15, 64))
    assert L.dsspk_conv_split_fwd(s, p1.data_ptr(), planes.data_ptr(), b2.data_ptr(), y.data_ptr(), batch, 15, 15, 64, 64, 5, 2, 1) == 0
    assert np.array_equal(host(y).ravel(), a2.ravel())
    assert np.isfinite(g).all() and all(np.abs(g[lo:hi]).max() > 0 for lo, hi in ((0, 4864), (4864, 107328)))
