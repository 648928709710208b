"""The 3x3 convolutions of a residual network's step work on filters that the step's first kernel has converted; callers of single layers have them
split in the convolution.  Both must give the same bits: the saved activations of a step, in every workgroup size (small batches, 33 to 96 images,
larger ones) and stage, against the raw launchers run on the step's own tensors.  (The d-input's filters: the gradient tests of the networks.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B, inputs       # noqa: E402
from paper_1908_11848_amd.emulation import Emulation        # noqa: E402
from gpu_util import dev, empty, host, stream_ptr           # noqa: E402


@pytest.mark.parametrize("batch", [1, 32, 33, 96, 97, 128])
def test_step_has_the_bits_of_the_single_layers(batch):
    ncls, L, s, eps = 10, B.lib(), stream_ptr(), 1e-5
    w = inputs.init_weights(B.dssp_model_segments(B.model_id("resnet8"), ncls), 4, jitter=0.1).astype(np.float32)
    xs, ys = inputs.batches(4, 1, 1, batch, ncls)
    em = Emulation("resnet8", 1, 0, 0, 0.05, w, batch, ncls, xs, ys)
    B.dssp_pull(em.ctx, 0, em.w_local[0])
    em.step(0, 0)
    act = [em.workspace_tensor(0, 0, i) for i in range(7)]          # stem, then the two of each block
    em.close()
    kind = "large" if batch > 96 else "small" if batch <= 32 else None

    def conv(x, filt, rec, H, C):
        y = empty((batch, H, H, C))
        if kind:
            rc = getattr(L, "dsspk_conv3x3_%s_fwd" % kind)(s, x.data_ptr(), None, 0, None, None, 0.0, None, None, None, filt.data_ptr(), y.data_ptr(),
                                                           rec.data_ptr(), 0, batch, H, C)
        else:
            rc = L.dsspk_conv_fwd(s, x.data_ptr(), filt.data_ptr(), None, y.data_ptr(), batch, H, H, C, C, 3, 3, 1, 1, 0, rec.data_ptr())
        assert rc == 0
        return y

    parts_of = getattr(L, "dsspk_conv3x3_%s_parts" % kind) if kind else lambda N, H, C: L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1)
    at, cin, H = 432 + 32, 16, 32
    for b, C in enumerate((16, 32, 64)):
        H //= 1 if b == 0 else 2
        w1 = dev(w[at:at + 9 * cin * C]); at += 9 * cin * C
        g1, b1 = dev(w[at:at + C]), dev(w[at + C:at + 2 * C]); at += 2 * C
        w2 = dev(w[at:at + 9 * C * C]); at += 9 * C * C
        g2, b2 = dev(w[at:at + C]), dev(w[at + C:at + 2 * C]); at += 2 * C
        parts, M, cin = parts_of(batch, H, C), batch * H * H, C
        rec, rec2, stats = empty(2 * parts * C), empty(2 * parts * C), empty(2 * C)
        below, a1, out = dev(act[2 * b]), dev(act[2 * b + 1]), empty((batch, H, H, C))
        if b == 0:                              # the block's first convolution, through the normalisation in the second one's loader
            c1, c2, got = conv(below, w1, rec, H, C), empty((batch, H, H, C)), empty((batch, H, H, C))
            if kind:
                rc = getattr(L, "dsspk_conv3x3_%s_fwd" % kind)(s, c1.data_ptr(), rec.data_ptr(), parts, g1.data_ptr(), b1.data_ptr(), eps, None, got.data_ptr(),
                                                               stats.data_ptr(), w2.data_ptr(), c2.data_ptr(), rec2.data_ptr(), 0, batch, H, C)
            else:
                rc = L.dsspk_conv_fwd_prebn(s, c1.data_ptr(), rec.data_ptr(), parts, g1.data_ptr(), b1.data_ptr(), eps, None, got.data_ptr(), stats.data_ptr(),
                                            w2.data_ptr(), c2.data_ptr(), rec2.data_ptr(), batch, H, C)
            assert rc == 0
            assert np.array_equal(host(got).ravel(), act[1].ravel()), "16 channels, first convolution"
        else:
            c2 = conv(a1, w2, rec2, H, C)
        if b < 2:
            assert L.dsspk_bn_fwd(s, c2.data_ptr(), g2.data_ptr(), b2.data_ptr(), out.data_ptr(), stats.data_ptr(), rec2.data_ptr(), M, C, eps, 1,
                                  1 if b == 0 else 2, below.data_ptr(), batch, H, H, parts) == 0
        else:
            pooled = empty((batch, C))
            assert L.dsspk_bn_fwd_gap(s, c2.data_ptr(), g2.data_ptr(), b2.data_ptr(), out.data_ptr(), stats.data_ptr(), rec2.data_ptr(), parts,
                                      below.data_ptr(), 1, pooled.data_ptr(), batch, H, C, eps) == 0
        assert np.array_equal(host(out).ravel(), act[2 * b + 2].ravel()), (C, "channels, second convolution")
