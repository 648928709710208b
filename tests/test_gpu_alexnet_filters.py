"""AlexNet-style steps where the way their wide filters are converted changes: carried by the first layer's kernel, by a launch of its own where that kernel
fills the chip exactly (104 to 128 images with one wide layer, from 95 with two), carried again beyond.  Every saved activation, the loss and the whole
gradient must have the bits of the step put together from the launchers of single layers, which convert each filter and reduce each filter gradient
by a launch of its own."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B, inputs       # noqa: E402
from paper_1908_11848_amd.emulation import Emulation        # noqa: E402
from gpu_util import dev, empty, host, stream_ptr           # noqa: E402


def single_layers(model, w, x, y, m, ncls):
    """(activations behind each ReLU, logits, loss, gradient)"""
    L, s, three = B.lib(), stream_ptr(), model == "alexnet_3c"
    bytes_ = lambda n: empty(n, dtype=torch.uint8)
    W, g, X, Y = dev(w), empty(w.size), dev(x), dev(y.astype(np.int32))
    at, off = 0, {}
    for name, n in [("w1", 4800), ("b1", 64), ("w2", 102400), ("b2", 64)] + ([("w3", 36864), ("b3", 64)] if three else []) + \
            [("f1", 3136 * 384), ("fb1", 384)] + ([] if three else [("f2", 384 * 192), ("fb2", 192)]):
        off[name] = at
        at += n
    last, n_last = at, 384 if three else 192
    p = lambda t, name: t[off[name]:].data_ptr()

    def ok(rc):
        assert rc == 0

    def planes(name, k):
        f, b = (empty(L.dsspk_conv_split_filter_bytes(64, 64, k) // 4) for _ in range(2))
        ok(L.dsspk_conv_split_filters(s, p(W, name), f.data_ptr(), b.data_ptr(), 64, 64, k))
        return f, b

    def filter_gradient(xi, dy, name, H, k, pad):
        scr = empty(L.dsspk_conv_split_wgrad_scratch_floats(m, H, H, 64, 64, k, pad))
        ok(L.dsspk_conv_split_bwd_weight(s, xi.data_ptr(), dy.data_ptr(), p(g, name), 1, scr.data_ptr(), m, H, H, 64, 64, k, pad))

    f15, f7 = (m, 15, 15, 64), (m, 7, 7, 64)
    a1, p1, arg1 = empty((m, 32, 32, 64)), empty(f15), bytes_(f15)
    ok(L.dsspk_conv_first_pool_fwd(s, X.data_ptr(), p(W, "w1"), p(W, "b1"), a1.data_ptr(), p1.data_ptr(), arg1.data_ptr(), m))
    fwd2, bwd2 = planes("w2", 5)
    a2, p2, arg2 = empty(f15), empty(f7), bytes_(f7)
    ok(L.dsspk_conv_split_fwd(s, p1.data_ptr(), fwd2.data_ptr(), p(W, "b2"), a2.data_ptr(), m, 15, 15, 64, 64, 5, 2, 1))
    ok(L.dsspk_maxpool_fwd(s, a2.data_ptr(), p2.data_ptr(), arg2.data_ptr(), m, 15, 15, 64))
    flat, acts = p2, [a1, a2]
    if three:
        fwd3, bwd3 = planes("w3", 3)
        flat = empty(f7)
        ok(L.dsspk_conv_split_fwd(s, p2.data_ptr(), fwd3.data_ptr(), p(W, "b3"), flat.data_ptr(), m, 7, 7, 64, 64, 3, 1, 1))
        acts.append(flat)
    a3 = empty((m, 384))
    ok(L.dsspk_gemm(s, flat.data_ptr(), 3136, 1, p(W, "f1"), 384, 1, a3.data_ptr(), 384, m, 384, 3136, p(W, "fb1"), 1))
    acts.append(a3)
    if not three:
        acts.append(empty((m, 192)))
        ok(L.dsspk_gemm(s, a3.data_ptr(), 384, 1, p(W, "f2"), 192, 1, acts[-1].data_ptr(), 192, m, 192, 384, p(W, "fb2"), 1))
    z, dz, rows, loss, wl, gl = empty((m, ncls)), empty((m, ncls)), empty(m), empty(1), W[last:], g[last:]
    ok(L.dsspk_fc_softmax_xent(s, acts[-1].data_ptr(), wl.data_ptr(), wl[n_last * ncls:].data_ptr(), Y.data_ptr(), z.data_ptr(), dz.data_ptr(), rows.data_ptr(),
                               m, n_last, ncls))
    d = empty((m, n_last))
    ok(L.dsspk_fc_bwd(s, acts[-1].data_ptr(), dz.data_ptr(), wl.data_ptr(), gl.data_ptr(), gl[n_last * ncls:].data_ptr(), d.data_ptr(), 1, rows.data_ptr(),
                      loss.data_ptr(), m, n_last, ncls))
    if not three:
        d, below = empty((m, 384)), d
        ok(L.dsspk_fc_bwd(s, a3.data_ptr(), below.data_ptr(), p(W, "f2"), p(g, "f2"), p(g, "fb2"), d.data_ptr(), 1, None, None, m, 384, 192))
    dflat = empty(f7)
    ok(L.dsspk_fc_bwd(s, flat.data_ptr(), d.data_ptr(), p(W, "f1"), p(g, "f1"), p(g, "fb1"), dflat.data_ptr(), int(three), None, None, m, 3136, 384))
    dp2 = dflat
    if three:
        filter_gradient(p2, dflat, "w3", 7, 3, 1)
        dp2 = empty(f7)
        ok(L.dsspk_conv_split_bwd_data(s, dflat.data_ptr(), bwd3.data_ptr(), None, dp2.data_ptr(), m, 7, 7, 64, 64, 3, 1))
    da2, dp1 = empty(f15), empty(f15)
    ok(L.dsspk_maxpool_bwd_relu(s, dp2.data_ptr(), arg2.data_ptr(), a2.data_ptr(), da2.data_ptr(), m, 15, 15, 64))
    filter_gradient(p1, da2, "w2", 15, 5, 2)
    ok(L.dsspk_conv_split_bwd_data(s, da2.data_ptr(), bwd2.data_ptr(), None, dp1.data_ptr(), m, 15, 15, 64, 64, 5, 2))
    scr = empty(L.dsspk_conv_first_scratch_floats(m))
    ok(L.dsspk_conv_first_pool_bwd_weight(s, X.data_ptr(), dp1.data_ptr(), p1.data_ptr(), arg1.data_ptr(), p(g, "w1"), scr.data_ptr(), m))
    return [host(a) for a in acts], host(z), host(loss)[0], host(g)


@pytest.mark.parametrize("model", ["alexnet_ds", "alexnet_3c"])
@pytest.mark.parametrize("batch", [1, 94, 97, 104, 128, 129])
def test_step_has_the_bits_of_the_single_layers(model, batch):
    ncls = 10
    w = inputs.init_weights(B.dssp_model_segments(B.model_id(model), ncls), 2, jitter=0.1).astype(np.float32)
    xs, ys = inputs.batches(2, 1, 1, batch, ncls)
    acts, logits, loss, grad = single_layers(model, w, xs[0][0].astype(np.float32), ys[0][0], batch, ncls)
    em = Emulation(model, 1, 0, 0, 0.01, w, batch, ncls, xs, ys)
    try:
        B.dssp_pull(em.ctx, 0, em.w_local[0])
        for way in ("launches", "captured", "replayed"):
            em.grad.fill_(float("nan"))
            torch.cuda.synchronize()
            em.step(0, 0)
            g, step_loss = em.worker_grad(0)
            assert np.isfinite(grad).all() and all(np.abs(grad[lo:hi]).max() > 0 for lo, hi in ((0, 4864), (4864, 107328)))
            for i, a in enumerate(acts):
                assert np.array_equal(em.workspace_tensor(0, 0, i), a.ravel()), (way, "activation", i)
            assert em.workspace_tensor(0, 0, len(acts)) is None
            assert np.array_equal(em.workspace_tensor(0, 2, 0), logits.ravel()) and step_loss == loss, way
            assert np.array_equal(g, grad), (way, np.flatnonzero(g != grad)[:4])
    finally:
        em.close()
