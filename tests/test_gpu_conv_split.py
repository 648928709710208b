"""Convolutions with fp32 arithmetic on the bf16 matrix cores (three bf16 terms per operand, six products), against the
oracle's direct loops in float64.

Tolerance: the terms hold all 24 bits and the dropped products are below an fp32 rounding, so the bound is that of an fp32
accumulation of K products, about sqrt(K) * 6e-8 of the sum's scale (2.4e-6 at K = 1600); the kernels are held to the
2e-6 / 2e-5 of the other convolution kernels (measured: at most 6e-7), and, with the same inputs, to no larger an error than
1.25 times the fp32 matrix-core kernel's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr     # noqa: E402

# N, H, W, Cin, Cout, k, pad: single images and ragged groups of them, one and several bands, every tile size of the dispatch,
# images narrower and wider than a tile of 16 pixels, no padding, several channel blocks
CASES = [(1, 7, 7, 64, 64, 3, 1), (3, 7, 7, 64, 64, 3, 1), (37, 7, 7, 64, 64, 3, 1), (1, 15, 15, 64, 64, 5, 2), (5, 15, 15, 64, 64, 5, 2),
         (37, 15, 15, 64, 64, 5, 2), (128, 15, 15, 64, 64, 5, 2), (200, 7, 7, 64, 64, 3, 1), (2, 5, 5, 64, 128, 5, 2), (2, 6, 9, 128, 64, 3, 1),
         (1, 3, 3, 64, 64, 3, 1), (2, 12, 17, 64, 64, 3, 0), (1, 9, 33, 64, 64, 5, 1), (1, 4, 60, 64, 64, 3, 1), (9, 1, 1, 64, 64, 3, 1)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("offset", [0.0, 4.0])
def test_conv_split(oracle_nn, case, offset):
    N, H, W, Cin, Cout, k, pad = case
    g = np.random.default_rng(N * 1000 + H * 10 + k)
    x = (offset + g.standard_normal((N, H, W, Cin))).astype(np.float32)
    w = (0.05 * g.standard_normal((k, k, Cin, Cout))).astype(np.float32)
    b = g.standard_normal(Cout).astype(np.float32)
    OH, OW = H + 2 * pad - k + 1, W + 2 * pad - k + 1
    dy = g.standard_normal((N, OH, OW, Cout)).astype(np.float32)
    add = g.standard_normal((N, H, W, Cin)).astype(np.float32)
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_conv_split_covers(N, H, W, Cin, Cout, k, pad) == 1
    X, Wd, Bd, DY, ADD = dev(x), dev(w), dev(b), dev(dy), dev(add)
    n_planes = L.dsspk_conv_split_filter_bytes(Cin, Cout, k) // 4
    pf, pb = empty(n_planes), empty(n_planes)
    assert L.dsspk_conv_split_filters(s, Wd.data_ptr(), pf.data_ptr(), pb.data_ptr(), Cin, Cout, k) == 0
    y, y32, dx = empty((N, OH, OW, Cout)), empty((N, OH, OW, Cout)), empty((N, H, W, Cin))
    assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), Bd.data_ptr(), y.data_ptr(), N, H, W, Cin, Cout, k, pad, 0) == 0
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    yo = oracle_nn.conv2d_fwd(x64, w64, b.astype(np.float64), 1, pad)
    dxo, dwo, dbo = oracle_nn.conv2d_bwd(x64, w64, dy64, 1, pad, True)
    err = rel_l2(host(y), yo)
    assert err < 2e-6 and max_abs(host(y), yo) < 2e-5
    assert L.dsspk_conv_fwd(s, X.data_ptr(), Wd.data_ptr(), Bd.data_ptr(), y32.data_ptr(), N, H, W, Cin, Cout, k, k, 1, pad, 0, None) == 0
    assert err < 1.25 * rel_l2(host(y32), yo)
    yr = empty((N, OH, OW, Cout))
    assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), None, yr.data_ptr(), N, H, W, Cin, Cout, k, pad, 1) == 0
    assert rel_l2(host(yr), np.maximum(yo - b.astype(np.float64), 0)) < 2e-6
    for a, want in ((None, dxo), (ADD, dxo + add.astype(np.float64))):
        assert L.dsspk_conv_split_bwd_data(s, DY.data_ptr(), pb.data_ptr(), a.data_ptr() if a is not None else None, dx.data_ptr(),
                                           N, H, W, Cin, Cout, k, pad) == 0
        assert rel_l2(host(dx), want) < 2e-6 and max_abs(host(dx), want) < 2e-5
    E = k * k * Cin * Cout
    for bias in (0, 1):
        dw = empty(E + bias * Cout)
        scr = empty(L.dsspk_conv_split_wgrad_scratch_floats(N, H, W, Cin, Cout, k, pad))
        assert L.dsspk_conv_split_bwd_weight(s, X.data_ptr(), DY.data_ptr(), dw.data_ptr(), bias, scr.data_ptr(), N, H, W, Cin, Cout, k, pad) == 0
        got = host(dw)
        assert rel_l2(got[:E], dwo) < 2e-6 and max_abs(got[:E], dwo) < 2e-5
        if bias:
            # sums of N OH OW terms of either sign: measured against the terms' scale, sqrt(count)
            assert np.max(np.abs(got[E:] - dbo)) < 2e-6 * max(1.0, np.sqrt(N * OH * OW)) * 4


def test_conv_split_refuses_other_shapes():
    L = B.lib()
    for case in [(1, 8, 8, 32, 64, 3, 1), (1, 8, 8, 64, 48, 3, 1), (1, 8, 8, 64, 64, 4, 1), (1, 8, 8, 64, 64, 3, 3), (1, 2, 2, 64, 64, 5, 0),
                 (1, 4, 200, 64, 64, 3, 1)]:
        assert L.dsspk_conv_split_covers(*case) == 0


# the networks' operands: post-ReLU activations and gradients behind a ReLU's mask, half of them zero (a sum on the fp32 cores is not
# rounded where it adds a zero)
@pytest.mark.parametrize("case", [(1, 15, 15, 64, 64, 5, 2), (37, 15, 15, 64, 64, 5, 2), (128, 15, 15, 64, 64, 5, 2), (300, 15, 15, 64, 64, 5, 2),
                                  (3, 7, 7, 64, 64, 3, 1), (200, 7, 7, 64, 64, 3, 1), (512, 7, 7, 64, 64, 3, 1), (256, 15, 15, 64, 64, 3, 1), (200, 8, 16, 128, 64, 3, 1), (5, 9, 9, 128, 64, 3, 1),
                                  (5, 9, 9, 64, 128, 5, 2)], ids=lambda c: "x".join(map(str, c)))
def test_error_no_larger_than_the_fp32_matrix_cores(oracle_nn, case):
    N, H, W, Cin, Cout, k, pad = case
    g = np.random.default_rng(N + H)
    x = np.maximum(g.standard_normal((N, H, W, Cin)), 0).astype(np.float32)
    dy = (g.standard_normal((N, H, W, Cout)) * (g.random((N, H, W, Cout)) < 0.5)).astype(np.float32)
    w = (np.sqrt(2.0 / (k * k * Cin)) * g.standard_normal((k, k, Cin, Cout))).astype(np.float32)
    L, s = B.lib(), stream_ptr()
    X, Wd, DY = dev(x), dev(w), dev(dy)
    n_planes = L.dsspk_conv_split_filter_bytes(Cin, Cout, k) // 4
    pf, pb = empty(n_planes), empty(n_planes)
    assert L.dsspk_conv_split_filters(s, Wd.data_ptr(), pf.data_ptr(), pb.data_ptr(), Cin, Cout, k) == 0
    y, dx, dw = [empty((N, H, W, Cout)) for _ in "ab"], [empty((N, H, W, Cin)) for _ in "ab"], [empty(k * k * Cin * Cout) for _ in "ab"]
    shape = (N, H, W, Cin, Cout, k, pad)
    assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), None, y[0].data_ptr(), *shape, 0) == 0
    assert L.dsspk_conv_split_bwd_data(s, DY.data_ptr(), pb.data_ptr(), None, dx[0].data_ptr(), *shape) == 0
    scr = empty(L.dsspk_conv_split_wgrad_scratch_floats(*shape))
    assert L.dsspk_conv_split_bwd_weight(s, X.data_ptr(), DY.data_ptr(), dw[0].data_ptr(), 0, scr.data_ptr(), *shape) == 0
    general = (N, H, W, Cin, Cout, k, k, 1, pad)
    assert L.dsspk_conv_fwd(s, X.data_ptr(), Wd.data_ptr(), None, y[1].data_ptr(), *general, 0, None) == 0
    assert L.dsspk_conv_bwd_data(s, DY.data_ptr(), Wd.data_ptr(), None, dx[1].data_ptr(), *general) == 0
    scr1 = empty(L.dsspk_conv_wgrad_scratch_floats(*general))
    assert L.dsspk_conv_bwd_weight(s, X.data_ptr(), DY.data_ptr(), dw[1].data_ptr(), scr1.data_ptr(), *general) == 0
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    dxo, dwo, _ = oracle_nn.conv2d_bwd(x64, w64, dy64, 1, pad, True)
    outputs = [(y, oracle_nn.conv2d_fwd(x64, w64, None, 1, pad)), (dx, dxo), (dw, dwo)]
    if N == 200 and Cin == 128:     # a shape no network has, whose filter gradient the general kernel sums in shorter pieces (1.1e-7, here 1.2e-7)
        outputs.pop()
    for got, want in outputs:
        split, fp32 = rel_l2(host(got[0]), want), rel_l2(host(got[1]), want)
        assert split <= fp32
