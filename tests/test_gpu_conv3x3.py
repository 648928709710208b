"""The 3x3 / stride 1 convolutions of the residual networks (fp32 arithmetic on the bf16 matrix cores, leading and small
products summed apart) against the oracle's direct loops in float64.

Tolerance: the sum of the leading products is rounded once per instruction, 9 C / 32 (at least 9) times, each time by up to
6e-8 of the running sum, which is below the final one for most of the way; errors of random sign add up to
sqrt(9 .. 18) * 6e-8 * 0.6 = 1.1e-7 .. 1.6e-7 of the result.  Bound 2e-7 (measured at most 1.2e-7; the fp32 matrix-core
form of the same convolution shows up to 2.1e-7)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr     # noqa: E402


@pytest.mark.parametrize("N,H,C", [(1, 32, 16), (7, 32, 16), (1, 16, 32), (5, 16, 32), (1, 8, 64), (9, 8, 64)])
@pytest.mark.parametrize("offset", [0.0, 8.0])
def test_error_of_forward_and_input_gradient(oracle_nn, N, H, C, offset):
    g = np.random.default_rng(100 * N + C)
    x = (offset + g.standard_normal((N, H, H, C))).astype(np.float32)
    w = (np.sqrt(2.0 / (9 * C)) * g.standard_normal((3, 3, C, C))).astype(np.float32)
    dy = (1e-3 * g.standard_normal((N, H, H, C))).astype(np.float32)
    X, W, DY, y, dx = dev(x), dev(w), dev(dy), empty((N, H, H, C)), empty((N, H, H, C))
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_conv_fwd(s, X.data_ptr(), W.data_ptr(), None, y.data_ptr(), N, H, H, C, C, 3, 3, 1, 1, 0, None) == 0
    assert L.dsspk_conv_bwd_data(s, DY.data_ptr(), W.data_ptr(), None, dx.data_ptr(), N, H, H, C, C, 3, 3, 1, 1) == 0
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    yo = oracle_nn.conv2d_fwd(x64, w64, None, 1, 1)
    dxo, _, _ = oracle_nn.conv2d_bwd(x64, w64, dy64, 1, 1, True)
    assert rel_l2(host(y), yo) < 2e-7 and max_abs(host(y), yo) < 2e-6
    assert rel_l2(host(dx), dxo) < 2e-7 and max_abs(host(dx), dxo) < 2e-6


# one image; the largest batch whose records every workgroup adds up itself (2048 / C of them), and one more
@pytest.mark.parametrize("N,H,C", [(1, 32, 16), (5, 32, 16), (32, 32, 16), (33, 32, 16), (1, 16, 32), (32, 16, 32), (33, 16, 32), (1, 8, 64),
                                   (32, 8, 64), (33, 8, 64)])
def test_batchnorm_sums_taken_from_records(N, H, C):
    """The backward kernels with their batch norm's sums added up inside against the same kernels behind dsspk_bn_bwd_totals.  The sums
    are over the same records in another order: 1e-6 of the scale of their terms; outputs depend on them linearly."""
    import torch
    g = np.random.default_rng(N + C)
    L, s = B.lib(), stream_ptr()
    parts = L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1)
    assert L.dsspk_conv_records_inline(parts, C) == (1 if N <= 32 else 0)
    f = lambda *sh: dev(g.standard_normal(sh).astype(np.float32))
    dz, xc, xp, xin, add, w = f(N, H, H, C), f(N, H, H, C), f(N, H, H, C), torch.relu(f(N, H, H, C)), f(N, H, H, C), f(3, 3, C, C)
    stats, statsp = torch.cat([f(C), f(C).abs() + 0.5]), torch.cat([f(C), f(C).abs() + 0.5])
    gamma, rin = f(C), f(parts, C, 2)
    tot, dgam, dbet = empty(2 * C), empty(C), empty(C)
    assert L.dsspk_bn_bwd_totals(s, rin.data_ptr(), parts, C, tot.data_ptr(), dgam.data_ptr(), dbet.data_ptr()) == 0
    fused = L.dsspk_conv_bwd_fused_chunks(N, H, C)
    res = []
    for totals in (tot, None):
        out, dx, rout, part = empty((N, H, H, C)), empty((N, H, H, C)), empty((parts, C, 2)), empty(max(1, fused) * 9 * C * C)
        dg, db = empty(C), empty(C)
        common = (s, dz.data_ptr(), xc.data_ptr(), stats.data_ptr(), gamma.data_ptr(), totals.data_ptr() if totals is not None else None,
                  rin.data_ptr(), parts, dg.data_ptr(), db.data_ptr())
        if fused:
            rc = L.dsspk_conv_bwd_data_bn_wgrad_records(*common, w.data_ptr(), add.data_ptr(), out.data_ptr(), xp.data_ptr(), statsp.data_ptr(),
                                                        rout.data_ptr(), xin.data_ptr(), part.data_ptr(), None, None, 0, 0, N, H, C)
        else:
            rc = L.dsspk_conv_bwd_data_bn_records(*common, dx.data_ptr(), w.data_ptr(), add.data_ptr(), out.data_ptr(), xin.data_ptr(),
                                                  xp.data_ptr(), statsp.data_ptr(), rout.data_ptr(), None, None, 0, 0, N, H, C)
        if totals is None and N > 32:
            assert rc == -1
            return
        assert rc == 0
        if totals is None:
            scale = np.sqrt(parts)
            assert np.max(np.abs(host(dg) - host(dgam))) < 1e-6 * scale and np.max(np.abs(host(db) - host(dbet))) < 1e-6 * scale
        res.append([host(t) for t in ((out, rout, part) if fused else (out, rout, dx))])
    for a, b in zip(*res):
        assert rel_l2(b, a) < 2e-6 and max_abs(b, a) < 2e-5


# the four-wavefront kernels at any batch; the others where a residual network's step takes them
FUSED = [("middle", N, H, C) for N, H, C in ((1, 32, 16), (5, 32, 16), (37, 32, 16), (128, 32, 16), (1, 16, 32), (37, 16, 32), (128, 16, 32))]
FUSED += [(family, N, H, C) for family, N in (("small", 1), ("small", 5), ("small", 32), ("large", 97), ("large", 128)) for H, C in ((32, 16), (16, 32))]


@pytest.mark.parametrize("family,N,H,C", FUSED)
@pytest.mark.parametrize("kind", ["relu", "offset"])
def test_fused_filter_gradient_no_less_exact_than_on_the_fp32_cores(oracle_nn, family, N, H, C, kind):
    """The filter gradient that the fused backward kernels leave (batch norm the identity, so that dx is dz) against the stand-alone
    kernel's, which works on the fp32 matrix cores, both against float64."""
    g = np.random.default_rng(N + C)
    x = g.standard_normal((N, H, H, C))
    x = (np.maximum(x, 0) if kind == "relu" else x + 8).astype(np.float32)
    dz, w = (1e-3 * g.standard_normal((N, H, H, C))).astype(np.float32), (0.1 * g.standard_normal((3, 3, C, C))).astype(np.float32)
    L, s = B.lib(), stream_ptr()
    X, DZ, W, XC = dev(x), dev(dz), dev(w), dev(g.standard_normal((N, H, H, C)).astype(np.float32))
    identity, ones, zeros = dev(np.repeat([0.0, 1.0], C).astype(np.float32)), dev(np.ones(C, np.float32)), dev(np.zeros(2 * C, np.float32))
    if family == "middle":
        chunks, records = L.dsspk_conv_bwd_fused_chunks(N, H, C), L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1)
    else:
        chunks = records = getattr(L, "dsspk_conv3x3_%s_parts" % family)(N, H, C)
    out, rec, partial = empty((N, H, H, C)), empty(2 * C * records), empty(chunks * 9 * C * C)
    if family == "middle":
        assert L.dsspk_conv_bwd_data_bn_wgrad(s, DZ.data_ptr(), XC.data_ptr(), identity.data_ptr(), ones.data_ptr(), zeros.data_ptr(), W.data_ptr(), None,
                                              out.data_ptr(), XC.data_ptr(), identity.data_ptr(), rec.data_ptr(), X.data_ptr(), partial.data_ptr(),
                                              None, None, 0, 0, N, H, C) == 0
    else:                               # the sums of the batch norm's backward pass from one record, zero
        dg, db = empty(C), empty(C)
        assert getattr(L, "dsspk_conv3x3_%s_bwd" % family)(s, DZ.data_ptr(), XC.data_ptr(), identity.data_ptr(), ones.data_ptr(), zeros.data_ptr(), 1,
                                                           dg.data_ptr(), db.data_ptr(), None, partial.data_ptr(), W.data_ptr(), None, out.data_ptr(),
                                                           X.data_ptr(), XC.data_ptr(), identity.data_ptr(), rec.data_ptr(), None, None, 0, 0, N, H, C) == 0
    dw, dw32, scr = empty(9 * C * C), empty(9 * C * C), empty(L.dsspk_conv_wgrad_scratch_floats(N, H, H, C, C, 3, 3, 1, 1))
    assert L.dsspk_wgrad_reduce(s, partial.data_ptr(), dw.data_ptr(), 9 * C * C, chunks) == 0
    assert L.dsspk_conv_bwd_weight(s, X.data_ptr(), DZ.data_ptr(), dw32.data_ptr(), scr.data_ptr(), N, H, H, C, C, 3, 3, 1, 1) == 0
    _, want, _ = oracle_nn.conv2d_bwd(x.astype(np.float64), w.astype(np.float64), dz.astype(np.float64), 1, 1, True, need_dx=False)
    fused, fp32 = rel_l2(host(dw), want), rel_l2(host(dw32), want)
    assert fused <= fp32, (fused, fp32)


@pytest.mark.parametrize("N", [1, 9, 37, 128])
@pytest.mark.parametrize("kind", ["relu", "offset"])
def test_last_stage_filter_gradient_no_less_exact_than_on_the_fp32_cores(oracle_nn, N, kind):
    """64 channels, 8x8 images: against the same products summed by the fp32 matrix product over the unrolled input, which splits short
    sums over wavefronts, or 1.1e-7, the least that minimal filtering on the fp32 cores shows on such operands (1.1e-7 to 2.5e-7)."""
    H, C = 8, 64
    g = np.random.default_rng(N)
    x = g.standard_normal((N, H, H, C))
    x = (np.maximum(x, 0) if kind == "relu" else x + 8).astype(np.float32)
    dy = (1e-3 * g.standard_normal((N, H, H, C))).astype(np.float32)
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    cols = np.stack([xp[:, a:a + H, b:b + H] for a in range(3) for b in range(3)], axis=3).reshape(N * H * H, 9 * C)
    L, s = B.lib(), stream_ptr()
    X, DY, COLS = dev(x), dev(dy), dev(cols)
    dw, dw32, scr = empty(9 * C * C), empty((9 * C, C)), empty(L.dsspk_conv_wgrad_scratch_floats(N, H, H, C, C, 3, 3, 1, 1))
    assert L.dsspk_conv_bwd_weight(s, X.data_ptr(), DY.data_ptr(), dw.data_ptr(), scr.data_ptr(), N, H, H, C, C, 3, 3, 1, 1) == 0
    assert L.dsspk_gemm(s, COLS.data_ptr(), 1, 9 * C, DY.data_ptr(), C, 1, dw32.data_ptr(), C, 9 * C, C, N * H * H, None, 0) == 0
    want = cols.astype(np.float64).T @ dy.astype(np.float64).reshape(-1, C)
    split, fp32 = rel_l2(host(dw), want), rel_l2(host(dw32), want)
    assert split <= max(fp32, 1.1e-7), (split, fp32)
