"""The convolutions that do fp32 arithmetic on the bf16 matrix cores, at the ends of fp32's range, against the oracle's direct loops in
float64: operands near and below the smallest normal number (three bf16 terms of the value itself would hold 1e-36 in 14 bits), products
beyond 1e35, single values above the largest bf16 number, infinities and NaN.

Tolerance: as for ordinary operands, 2e-6 of the result (fp32 accumulation of up to 1600 products); a result that is not finite in fp32
arithmetic has to be that infinity or NaN.  Padding is a zero operand: times an infinity it is NaN."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, stream_ptr           # noqa: E402
import torch                                                 # noqa: E402

ABOVE_BF16 = np.float32(3.395e38)       # a finite fp32 value that rounds to an infinite bf16 one


def check(got, want, tol=2e-6):
    got, want = np.asarray(got, dtype=np.float64).ravel(), np.asarray(want, dtype=np.float64).ravel()
    with np.errstate(over="ignore"):
        want32 = want.astype(np.float32)
    fin = np.isfinite(want32)
    same = np.where(fin, np.isfinite(got), np.isnan(got) == np.isnan(want32)) & (~np.isinf(want32) | (got == want32))
    assert same.all(), (int((~same).sum()), np.flatnonzero(~same)[:8], got[~same][:8], want[~same][:8])
    scale = np.max(np.abs(want[fin]), initial=1e-300)           # norms of values near 1e38 in float64: no overflow
    d, w = (got[fin] - want[fin]) / scale, want[fin] / scale
    assert np.linalg.norm(d) <= tol * max(np.linalg.norm(w), 1e-300), np.linalg.norm(d) / np.linalg.norm(w)
    assert np.max(np.abs(d), initial=0.0) <= 10 * tol


def operands(kind, g, a_shape, b_shape):
    """Two operands of a product whose results are ordinary or large numbers; `kind` says what is special about the first or second."""
    a, b = g.standard_normal(a_shape), 0.05 * g.standard_normal(b_shape)
    scale = {"tiny-first": (1e-37, 1e6), "tiny-second": (1e6, 1e-36), "huge": (1e20, 1e15)}.get(kind, (1.0, 1.0))
    a, b = (scale[0] * a).astype(np.float32), (scale[1] * b).astype(np.float32)
    if kind == "special":               # in the middle of an image, far apart where there is room
        h, w = a_shape[1] // 2, a_shape[2] // 2
        a[0, h, w, 1] = np.inf
        a[-1, h, w, 2] = -np.inf
        a[0, -1, -1, 0] = ABOVE_BF16
        if a_shape[0] > 2:
            a[1, h, w, 0] = np.nan
    return a, b


KINDS = ["tiny-first", "tiny-second", "huge", "special"]


def f64(*arrays):
    return [x.astype(np.float64) for x in arrays]


# every tile size of the dispatch, ragged groups of images, bands, several blocks of channels, no padding
@pytest.mark.parametrize("case", [(1, 7, 7, 64, 64, 3, 1), (5, 15, 15, 64, 64, 5, 2), (37, 15, 15, 64, 64, 5, 2), (128, 15, 15, 64, 64, 5, 2),
                                  (200, 7, 7, 64, 64, 3, 1), (2, 6, 9, 128, 64, 3, 1), (2, 5, 5, 64, 128, 5, 2), (3, 12, 17, 64, 64, 3, 0)],
                         ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("kind", KINDS)
def test_wide_convolutions(oracle_nn, case, kind):
    N, H, W, Cin, Cout, k, pad = case
    g = np.random.default_rng(N + H + k)
    OH, OW = H + 2 * pad - k + 1, W + 2 * pad - k + 1
    L, s = B.lib(), stream_ptr()
    n_planes = L.dsspk_conv_split_filter_bytes(Cin, Cout, k) // 4
    pf, pb = empty(n_planes), empty(n_planes)

    def planes(w):
        assert L.dsspk_conv_split_filters(s, dev(w).data_ptr(), pf.data_ptr(), pb.data_ptr(), Cin, Cout, k) == 0
        torch.cuda.synchronize()

    with np.errstate(all="ignore"):
        x, w = operands(kind, g, (N, H, W, Cin), (k, k, Cin, Cout))
        planes(w)
        y = empty((N, OH, OW, Cout))
        X = dev(x)
        assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), None, y.data_ptr(), N, H, W, Cin, Cout, k, pad, 0) == 0
        want = oracle_nn.conv2d_fwd(*f64(x, w), None, 1, pad)
        check(host(y), want)
        assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), None, y.data_ptr(), N, H, W, Cin, Cout, k, pad, 1) == 0
        check(host(y), np.fmax(want, 0))                        # the ReLU of a NaN is 0
        dy, w = operands(kind, g, (N, OH, OW, Cout), (k, k, Cin, Cout))
        planes(w)
        DY, dx = dev(dy), empty((N, H, W, Cin))
        assert L.dsspk_conv_split_bwd_data(s, DY.data_ptr(), pb.data_ptr(), None, dx.data_ptr(), N, H, W, Cin, Cout, k, pad) == 0
        check(host(dx), oracle_nn.conv2d_bwd(np.zeros((N, H, W, Cin)), *f64(w, dy), 1, pad, True)[0])
        x, dy = operands(kind, g, (N, H, W, Cin), (N, OH, OW, Cout))
        E = k * k * Cin * Cout
        dw, scr = empty(E + Cout), empty(L.dsspk_conv_split_wgrad_scratch_floats(N, H, W, Cin, Cout, k, pad))
        X, DY = dev(x), dev(dy)
        assert L.dsspk_conv_split_bwd_weight(s, X.data_ptr(), DY.data_ptr(), dw.data_ptr(), 1, scr.data_ptr(), N, H, W, Cin, Cout, k, pad) == 0
        _, dwo, dbo = oracle_nn.conv2d_bwd(*f64(x, w, dy), 1, pad, True)
        check(host(dw)[:E], dwo)
        check(host(dw)[E:], dbo, 2e-5)


@pytest.mark.parametrize("value", [float("inf"), float(ABOVE_BF16), float("nan")])
def test_wide_convolutions_special_weight(oracle_nn, value):
    """One weight that three terms cannot hold, in the filter planes of both passes."""
    N, H, W, C, k, pad = 3, 15, 15, 64, 5, 2
    g = np.random.default_rng(7)
    x, w = (0.1 * g.standard_normal((N, H, W, C))).astype(np.float32), (0.05 * g.standard_normal((k, k, C, C))).astype(np.float32)
    w[1, 3, 5, 40] = value
    L, s = B.lib(), stream_ptr()
    n_planes = L.dsspk_conv_split_filter_bytes(C, C, k) // 4
    pf, pb, X, Wd, y, dx = empty(n_planes), empty(n_planes), dev(x), dev(w), empty(x.shape), empty(x.shape)
    assert L.dsspk_conv_split_filters(s, Wd.data_ptr(), pf.data_ptr(), pb.data_ptr(), C, C, k) == 0
    assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), None, y.data_ptr(), N, H, W, C, C, k, pad, 0) == 0
    assert L.dsspk_conv_split_bwd_data(s, X.data_ptr(), pb.data_ptr(), None, dx.data_ptr(), N, H, W, C, C, k, pad) == 0
    xp = np.pad(x, ((0, 0), (pad, pad), (pad, pad), (0, 0)))
    with np.errstate(all="ignore"):
        check(host(y), oracle_nn.conv2d_fwd(*f64(xp, w), None, 1, 0))
        # the input gradient is a convolution of the padded dy with the transposed, reversed filter
        wt = np.ascontiguousarray(w[::-1, ::-1].transpose(0, 1, 3, 2))
        check(host(dx), oracle_nn.conv2d_fwd(*f64(xp, wt), None, 1, 0))


@pytest.mark.parametrize("N", [1, 3, 130])
@pytest.mark.parametrize("kind", KINDS)
def test_first_layer(oracle_nn, N, kind):
    g = np.random.default_rng(N)
    L, s = B.lib(), stream_ptr()
    shape, wshape, pshape = (N, 32, 32, 3), (5, 5, 3, 64), (N, 15, 15, 64)

    def forward(x, w, bias):
        a, p, arg = empty((N, 32, 32, 64)), empty(pshape), torch.empty(N * 225 * 64, dtype=torch.uint8, device="cuda")
        X, W, Bd = dev(x), dev(w), dev(bias)
        assert L.dsspk_conv_first_pool_fwd(s, X.data_ptr(), W.data_ptr(), Bd.data_ptr(), a.data_ptr(), p.data_ptr(), arg.data_ptr(), N) == 0
        torch.cuda.synchronize()
        return X, a, p, arg

    with np.errstate(all="ignore"):
        x, w = operands(kind, g, shape, wshape)
        _, a, p, arg = forward(x, w, np.zeros(64, np.float32))
        check(host(a), np.fmax(oracle_nn.conv2d_fwd(*f64(x, w), None, 1, 2), 0))
        p1, arg1 = empty(pshape), torch.empty_like(arg)
        assert L.dsspk_maxpool_fwd(s, a.data_ptr(), p1.data_ptr(), arg1.data_ptr(), N, 32, 32, 64) == 0
        assert np.array_equal(host(p), host(p1)) and np.array_equal(arg.cpu().numpy(), arg1.cpu().numpy())
        # gradients: pooling decisions of an ordinary forward pass, special images or a special pooled gradient
        _, a, p, arg = forward(g.standard_normal(shape), 0.1 * g.standard_normal(wshape), g.standard_normal(64))
        x, dp = operands(kind, g, shape, pshape)
        if kind == "special":                           # ordinary values below 1, so that a product with ABOVE_BF16 stays finite
            dp[np.isfinite(dp)] *= np.float32(0.1)
            x[np.abs(x) < 10] *= np.float32(0.1)
            dp[-1, 7, 7, 5] = np.inf
            dp[0, 3, 11, 9] = ABOVE_BF16
        X, DP, da = dev(x), dev(dp), empty((N, 32, 32, 64))
        assert L.dsspk_maxpool_bwd_relu(s, DP.data_ptr(), arg.data_ptr(), a.data_ptr(), da.data_ptr(), N, 32, 32, 64) == 0
        da64 = host(da).astype(np.float64).reshape(N, 32, 32, 64)
        xz, dz = f64(x, da64)
        # as the matrix cores do it: a zero gradient takes part in the product, and a zero times an infinity is NaN
        xp = np.pad(xz, ((0, 0), (2, 2), (2, 2), (0, 0)))
        dwo = np.stack([np.einsum("nhwc,nhwo->co", xp[:, kh:kh + 32, kw:kw + 32], dz) for kh in range(5) for kw in range(5)])
        dw, scr = empty(4864), empty(L.dsspk_conv_first_scratch_floats(N))
        assert L.dsspk_conv_first_pool_bwd_weight(s, X.data_ptr(), DP.data_ptr(), p.data_ptr(), arg.data_ptr(), dw.data_ptr(), scr.data_ptr(), N) == 0
        out = host(dw)
        check(out[:4800], dwo)
        check(out[4800:], dz.sum(axis=(0, 1, 2)), 2e-5)


SHAPES3 = [(1, 32, 16), (3, 32, 16), (3, 16, 32), (1, 8, 64), (6, 8, 64)]


def dfilter(x, d):
    """Filter gradient of a 3x3, pad 1 convolution as the matrix cores sum it: padding and masked-out elements take part as zeros."""
    H = x.shape[1]
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    return np.stack([np.einsum("nhwc,nhwo->co", xp[:, kh:kh + H, kw:kw + H], d) for kh in range(3) for kw in range(3)])


@pytest.mark.parametrize("N,H,C", SHAPES3)
@pytest.mark.parametrize("kind", KINDS)
def test_residual_convolutions(oracle_nn, N, H, C, kind):
    g = np.random.default_rng(N + C)
    L, s = B.lib(), stream_ptr()
    with np.errstate(all="ignore"):
        x, w = operands(kind, g, (N, H, H, C), (3, 3, C, C))
        X, W, y, dx = dev(x), dev(w), empty(x.shape), empty(x.shape)
        assert L.dsspk_conv_fwd(s, X.data_ptr(), W.data_ptr(), None, y.data_ptr(), N, H, H, C, C, 3, 3, 1, 1, 0, None) == 0
        check(host(y), oracle_nn.conv2d_fwd(*f64(x, w), None, 1, 1))
        assert L.dsspk_conv_bwd_data(s, X.data_ptr(), W.data_ptr(), None, dx.data_ptr(), N, H, H, C, C, 3, 3, 1, 1) == 0
        check(host(dx), oracle_nn.conv2d_bwd(np.zeros(x.shape), *f64(w, x), 1, 1, True)[0])
        if C == 64:
            x, dy = operands(kind, g, (N, H, H, C), (N, H, H, C))
            X, DY, dw = dev(x), dev(dy), empty(9 * C * C)
            scr = empty(L.dsspk_conv_wgrad_scratch_floats(N, H, H, C, C, 3, 3, 1, 1))
            assert L.dsspk_conv_bwd_weight(s, X.data_ptr(), DY.data_ptr(), dw.data_ptr(), scr.data_ptr(), N, H, H, C, C, 3, 3, 1, 1) == 0
            check(host(dw), dfilter(*f64(x, dy)))


@pytest.mark.parametrize("N,H,C", SHAPES3 + [(33, 16, 32)])      # the last: sums merged by a kernel of their own
@pytest.mark.parametrize("with_shortcut", [False, True])
@pytest.mark.parametrize("kind", KINDS)
def test_residual_convolution_behind_batchnorm(oracle_nn, N, H, C, with_shortcut, kind):
    g = np.random.default_rng(N + C)
    L, s = B.lib(), stream_ptr()
    parts = L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1)
    shape = (N, H, H, C)
    first, second = {"tiny-first": (1e-37, 1e6), "tiny-second": (1e6, 1e-36), "huge": (1e20, 1e15)}.get(kind, (1.0, 1.0))
    x, w0 = g.standard_normal(shape), 0.1 * g.standard_normal((3, 3, C, C))
    gamma, beta = first * (1 + 0.2 * g.standard_normal(C)), first * 0.3 * g.standard_normal(C)
    w1, sc = second * 0.05 * g.standard_normal((3, 3, C, C)), first * g.standard_normal(shape)
    if kind == "special":
        gamma[3], sc[0, H // 2, H // 2, 5], sc[0, H // 2, H // 2, 6] = np.inf, np.nan, ABOVE_BF16
    X, W0, W1, Ga, Be, SC = dev(x), dev(w0), dev(w1), dev(gamma), dev(beta), dev(sc)
    c, a, y, stats = empty(shape), empty(shape), empty(shape), empty(2 * C)
    rec, rec1 = empty(L.dsspk_bn_scratch_floats(N * H * H, C)), empty(L.dsspk_bn_scratch_floats(N * H * H, C))
    assert L.dsspk_conv_fwd(s, X.data_ptr(), W0.data_ptr(), None, c.data_ptr(), N, H, H, C, C, 3, 3, 1, 1, 0, rec.data_ptr()) == 0
    assert L.dsspk_conv_fwd_prebn(s, c.data_ptr(), rec.data_ptr(), parts, Ga.data_ptr(), Be.data_ptr(), 1e-5, SC.data_ptr() if with_shortcut else None,
                                  a.data_ptr(), stats.data_ptr(), W1.data_ptr(), y.data_ptr(), rec1.data_ptr(), N, H, C) == 0
    with np.errstate(all="ignore"):
        st = host(stats).astype(np.float64)
        ao = (host(c).astype(np.float64) - st[:C]) * st[C:] * host(Ga) + host(Be) + (host(SC) if with_shortcut else 0)
        check(host(a), np.fmax(ao, 0), 1e-6)
        check(host(y), oracle_nn.conv2d_fwd(host(a).astype(np.float64), host(W1).astype(np.float64), None, 1, 1))


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N,H,C", SHAPES3)
@pytest.mark.parametrize("kind", KINDS)
def test_residual_backward(oracle_nn, N, H, C, kind, fused):
    """Batch-norm backward, input gradient, ReLU mask and (fused) filter gradient.  The mask is that of the activation, subnormal ones
    included."""
    g = np.random.default_rng(N + C)
    L, s = B.lib(), stream_ptr()
    if fused and L.dsspk_conv_bwd_fused_chunks(N, H, C) == 0:
        pytest.skip("no fused form for this shape")
    shape, M = (N, H, H, C), N * H * H
    dz, w = operands(kind, g, shape, (3, 3, C, C))
    scale = {"tiny-first": (1e-37, 1e6), "tiny-second": (1e6, 1e-36), "huge": (1e20, 1e15)}.get(kind, (1.0, 1.0))
    x_in = np.maximum(scale[1] * g.standard_normal(shape), 0)
    x_in[g.random(shape) < 0.1] = 1e-44
    xc, xp, add = g.standard_normal(shape), g.standard_normal(shape), scale[0] * scale[1] * g.standard_normal(shape)
    stats = np.concatenate([0.1 * g.standard_normal(C), 1 + 0.1 * g.random(C)])
    gamma, totals = 1 + 0.1 * g.standard_normal(C), scale[0] * 0.1 * M * g.standard_normal(2 * C)
    DZ, W, XI, XC, XP, ADD, ST, GA, TOT = (dev(np.asarray(t, dtype=np.float32)) for t in (dz, w, x_in, xc, xp, add, stats, gamma, totals))
    out, dx, rec = empty(shape), empty(shape), empty(2 * C * L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1))
    front = (s, DZ.data_ptr(), XC.data_ptr(), ST.data_ptr(), GA.data_ptr(), TOT.data_ptr())
    if fused:
        chunks = L.dsspk_conv_bwd_fused_chunks(N, H, C)
        partial = empty((chunks, 9 * C * C))
        rc = L.dsspk_conv_bwd_data_bn_wgrad(*front, W.data_ptr(), ADD.data_ptr(), out.data_ptr(), XP.data_ptr(), ST.data_ptr(), rec.data_ptr(),
                                            XI.data_ptr(), partial.data_ptr(), None, None, 0, 0, N, H, C)
    else:
        rc = L.dsspk_conv_bwd_data_bn(*front, dx.data_ptr(), W.data_ptr(), ADD.data_ptr(), out.data_ptr(), XI.data_ptr(), XP.data_ptr(), ST.data_ptr(),
                                      rec.data_ptr(), None, None, 0, 0, N, H, C)
    assert rc == 0
    with np.errstate(all="ignore"):
        z, xi, cc, st, ga, tot = f64(*(host(t) for t in (DZ, XI, XC, ST, GA, TOT)))
        d = ga * st[C:] * (z - tot[:C] / M - (cc - st[:C]) * st[C:] * tot[C:] / M)
        d = d.astype(np.float32).astype(np.float64)         # overflows where the kernel's does
        if not fused:
            check(host(dx), d)
            d = host(dx).astype(np.float64)
        want = oracle_nn.conv2d_bwd(np.zeros(shape), w.astype(np.float64), d, 1, 1, True)[0] + host(ADD)
        check(host(out), np.where(xi > 0, want, 0))
        if fused:
            check(host(partial).astype(np.float64).sum(axis=0), dfilter(xi, d))
