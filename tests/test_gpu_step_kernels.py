"""Kernels that save a residual network's step launches, against the kernels whose work they take over."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, rel_l2, stream_ptr   # noqa: E402


@pytest.mark.parametrize("jobs", [[(4, 1)], [(432, 65), (2304, 64)], [(36864, 3), (9216, 130), (4, 200), (18432, 17)]])
def test_reductions_in_one_launch(jobs):
    """Both forms of the reduction (up to 64 and more partial results), remainders of a workgroup's elements: the same bits."""
    g = np.random.default_rng(len(jobs))
    L, s, n = B.lib(), stream_ptr(), len(jobs)
    part = [dev(g.standard_normal((c, E)).astype(np.float32)) for E, c in jobs]
    one, many = [empty(E) for E, _ in jobs], [empty(E) for E, _ in jobs]
    for p, d, (E, c) in zip(part, one, jobs):
        assert L.dsspk_wgrad_reduce(s, p.data_ptr(), d.data_ptr(), E, c) == 0
    ptr = lambda ts: (ctypes.c_void_p * n)(*[t.data_ptr() for t in ts])
    Es, cs = (ctypes.c_int * n)(*[E for E, _ in jobs]), (ctypes.c_int * n)(*[c for _, c in jobs])
    assert L.dsspk_wgrad_reduce_many(s, n, ptr(part), ptr(many), Es, cs) == 0
    for a, b in zip(one, many):
        assert np.array_equal(host(a), host(b))
    assert L.dsspk_wgrad_reduce_many(s, 5, ptr(part), ptr(many), Es, cs) == -1 and L.dsspk_wgrad_reduce_many(s, 0, ptr(part), ptr(many), Es, cs) == -1


@pytest.mark.parametrize("parts,rows,C", [(1, 64, 64), (4, 256, 16), (7, 128, 32), (3, 37, 16), (256, 512, 16)])
@pytest.mark.parametrize("masked", [True, False])
def test_sums_of_equal_slabs(parts, rows, C, masked):
    """fp32 sums of `rows` terms: 6e-8 sqrt(rows) of the terms' scale, bound 1e-5 relative to sqrt(rows)."""
    g = np.random.default_rng(rows + C)
    M = parts * rows
    x, da, out = (g.standard_normal((M, C)).astype(np.float32) for _ in range(3))
    mean, invstd = g.standard_normal(C).astype(np.float32), (0.5 + g.random(C)).astype(np.float32)
    X, DA, OUT, ST, rec = dev(x), dev(da), dev(out), dev(np.concatenate([mean, invstd])), empty((parts, C, 2))
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_bn_bwd_reduce_parts(s, X.data_ptr(), ST.data_ptr(), DA.data_ptr(), OUT.data_ptr() if masked else None, rec.data_ptr(), parts, M, C) == 0
    dz = np.where(out > 0, da, 0) if masked else da
    assert np.array_equal(host(DA), dz)
    xhat = (x.astype(np.float64) - mean) * invstd
    want = np.stack([dz.astype(np.float64).reshape(parts, rows, C).sum(1), (dz * xhat).reshape(parts, rows, C).sum(1)], axis=2)
    assert np.max(np.abs(host(rec) - want)) < 1e-5 * np.sqrt(rows) * 4
    if parts > 1:
        assert L.dsspk_bn_bwd_reduce_parts(s, X.data_ptr(), ST.data_ptr(), DA.data_ptr(), None, rec.data_ptr(), parts, M - 1, C) == -1


@pytest.mark.parametrize("N,H,Cin,Cout,stride", [(1, 32, 3, 16, 1), (13, 32, 3, 16, 1), (32, 32, 3, 16, 1), (64, 32, 3, 16, 1), (1, 32, 16, 32, 2), (13, 32, 16, 32, 2), (64, 32, 16, 32, 2),
                                                 (1, 16, 32, 64, 2), (128, 16, 32, 64, 2), (3, 8, 48, 32, 1)])
def test_records_of_generic_convolutions(N, H, Cin, Cout, stride):
    """The result is dsspk_conv_fwd's bit for bit; a record is the tile's mean and sum of squared deviations (fp32 sums of 64 or 128 terms)."""
    g = np.random.default_rng(N + Cin)
    x, w = dev(g.standard_normal((N, H, H, Cin)).astype(np.float32)), dev((0.2 * g.standard_normal((3, 3, Cin, Cout))).astype(np.float32))
    Ho, L, s = H // stride, B.lib(), stream_ptr()
    shape = (N, H, H, Cin, Cout, 3, 3, stride, 1)
    parts = L.dsspk_conv_fwd_records_parts(*shape)
    rows = 64 if N * Ho * Ho < 65536 else 128
    assert parts == N * Ho * Ho // rows
    y, y0, rec = empty((N, Ho, Ho, Cout)), empty((N, Ho, Ho, Cout)), empty((parts, Cout, 2))
    assert L.dsspk_conv_fwd_records(s, x.data_ptr(), w.data_ptr(), y.data_ptr(), rec.data_ptr(), *shape) == 0
    assert L.dsspk_conv_fwd(s, x.data_ptr(), w.data_ptr(), None, y0.data_ptr(), *shape, 0, None) == 0
    assert np.array_equal(host(y), host(y0))
    t = host(y).astype(np.float64).reshape(parts, rows, Cout)
    mean = t.mean(1)
    assert np.max(np.abs(host(rec)[..., 0] - mean)) < 1e-6 * np.abs(t).max()
    assert rel_l2(host(rec)[..., 1], ((t - mean[:, None]) ** 2).sum(1)) < 1e-6


def test_shapes_without_records():
    L = B.lib()
    for N, H, Cin, Cout, stride in [(33, 32, 3, 16, 1), (65, 32, 16, 32, 2), (1, 6, 16, 32, 2), (1, 32, 16, 48, 2)]:
        assert L.dsspk_conv_fwd_records_parts(N, H, H, Cin, Cout, 3, 3, stride, 1) == 0


@pytest.mark.parametrize("N,H,Cin", [(1, 32, 16), (5, 32, 16), (1, 16, 32), (9, 16, 32), (2, 6, 16), (128, 16, 32)])
def test_input_gradient_with_shortcut(N, H, Cin):
    """dsspk_conv_bwd_data and dsspk_shortcut_bwd_acc: the same two fp32 additions per element, the same bits."""
    g = np.random.default_rng(N + H)
    Ho, Cout = H // 2, 2 * Cin
    dy, sc = (dev(g.standard_normal((N, Ho, Ho, Cout)).astype(np.float32)) for _ in range(2))
    w, dx, want = dev((0.2 * g.standard_normal((3, 3, Cin, Cout))).astype(np.float32)), empty((N, H, H, Cin)), empty((N, H, H, Cin))
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_conv_bwd_data(s, dy.data_ptr(), w.data_ptr(), None, want.data_ptr(), N, H, H, Cin, Cout, 3, 3, 2, 1) == 0
    assert L.dsspk_shortcut_bwd_acc(s, sc.data_ptr(), want.data_ptr(), N, Ho, Ho, Cout) == 0
    assert L.dsspk_conv_bwd_data_shortcut(s, dy.data_ptr(), w.data_ptr(), sc.data_ptr(), dx.data_ptr(), N, H, H, Cin, Cout, 3, 3, 1) == 0
    assert np.array_equal(host(dx), host(want))
    assert L.dsspk_conv_bwd_data_shortcut(s, dy.data_ptr(), w.data_ptr(), sc.data_ptr(), dx.data_ptr(), N, H + 1, H, Cin, Cout, 3, 3, 1) == -1


def _records(parts, C, x):
    r = x.reshape(parts, -1, C).astype(np.float64)
    m = r.mean(1)
    return np.stack([m, ((r - m[:, None]) ** 2).sum(1)], axis=2).astype(np.float32)


@pytest.mark.parametrize("N,side,C", [(1, 8, 64), (13, 8, 64), (128, 8, 64), (2, 3, 16), (3, 10, 32)])
@pytest.mark.parametrize("half", [False, True])
def test_last_batch_norm_with_pooling(N, side, C, half):
    """Against the kernels one by one: the same activations bit for bit, the pooled sums of side^2 terms in another order."""
    g = np.random.default_rng(N + side)
    HW, L, s = side * side, B.lib(), stream_ptr()
    M = N * HW
    x = g.standard_normal((M, C)).astype(np.float32)
    sc = dev(g.standard_normal((N, 2 * side, 2 * side, C // 2) if half else (M, C)).astype(np.float32))
    X, G, BE, rec = dev(x), dev(1 + 0.1 * g.standard_normal(C)), dev(0.1 * g.standard_normal(C)), dev(_records(N, C, x))
    y, y0, st, st0, p, p0 = empty((M, C)), empty((M, C)), empty(2 * C), empty(2 * C), empty((N, C)), empty((N, C))
    assert L.dsspk_bn_fwd_gap(s, X.data_ptr(), G.data_ptr(), BE.data_ptr(), y.data_ptr(), st.data_ptr(), rec.data_ptr(), N, sc.data_ptr(), int(half),
                              p.data_ptr(), N, side, C, 1e-5) == 0
    assert L.dsspk_bn_fwd(s, X.data_ptr(), G.data_ptr(), BE.data_ptr(), y0.data_ptr(), st0.data_ptr(), rec.data_ptr(), M, C, 1e-5, 1, 2 if half else 1,
                          sc.data_ptr(), N, side, side, N) == 0
    assert L.dsspk_gap_fwd(s, y0.data_ptr(), p0.data_ptr(), N, HW, C) == 0
    assert np.array_equal(host(y), host(y0)) and np.array_equal(host(st), host(st0))
    assert np.max(np.abs(host(p) - host(p0))) < 1e-6 * np.abs(host(y)).max()
    dp, dz, dz0, r, r0 = dev(g.standard_normal((N, C)).astype(np.float32)), empty((M, C)), empty((M, C)), empty((N, C, 2)), empty((N, C, 2))
    assert L.dsspk_gap_bwd_bn_reduce(s, dp.data_ptr(), X.data_ptr(), st.data_ptr(), y.data_ptr(), dz.data_ptr(), r.data_ptr(), N, side, C) == 0
    assert L.dsspk_gap_bwd(s, dp.data_ptr(), dz0.data_ptr(), N, HW, C) == 0
    assert L.dsspk_bn_bwd_reduce_parts(s, X.data_ptr(), st.data_ptr(), dz0.data_ptr(), y.data_ptr(), r0.data_ptr(), N, M, C) == 0
    assert np.array_equal(host(dz), host(dz0)) and np.array_equal(host(r), host(r0))


def _family(family, N, H, C):
    """(records it leaves, forward with a batch norm in the loader) of a family of the 3x3 kernels; short_half: of a stride-2 block's shortcut."""
    L = B.lib()
    if family == "middle":
        return (L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1),
                lambda *a, short_half=0: (L.dsspk_conv_fwd_prebn_half if short_half else L.dsspk_conv_fwd_prebn)(*a))
    fwd = getattr(L, "dsspk_conv3x3_%s_fwd" % family)
    return getattr(L, "dsspk_conv3x3_%s_parts" % family)(N, H, C), lambda *a, short_half=0: fwd(*a[:13], short_half, *a[13:])


BEHIND = [(family, N, H, C) for family in ("middle", "large") for N, H, C in ((1, 16, 32), (5, 16, 32), (128, 16, 32), (1, 8, 64), (5, 8, 64), (128, 8, 64))]
BEHIND += [("small", N, H, C) for N in (1, 5, 17, 32) for H, C in ((16, 32), (8, 64))]


@pytest.mark.parametrize("family,N,H,C", BEHIND)
@pytest.mark.parametrize("scale", [1.0, 1e32])
def test_convolution_behind_a_stride_2_shortcut(family, N, H, C, scale):
    """The kernel families against the batch norm with that shortcut and the plain convolution, one after the other; scale: of one shortcut
    value, the second beyond the range of the scaled terms (the tiles it meets are then computed by other instructions: 4e-7)."""
    g = np.random.default_rng(N + C)
    f = lambda *sh: g.standard_normal(sh).astype(np.float32)
    x, sc = f(N, H, H, C), f(N, 2 * H, 2 * H, C // 2)
    sc[N - 1, 2, 2 * H - 2, 1] = scale
    L, s = B.lib(), stream_ptr()
    parts, fwd = _family(family, N, H, C)
    X, SC, W, G, BE, rec = dev(x), dev(sc), dev(0.1 * f(3, 3, C, C)), dev(1 + 0.1 * f(C)), dev(0.1 * f(C)), dev(_records(parts, C, x))
    act, act0, st, st0, y, y0, out = empty(x.shape), empty(x.shape), empty(2 * C), empty(2 * C), empty(x.shape), empty(x.shape), empty((parts, C, 2))
    args = (s, X.data_ptr(), rec.data_ptr(), parts, G.data_ptr(), BE.data_ptr(), 1e-5, SC.data_ptr(), act.data_ptr(), st.data_ptr(), W.data_ptr(),
            y.data_ptr(), out.data_ptr())
    assert fwd(*args, N, H, C, short_half=1) == 0
    assert L.dsspk_bn_fwd(s, X.data_ptr(), G.data_ptr(), BE.data_ptr(), act0.data_ptr(), st0.data_ptr(), rec.data_ptr(), N * H * H, C, 1e-5, 1, 2,
                          SC.data_ptr(), N, H, H, parts) == 0
    assert L.dsspk_conv_fwd(s, act0.data_ptr(), W.data_ptr(), None, y0.data_ptr(), N, H, H, C, C, 3, 3, 1, 1, 0, None) == 0
    a, a0, c, c0 = host(act), host(act0), host(y), host(y0)
    quiet = np.abs(c0) < 1e6
    assert np.isfinite(c).all() and np.max(np.abs(a - a0) / np.maximum(np.abs(a0), 1)) < 4e-6
    assert rel_l2(c[quiet], c0[quiet]) < 2e-6 and rel_l2(c, c0) < 2e-6
    assert fwd(*args, N, 32, 16, short_half=1) == -1


# family, images, channels in front, stride, height and width of the result, channels: the stem and the stride-2 convolutions in front of each
# family, at the ends of the batches for which a residual network's step has the records merged by the kernel behind
FRONT = [("small", N, 3, 1, 32, 16) for N in (1, 16)] + [("middle", 64, 3, 1, 32, 16)]
FRONT += [("small", N, 16, 2, 16, 32) for N in (1, 32)] + [("middle", N, 16, 2, 16, 32) for N in (33, 64)]
FRONT += [("small", N, 32, 2, 8, 64) for N in (1, 32)] + [("middle", N, 32, 2, 8, 64) for N in (33, 96)] + [("large", N, 32, 2, 8, 64) for N in (97, 128)]


@pytest.mark.parametrize("family,N,Cin,stride,H,C", FRONT)
def test_convolution_behind_a_generic_one(family, N, Cin, stride, H, C):
    """Records of a generic convolution, another number than the family's own leaves, merged in the loader of the 3x3 kernel behind it, against
    the batch norm by itself on the same records (the same sums in another order) and the plain convolution."""
    g = np.random.default_rng(N + C)
    f = lambda *sh: dev(g.standard_normal(sh).astype(np.float32))
    L, s = B.lib(), stream_ptr()
    shape = (N, H * stride, H * stride, Cin, C, 3, 3, stride, 1)
    parts = L.dsspk_conv_fwd_records_parts(*shape)
    assert parts > 0
    own, fwd = _family(family, N, H, C)
    x0, w0, W, G, BE = f(N, H * stride, H * stride, Cin), 0.3 * f(3, 3, Cin, C), 0.1 * f(3, 3, C, C), 1 + 0.1 * f(C), 0.1 * f(C)
    x, rec, out = empty((N, H, H, C)), empty((parts, C, 2)), empty((own, C, 2))
    assert L.dsspk_conv_fwd_records(s, x0.data_ptr(), w0.data_ptr(), x.data_ptr(), rec.data_ptr(), *shape) == 0
    act, act0, st, st0, y, y0 = empty(x.shape), empty(x.shape), empty(2 * C), empty(2 * C), empty(x.shape), empty(x.shape)
    assert fwd(s, x.data_ptr(), rec.data_ptr(), parts, G.data_ptr(), BE.data_ptr(), 1e-5, None, act.data_ptr(), st.data_ptr(), W.data_ptr(), y.data_ptr(),
               out.data_ptr(), N, H, C) == 0
    assert L.dsspk_bn_fwd(s, x.data_ptr(), G.data_ptr(), BE.data_ptr(), act0.data_ptr(), st0.data_ptr(), rec.data_ptr(), N * H * H, C, 1e-5, 1, 0,
                          None, 0, 0, 0, parts) == 0
    assert L.dsspk_conv_fwd(s, act0.data_ptr(), W.data_ptr(), None, y0.data_ptr(), N, H, H, C, C, 3, 3, 1, 1, 0, None) == 0
    assert rel_l2(host(st), host(st0)) < 1e-6 and rel_l2(host(act), host(act0)) < 1e-6 and rel_l2(host(y), host(y0)) < 2e-6
    want = _records(own, C, host(y))
    assert np.max(np.abs(host(out)[..., 0] - want[..., 0])) < 2e-6 * np.abs(host(y)).max() and rel_l2(host(out)[..., 1], want[..., 1]) < 2e-6
