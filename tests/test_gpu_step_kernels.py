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
