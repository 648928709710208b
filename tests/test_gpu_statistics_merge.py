"""Sums over the records of a batch norm.  In the loaders of the 3x3 kernels: error of mean and invstd against float64 over many channels, no larger than that of
the plain formula in fp32 (the mean of all records, then all deviations from it; a lane's records in turn, lanes in pairs, wavefronts in turn).  In the kernels
of their own: the order of the sums, bit for bit."""
import numpy as np
import pytest

from paper_1908_11848_amd import binding as B
from gpu_util import dev, empty, host, stream_ptr
from test_gpu_conv3x3_large import SHAPES

EPS, DRAWS = 1e-5, 12
f32 = np.float32


def plain(rec, n, waves):
    """rec: (mean, sum of squared deviations) of n rows each, [parts][C] float32 -> mean, invstd."""
    parts, C = rec.shape[:2]
    lanes = 64 * waves // C
    v = np.zeros((-(-parts // lanes) * lanes, C, 2), f32)
    v[:parts] = rec
    v = v.reshape(-1, waves, 64 // C, C, 2)
    there = (np.arange(v.shape[0] * lanes) < parts).reshape(v.shape[:3] + (1,))

    def total(t):
        s = np.zeros(t.shape[1:], f32)
        for u in t:
            s = s + u
        while s.shape[1] > 1:
            s = s[:, :s.shape[1] // 2] + s[:, s.shape[1] // 2:]
        out = s[0, 0]
        for w in s[1:, 0]:
            out = out + w
        return out

    M = f32(n * parts)
    mean = total(f32(n) * v[..., 0]) / M                        # (n is a power of two: the product is exact)
    d = v[..., 0] - mean
    m2 = total(np.where(there, (v[..., 1] + (f32(n) * d).astype(np.float64) * d).astype(f32), f32(0)))
    return mean, f32(1) / np.sqrt(m2 / M + f32(EPS))


def drawn(g, parts, n, C, spread):
    sd = 1 + np.abs(g.standard_normal(C))
    m = sd * g.standard_normal(C) + spread * sd / np.sqrt(n) * g.standard_normal((parts, C))
    return np.stack([m, np.abs(n * sd ** 2 * (1 + 0.2 * g.standard_normal((parts, C))))], axis=2).astype(f32)


def exact(rec, n):
    r = rec.astype(np.float64)
    mean = r[..., 0].mean(0)
    var = (r[..., 1].sum(0) + n * ((r[..., 0] - mean) ** 2).sum(0)) / (n * len(r))
    return mean, 1 / np.sqrt(var + EPS)


def errors(got, want):
    """Of the mean in units of the standard deviation, of invstd relative."""
    return np.stack([(got[0] - want[0]) * want[1], got[1] / want[1] - 1])


@pytest.mark.gpu
@pytest.mark.parametrize("family,batches", [("small", (1, 3, 8, 13, 32)), ("large", (97, 110, 128))])
@pytest.mark.parametrize("H,C", SHAPES)
@pytest.mark.parametrize("spread", [1, 30])                     # of the records' means, 1: rows that do not depend on each other
def test_error(family, batches, H, C, spread):
    """Root mean square over 576 to 3840 channels.  The same arithmetic in numpy: 0.81 to 0.998 of the plain formula's; with the shares' sums put together
    in fp32 up to 1.065."""
    L, s = B.lib(), stream_ptr()
    ours, theirs = [], []
    for N in batches:
        parts = getattr(L, "dsspk_conv3x3_%s_parts" % family)(N, H, C)
        n = N * H * H // parts
        x, w = dev(np.zeros((N, H, H, C), f32)), dev(np.zeros((3, 3, C, C), f32))
        gamma, beta, act, y, rec = dev(np.ones(C, f32)), dev(np.zeros(C, f32)), empty((N, H, H, C)), empty((N, H, H, C)), empty((parts, C, 2))
        for draw in range(DRAWS):
            r = drawn(np.random.default_rng((N, draw)), parts, n, C, spread)
            R, st = dev(r), empty(2 * C)
            assert getattr(L, "dsspk_conv3x3_%s_fwd" % family)(s, x.data_ptr(), R.data_ptr(), parts, gamma.data_ptr(), beta.data_ptr(), EPS, None,
                                                              act.data_ptr(), st.data_ptr(), w.data_ptr(), y.data_ptr(), rec.data_ptr(), 0, N, H, C) == 0
            want = exact(r, n)
            ours.append(errors(host(st).astype(np.float64).reshape(2, C), want))
            theirs.append(errors(plain(r, n, 8 if family == "large" else 4), want))
    rms = lambda e: np.sqrt(np.mean(np.square(np.concatenate(e, axis=1)), axis=1))
    ours, theirs = rms(ours), rms(theirs)
    assert (ours <= theirs).all(), (ours, theirs)


@pytest.mark.gpu
@pytest.mark.parametrize("N", [33, 48, 96])
@pytest.mark.parametrize("H,C", SHAPES)
def test_tree_of_sums(N, H, C):
    """The merge ahead of the four-wavefront kernels, 64 lanes a channel: a lane's records in turn, then a tree that adds the farther half of the lanes, bit
    for bit (of the products one is exact and one is in an fma: one element in 100 for the emulation's double roundings)."""
    L, s = B.lib(), stream_ptr()
    parts = L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1)
    n, M = N * H * H // parts, f32(N * H * H)
    r = drawn(np.random.default_rng(N), parts, n, C, 1)
    R, x, w = dev(r), dev(np.zeros((N, H, H, C), f32)), dev(np.zeros((3, 3, C, C), f32))
    gamma, beta, act, y, st, rec = dev(np.ones(C, f32)), dev(np.zeros(C, f32)), empty((N, H, H, C)), empty((N, H, H, C)), empty(2 * C), empty((parts, C, 2))
    assert L.dsspk_conv_records_inline(parts, C) == 0
    assert L.dsspk_conv_fwd_prebn(s, x.data_ptr(), R.data_ptr(), parts, gamma.data_ptr(), beta.data_ptr(), EPS, None, act.data_ptr(), st.data_ptr(),
                                  w.data_ptr(), y.data_ptr(), rec.data_ptr(), N, H, C) == 0
    v = np.zeros((-(-parts // 64) * 64, C, 2), f32)
    v[:parts] = r
    v, there = v.reshape(-1, 64, C, 2), (np.arange(-(-parts // 64) * 64) < parts).reshape(-1, 64, 1)

    def tree(t):
        s = np.zeros(t.shape[1:], f32)
        for u in t:
            s = s + u
        while len(s) > 1:
            s = s[:len(s) // 2] + s[len(s) // 2:]
        return s[0]

    mean = tree(f32(n) * v[..., 0]) / M
    d = v[..., 0] - mean
    m2 = tree(np.where(there, (v[..., 1] + (f32(n) * d).astype(np.float64) * d).astype(f32), f32(0)))
    got = host(st)
    assert np.array_equal(got[:C], mean)
    assert np.mean(got[C:] != f32(1) / np.sqrt(m2 / M + f32(EPS))) <= 0.01


@pytest.mark.gpu
@pytest.mark.parametrize("M,C", [(100, 4), (100, 64), (3000, 16), (50001, 32)])
def test_gradient_behind_a_batch_norm(M, C):
    """dx of gradients with a large mean, which cancels, from the sums the kernel stored: one rounding for d - mean, bit for bit.  (Double roundings of this
    emulation: fewer than one element in 1000.)"""
    g = np.random.default_rng(M + C)
    L, s, f = B.lib(), stream_ptr(), lambda *sh: g.standard_normal(sh).astype(f32)
    x, gamma, da = f(M, C), 1 + 0.1 * f(C), 100 + f(M, C)
    X, G, BE, DA, y, st, dx = dev(x), dev(gamma), dev(f(C)), dev(da), empty((M, C)), empty(2 * C), empty((M, C))
    scr, dg, db = empty(L.dsspk_bn_scratch_floats(M, C)), empty(C), empty(C)
    assert L.dsspk_bn_fwd(s, X.data_ptr(), G.data_ptr(), BE.data_ptr(), y.data_ptr(), st.data_ptr(), scr.data_ptr(), M, C, EPS, 0, 0, None, 0, 0, 0, 0) == 0
    assert L.dsspk_bn_bwd(s, X.data_ptr(), G.data_ptr(), st.data_ptr(), DA.data_ptr(), None, dx.data_ptr(), dg.data_ptr(), db.data_ptr(), scr.data_ptr(), M, C) == 0
    st, dg, db, inv = host(st), host(dg), host(db), f32(1) / f32(M)
    fma = lambda a, b, c: (a.astype(np.float64) * b + c).astype(f32)
    d, hat = fma(-db, inv, da), (x - st[:C]) * st[C:]
    want = gamma * st[C:] * fma(-hat, (dg * inv).astype(np.float64), d)
    assert np.mean(host(dx) != want) < 1e-3
