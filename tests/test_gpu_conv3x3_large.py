"""The 3x3 kernels with larger workgroups (dsspk_conv3x3_large_*) against float64 and against the kernels with four wavefronts, which
test_gpu_conv3x3.py and test_gpu_range.py hold to the oracle.  Sizes: one image, a few, the smallest batch that takes them and the
largest they cover (16 channels: two bands an image; each thread then holds its full number of records)."""
import numpy as np
import pytest

from paper_1908_11848_amd import binding as B
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr

SHAPES = [(32, 16), (16, 32), (8, 64)]
SIZES = [(N, H, C) for N in (1, 3, 33, 128) for H, C in SHAPES]


def test_what_is_covered():
    L = B.lib()
    for H, C in SHAPES:
        assert [L.dsspk_conv3x3_large_parts(N, H, C) for N in (0, 1, 128, 129)] == [0, 2 if C == 16 else 1, 256 if C == 16 else 128, 0]
        assert L.dsspk_conv3x3_large_parts(4, H + 1, C) == 0 and L.dsspk_conv3x3_large_parts(4, H, C + 16) == 0
    assert L.dsspk_conv3x3_large_fwd(None, None, None, 0, None, None, 1e-5, None, None, None, None, None, None, 0, 4, 32, 16) == -1


def _records(parts, C, x):
    """(mean, sum of squared deviations) of equal slabs of the rows of x."""
    r = x.reshape(parts, -1, C).astype(np.float64)
    m = r.mean(1)
    return np.stack([m, ((r - m[:, None]) ** 2).sum(1)], axis=2).astype(np.float32)


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,C", SIZES)
@pytest.mark.parametrize("form", ["plain", "bn", "bn+shortcut"])
def test_forward(oracle_nn, N, H, C, form):
    forward(oracle_nn, "large", N, H, C, form)


def forward(oracle_nn, family, N, H, C, form):
    """dsspk_conv3x3_<family>_fwd.  Convolution 2e-7 as in test_gpu_conv3x3.py plus the activations' rounding (about 1e-7 each): 4e-7."""
    g = np.random.default_rng(N + C)
    f = lambda *sh: g.standard_normal(sh).astype(np.float32)
    x, sc, w = f(N, H, H, C) + 0.5, f(N, H, H, C), (np.sqrt(2.0 / (9 * C)) * f(3, 3, C, C)).astype(np.float32)
    gamma, beta = 1 + 0.1 * f(C), 0.1 * f(C)
    L, s = B.lib(), stream_ptr()
    parts, fwd = getattr(L, "dsspk_conv3x3_%s_parts" % family)(N, H, C), getattr(L, "dsspk_conv3x3_%s_fwd" % family)
    X, SC, W, G, BE, REC = dev(x), dev(sc), dev(w), dev(gamma), dev(beta), dev(_records(parts, C, x))
    act, stats, y, rec = empty((N, H, H, C)), empty(2 * C), empty((N, H, H, C)), empty((parts, C, 2))
    a = x.astype(np.float64)
    if form == "plain":
        assert fwd(s, X.data_ptr(), None, 0, None, None, 1e-5, None, None, None, W.data_ptr(), y.data_ptr(), rec.data_ptr(), 0, N, H, C) == 0
    else:
        short = SC.data_ptr() if form == "bn+shortcut" else None
        assert fwd(s, X.data_ptr(), REC.data_ptr(), parts, G.data_ptr(), BE.data_ptr(), 1e-5, short, act.data_ptr(), stats.data_ptr(), W.data_ptr(),
                   y.data_ptr(), rec.data_ptr(), 0, N, H, C) == 0
        mean, var = a.mean((0, 1, 2)), a.var((0, 1, 2))
        st = host(stats).reshape(2, C)
        assert max_abs(st[0], mean) < 2e-6 and rel_l2(st[1], 1 / np.sqrt(var + 1e-5)) < 1e-6
        a = (a - mean) / np.sqrt(var + 1e-5) * gamma + beta
        if short:
            a = a + sc
        a = np.maximum(a, 0)
        assert rel_l2(host(act), a) < 4e-7
    want = oracle_nn.conv2d_fwd(a, w.astype(np.float64), None, 1, 1)
    assert rel_l2(host(y), want) < 4e-7 and max_abs(host(y), want) < 4e-6
    got = _records(parts, C, host(y))
    assert np.max(np.abs(host(rec)[..., 0] - got[..., 0])) < 2e-6 * np.abs(want).max() and rel_l2(host(rec)[..., 1], got[..., 1]) < 2e-6


def _backward_inputs(N, H, C, large):
    import torch
    g = np.random.default_rng(N + C)
    f = lambda *sh: dev(g.standard_normal(sh).astype(np.float32))
    d = {"dz": f(N, H, H, C), "xc": f(N, H, H, C), "xp": f(N, H, H, C), "xin": torch.relu(f(N, H, H, C)), "add": f(N, H, H, C), "w": f(3, 3, C, C),
         "stats": torch.cat([f(C), f(C).abs() + 0.5]), "statsp": torch.cat([f(C), f(C).abs() + 0.5]), "gamma": f(C)}
    if large:                       # beyond the range of the scaled terms, in dz and in x, in the first and the last image
        d["dz"][0, 1, 2, 3], d["xin"][N - 1, H - 1, 0, C - 1] = 3e31, 2e32
    return d


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,C", SIZES)
@pytest.mark.parametrize("large", [False, True])
def test_backward(N, H, C, large):
    backward("large", N, H, C, large)


def backward(family, N, H, C, large):
    """dsspk_conv3x3_<family>_bwd against dsspk_conv_bwd_data_bn(_wgrad) behind dsspk_bn_bwd_totals: the same products in the same order per output; sums over the
    batch and over the records in another: 2e-6 of the result, as between those kernels' own forms."""
    L, s = B.lib(), stream_ptr()
    t = _backward_inputs(N, H, C, large)
    P = {k: v.data_ptr() for k, v in t.items()}
    parts, parts4 = getattr(L, "dsspk_conv3x3_%s_parts" % family)(N, H, C), L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1)
    bwd = getattr(L, "dsspk_conv3x3_%s_bwd" % family)
    rin = dev(np.random.default_rng(1).standard_normal((parts, C, 2)).astype(np.float32))
    tot, dgam, dbet, dg, db = empty(2 * C), empty(C), empty(C), empty(C), empty(C)
    assert L.dsspk_bn_bwd_totals(s, rin.data_ptr(), parts, C, tot.data_ptr(), dgam.data_ptr(), dbet.data_ptr()) == 0
    E, fused = 9 * C * C, C < 64
    out, rec, other = empty((N, H, H, C)), empty((parts, C, 2)), empty(parts * E) if fused else empty((N, H, H, C))
    out4, rec4, other4 = empty((N, H, H, C)), empty((parts4, C, 2)), empty(parts4 * E) if fused else empty((N, H, H, C))
    # an unrelated d-filter reduction that both carry
    job = dev(np.random.default_rng(2).standard_normal((70, 2304)).astype(np.float32))
    jw, jw4 = empty(2304), empty(2304)
    o = other.data_ptr()
    assert bwd(s, P["dz"], P["xc"], P["stats"], P["gamma"], rin.data_ptr(), parts, dg.data_ptr(), db.data_ptr(), None if fused else o,
               o if fused else None, P["w"], P["add"], out.data_ptr(), P["xin"], P["xp"], P["statsp"], rec.data_ptr(), job.data_ptr(), jw.data_ptr(), 2304,
               70, N, H, C) == 0
    red = (job.data_ptr(), jw4.data_ptr(), 2304, 70, N, H, C)
    if fused:
        assert L.dsspk_conv_bwd_data_bn_wgrad(s, P["dz"], P["xc"], P["stats"], P["gamma"], tot.data_ptr(), P["w"], P["add"], out4.data_ptr(), P["xp"],
                                              P["statsp"], rec4.data_ptr(), P["xin"], other4.data_ptr(), *red) == 0
        sums = []
        for part, n in ((other, parts), (other4, parts4)):
            dw = empty(E)
            assert L.dsspk_wgrad_reduce(s, part.data_ptr(), dw.data_ptr(), E, n) == 0
            sums.append(host(dw))
    else:
        assert L.dsspk_conv_bwd_data_bn(s, P["dz"], P["xc"], P["stats"], P["gamma"], tot.data_ptr(), other4.data_ptr(), P["w"], P["add"], out4.data_ptr(),
                                        P["xin"], P["xp"], P["statsp"], rec4.data_ptr(), *red) == 0
        sums = [host(other), host(other4)]
    assert np.array_equal(host(jw), host(jw4))
    assert np.max(np.abs(host(dg) - host(dgam))) < 1e-6 * np.sqrt(parts) and np.max(np.abs(host(db) - host(dbet))) < 1e-6 * np.sqrt(parts)
    r, r4 = host(rec).astype(np.float64).sum(0), host(rec4).astype(np.float64).sum(0)
    for a, b in [(host(out), host(out4)), tuple(sums), (r, r4)]:
        assert np.isfinite(b).all()
        assert rel_l2(a, b) < 2e-6 and np.max(np.abs(a - b)) < 2e-5 * np.abs(b).max()
