"""The 3x3 kernels as a residual network's step launches them (dsspk_conv3x3_step_*: converted filters, a block's inner activation worked out again, the
last stage's d-filter beside its d-input) against the launchers of single layers, which test_gpu_conv3x3*.py, test_gpu_range.py and
test_gpu_step_kernels.py hold to the oracle: the same bits, in every size of workgroup, also where operands or one filter value leave the range of the
bf16 terms.  (There the fused last stage recomputes other tiles than the d-filter kernel of its own: 2e-6, as between those kernels' forms.)"""
import ctypes

import numpy as np
import pytest

from paper_1908_11848_amd import binding as B
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr
from test_gpu_conv3x3_large import SHAPES, _records
from test_gpu_range import check, f64

MEDIUM, LARGE, SMALL = 0, 1, 2
NAMES = {LARGE: "large", SMALL: "small"}
VALUES = ("inf", "nan", "3.395e38", "1.1e31")       # of one weight: not held by three terms, or too large for the sums
SIZES = [(size, N, H, C) for size, batches in ((SMALL, (1, 3, 13, 32)), (MEDIUM, (1, 33, 96)), (LARGE, (3, 128))) for N in batches for H, C in SHAPES]


def same(a, b, what):
    a, b = host(a), host(b)
    assert np.array_equal(a, b, equal_nan=True), (what, int((a != b).sum()), a.size)


def parts_of(size, N, H, C):
    L = B.lib()
    return L.dsspk_conv_fwd_stat_parts(N, H, H, C, C, 3, 3, 1, 1) if size == MEDIUM else getattr(L, "dsspk_conv3x3_%s_parts" % NAMES[size])(N, H, C)


def planes_of(w, C):
    p = empty(B.lib().dsspk_conv3x3_filter_bytes(C) // 4)
    assert B.lib().dsspk_conv3x3_filters(stream_ptr(), w.data_ptr(), p.data_ptr(), C) == 0
    return p


def test_what_is_refused():
    """Before anything is launched (no pointer is read)."""
    L, p, q, r, n = B.lib(), 4096, 8192, 12288, None
    assert [L.dsspk_conv3x3_filter_bytes(C) for C in (16, 32, 48, 64)] == [9 * 16 * 16 * 16, 9 * 32 * 32 * 12, 0, 9 * 64 * 64 * 12]
    assert L.dsspk_conv3x3_filters(n, p, q, 48) == -1 and L.dsspk_conv3x3_filters(n, n, q, 16) == -1

    def fwd(size, planes=q, parts=0, shortcut=n, half=0, N=4, H=32, C=16, src=p):
        return L.dsspk_conv3x3_step_fwd(n, size, src, n, parts, n, n, 1e-5, shortcut, n, n, p, planes, r, r, half, N, H, C)

    def bwd(size, planes=q, totals=n, dx=n, partial=n, gp=n, quads=0, chunks=0, red=n, N=4, H=32, C=16):
        return L.dsspk_conv3x3_step_bwd(n, size, p, p, p, p, totals, q, 4, p, p, dx, partial, p, planes, n, r, p, p, p, gp, n, p, red, n, 0, chunks, quads, N,
                                        H, C)

    for size in (MEDIUM, LARGE, SMALL):
        assert fwd(size, planes=n) == -1 and fwd(size, src=r) == -1 and fwd(size, parts=3) == -1 and fwd(size, H=31) == -1 and fwd(size, N=0) == -1
        assert fwd(size, half=1) == -1 and fwd(size, shortcut=p) == -1
        assert bwd(size, planes=n, partial=r) == -1 and bwd(size) == -1 and bwd(size, dx=r, partial=r) == -1 and bwd(size, gp=p, partial=r) == -1
        assert bwd(size, partial=r, quads=1, chunks=65) == -1 and bwd(size, H=8, C=64) == -1 and bwd(size, partial=r, red=p) == -1
    assert bwd(MEDIUM, partial=r) == -1 and bwd(LARGE, totals=p, partial=r) == -1 and bwd(LARGE, H=8, C=64, partial=r) == -1 and fwd(3) == -1
    assert fwd(SMALL, N=33) == -1 and fwd(LARGE, N=129) == -1


def forward(size, N, H, C, w, x, rec, gamma, beta, shortcut, half):
    """(destination, activation, mean and invstd, records) of a step's launch and of the single layers'."""
    L, s, parts = B.lib(), stream_ptr(), parts_of(size, N, H, C)
    planes, out = planes_of(w, C), []
    for step in (True, False):
        y, act, st, r = empty((N, H, H, C)), empty((N, H, H, C)), empty(2 * C), empty((parts, C, 2))
        bn = (None, 0, None, None, 1e-5, None, None, None) if gamma is None else (
            rec.data_ptr(), parts, gamma.data_ptr(), beta.data_ptr(), 1e-5, None if shortcut is None else shortcut.data_ptr(), act.data_ptr(), st.data_ptr())
        if step:
            rc = L.dsspk_conv3x3_step_fwd(s, size, x.data_ptr(), *bn, w.data_ptr(), planes.data_ptr(), y.data_ptr(), r.data_ptr(), half, N, H, C)
        elif size != MEDIUM:
            rc = getattr(L, "dsspk_conv3x3_%s_fwd" % NAMES[size])(s, x.data_ptr(), *bn, w.data_ptr(), y.data_ptr(), r.data_ptr(), half, N, H, C)
        elif gamma is None:
            rc = L.dsspk_conv_fwd(s, x.data_ptr(), w.data_ptr(), None, y.data_ptr(), N, H, H, C, C, 3, 3, 1, 1, 0, r.data_ptr())
        else:
            rc = (L.dsspk_conv_fwd_prebn_half if half else L.dsspk_conv_fwd_prebn)(s, x.data_ptr(), *bn, w.data_ptr(), y.data_ptr(), r.data_ptr(), N, H, C)
        assert rc == 0
        out.append((y, act, st, r))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("form,size,N,H,C", [(form, *at) for form in ("plain", "bn", "bn+shortcut", "bn+half") for at in SIZES
                                             if form != "bn+half" or at[3] > 16])       # no stage has a shortcut from 8 channels
def test_forward(size, N, H, C, form):
    g = np.random.default_rng(N + C)
    f = lambda *sh: g.standard_normal(sh).astype(np.float32)
    x, w = f(N, H, H, C) + 0.5, dev(np.sqrt(2.0 / (9 * C)) * f(3, 3, C, C))
    gamma, beta = (None, None) if form == "plain" else (dev(1 + 0.1 * f(C)), dev(0.1 * f(C)))
    half = form == "bn+half"
    shortcut = dev(f(N, 2 * H, 2 * H, C // 2)) if half else dev(f(N, H, H, C)) if form == "bn+shortcut" else None
    a, b = forward(size, N, H, C, w, dev(x), dev(_records(parts_of(size, N, H, C), C, x)), gamma, beta, shortcut, int(half))
    assert np.isfinite(host(a[0])).all()
    for i, what in enumerate(("convolution", "activation", "mean, invstd", "records")):
        same(a[i], b[i], what)


def backward_inputs(size, N, H, C, kind):
    """What the backward pass of a block's second convolution meets: x_in is ReLU(BN(xp)) as the forward pass left it.  far-x, far-dz: one channel of
    it, or one element of dz, beyond the range of the scaled terms (not both: their products would be infinite)."""
    g = np.random.default_rng(N + C)
    f = lambda *sh: g.standard_normal(sh).astype(np.float32)
    w, xp = f(3, 3, C, C), f(N, H, H, C)
    gp, bp, ga, stats = f(C), f(C), f(C), np.concatenate([f(C), np.abs(f(C)) + 0.5])
    dz = f(N, H, H, C)
    if kind == "far-x":
        gp[C - 1] = 2e32
    elif kind == "far-dz":
        dz[0, 1, 2, 3], ga[3] = 3e31, 1         # invstd is 0.5 at least: a gradient of 1.5e31 or more goes into the products, the terms hold 1.01e31
    elif kind != "ordinary":
        w[1, 2, 5, 7] = float(kind)
    t = {"dz": dev(dz), "xc": dev(f(N, H, H, C)), "add": dev(f(N, H, H, C)), "w": dev(w), "gamma": dev(ga), "xp": dev(xp), "gp": dev(gp), "bp": dev(bp),
         "stats": dev(stats)}
    plain = dev(np.zeros((3, 3, C, C), np.float32))
    (_, t["xin"], t["statsp"], _), _ = forward(size, N, H, C, plain, t["xp"], dev(_records(parts_of(size, N, H, C), C, xp)), t["gp"], t["bp"], None, 0)
    return t


@pytest.mark.gpu
@pytest.mark.parametrize("kind,size,N,H,C", [(kind, *at) for kind in ("ordinary", "far-x", "far-dz") + VALUES for at in SIZES
                                             if kind not in VALUES or at[1] <= 33])
def test_backward(size, N, H, C, kind):
    """Without and with the inner activation worked out again; with and without a shortcut's gradient (the first and the second convolution of a block)."""
    L, s = B.lib(), stream_ptr()
    t = backward_inputs(size, N, H, C, kind)
    planes, parts, E = planes_of(t["w"], C), parts_of(size, N, H, C), 9 * C * C
    P = {k: v.data_ptr() for k, v in t.items()}
    g = np.random.default_rng(1)
    rin, job = dev(g.standard_normal((parts, C, 2)).astype(np.float32)), dev(g.standard_normal((11, 2304)).astype(np.float32))
    tot, dg0, db0 = empty(2 * C), empty(C), empty(C)
    assert L.dsspk_bn_bwd_totals(s, rin.data_ptr(), parts, C, tot.data_ptr(), dg0.data_ptr(), db0.data_ptr()) == 0
    wide = size == SMALL and C == 64                    # d-filter beside the d-input; the single layers have a kernel of its own for it
    chunks = N if wide else parts if C < 64 else 0

    def run(step, repeat, add):
        d = dict(out=empty((N, H, H, C)), rec=empty((parts, C, 2)), jw=empty(2304), dg=empty(C), db=empty(C))
        d["partial" if C < 64 or (wide and step) else "dx"] = o = empty((chunks, E)) if C < 64 or (wide and step) else empty((N, H, H, C))
        dx, partial = (None, o.data_ptr()) if "partial" in d else (o.data_ptr(), None)
        add = P["add"] if add else None
        red = (job.data_ptr(), d["jw"].data_ptr(), 2304, 11)
        sums = (None, rin.data_ptr(), parts, d["dg"].data_ptr(), d["db"].data_ptr()) if size != MEDIUM else (tot.data_ptr(), None, 0, None, None)
        if step:
            rc = L.dsspk_conv3x3_step_bwd(s, size, P["dz"], P["xc"], P["stats"], P["gamma"], *sums, dx, partial, P["w"], planes.data_ptr(), add,
                                          d["out"].data_ptr(), P["xin"], P["xp"], P["statsp"], P["gp"] if repeat else None, P["bp"] if repeat else None,
                                          d["rec"].data_ptr(), *red, 0, N, H, C)
        elif size != MEDIUM:
            rc = getattr(L, "dsspk_conv3x3_%s_bwd" % NAMES[size])(s, P["dz"], P["xc"], P["stats"], P["gamma"], *sums[1:], dx, partial, P["w"], add,
                                                                  d["out"].data_ptr(), P["xin"], P["xp"], P["statsp"], d["rec"].data_ptr(), *red, N, H, C)
        elif C < 64:
            rc = L.dsspk_conv_bwd_data_bn_wgrad(s, P["dz"], P["xc"], P["stats"], P["gamma"], tot.data_ptr(), P["w"], add, d["out"].data_ptr(), P["xp"],
                                                P["statsp"], d["rec"].data_ptr(), P["xin"], partial, *red, N, H, C)
        else:
            rc = L.dsspk_conv_bwd_data_bn(s, P["dz"], P["xc"], P["stats"], P["gamma"], tot.data_ptr(), dx, P["w"], add, d["out"].data_ptr(), P["xin"],
                                          P["xp"], P["statsp"], d["rec"].data_ptr(), *red, N, H, C)
        assert rc == 0
        return d

    for add in (True, False):
        want = run(False, False, add)
        if kind == "ordinary":
            assert all(np.isfinite(host(v)).all() for k, v in want.items() if size != MEDIUM or k not in ("dg", "db"))
        elif kind == "far-dz":
            assert np.abs(host(want["out"])).max() > 1e30
        elif kind == "far-x":
            assert np.abs(host(t["xin"])).max() > 1e32
        if wide:
            scr, dw, n = empty(L.dsspk_conv_wgrad_scratch_floats(N, H, H, C, C, 3, 3, 1, 1)), empty(E), ctypes.c_int(0)
            assert L.dsspk_conv_bwd_weight_parts(s, P["xin"], want["dx"].data_ptr(), scr.data_ptr(), N, H, H, C, C, 3, 3, 1, 1, None, 0, 0, None, None, None,
                                                 ctypes.byref(n)) == 0
            assert L.dsspk_wgrad_reduce(s, scr.data_ptr(), dw.data_ptr(), E, n.value) == 0
        for repeat in (False, True):
            got = run(True, repeat, add)
            for k in set(got) & set(want):
                same(got[k], want[k], (k, "repeat" if repeat else "read", add))
            if wide:                    # the partial results, added up as a job that the next launch carries
                sums, again = empty(E), run(True, repeat, add)
                assert L.dsspk_conv3x3_step_bwd(s, size, P["dz"], P["xc"], P["stats"], P["gamma"], None, rin.data_ptr(), parts, again["dg"].data_ptr(),
                                                again["db"].data_ptr(), None, again["partial"].data_ptr(), P["w"], planes.data_ptr(), None,
                                                again["out"].data_ptr(), P["xin"], P["xp"], P["statsp"], None, None, again["rec"].data_ptr(),
                                                got["partial"].data_ptr(), sums.data_ptr(), E, N, 1, N, H, C) == 0
                if kind in ("far-x", "far-dz"):
                    assert rel_l2(host(sums), host(dw)) < 2e-6 and max_abs(host(sums), host(dw)) < 2e-5
                else:
                    same(sums, dw, ("d-filter", repeat, add))


@pytest.mark.gpu
@pytest.mark.parametrize("size,N", [(SMALL, 3), (MEDIUM, 3), (LARGE, 3)])
@pytest.mark.parametrize("H,C", SHAPES)
@pytest.mark.parametrize("value", VALUES)
def test_filter_value_beyond_the_terms(oracle_nn, size, N, H, C, value):
    """One weight that three terms cannot hold (or that is too large for the sums), through the conversion: against float64."""
    g = np.random.default_rng(C)
    x, w = (0.1 * g.standard_normal((N, H, H, C))).astype(np.float32), (0.05 * g.standard_normal((3, 3, C, C))).astype(np.float32)
    w[1, 2, 5, 7] = float(value)
    (y, _, _, r), (y1, _, _, r1) = forward(size, N, H, C, dev(w), dev(x), None, None, None, None, 0)
    same(y, y1, "convolution")
    same(r, r1, "records")
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    with np.errstate(all="ignore"):
        check(host(y), oracle_nn.conv2d_fwd(*f64(xp, w), None, 1, 0))
