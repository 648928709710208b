"""The launches of a residual network's step that stand for several others, on their own: its end in one kernel (dsspk_head_step) and both gradients of a
stride-2 convolution in one (dsspk_stride2_step_bwd).  What is worked out as in the launches they replace has their bits; sums in another order
are held to float64 element by element, within the rounding errors of their terms; infinities and NaN come out where the launches one by one have them."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1908_11848_amd import binding as B
from gpu_util import dev, empty, host, stream_ptr

U = 2.0 ** -24                                      # a rounding of fp32
f64 = lambda t: host(t).astype(np.float64)


def same(a, b, what):
    a, b = host(a), host(b)
    assert np.array_equal(a, b, equal_nan=True), (what, int((a != b).sum()), a.size)


def within(got, want, bound, what):
    worst = np.max(np.abs(f64(got) - want) - bound)
    assert worst <= 0, (what, worst, np.max(np.abs(want)))


def not_finite_alike(a, b, what):
    """The same infinities and NaN, and 1e-4 on what remains (two fp32 sums of up to 64 terms; values up to the largest finite one)."""
    a, b = host(a).astype(np.float64), host(b).astype(np.float64)
    assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a == np.inf, b == np.inf) and np.array_equal(a == -np.inf, b == -np.inf), what
    ok = np.isfinite(a)
    scale = np.max(np.abs(b[ok]), initial=0)
    assert np.max(np.abs(a[ok] - b[ok]), initial=0) <= 1e-4 * scale, what


def test_what_is_refused():
    """Before anything is launched (no pointer is read)."""
    L, n, p, ch = B.lib(), None, [4096 * (i + 1) for i in range(16)], ctypes.c_int(0)
    assert [L.dsspk_head_step_takes(*a) for a in ((4, 4, 10), (0, 4, 10), (4, 0, 10), (4, 3, 10), (4, 4, 0), (4, 4, 128), (4, 4, 129), (129, 129, 10), (128, 128, 2))] == [
        1, 0, 0, 0, 0, 1, 0, 0, 1]

    def head(parts=4, classes=10, N=4, x=p[0], rec=p[1], out=p[6], dz=p[12], rout=p[13], label=p[5]):
        return L.dsspk_head_step(n, x, rec, parts, p[2], p[3], 0, p[4], label, 1e-5, out, p[7], p[8], p[9], p[10], p[11], dz, rout, N, classes)

    assert head(parts=3) == head(classes=129) == head(N=0) == head(x=n) == head(label=n) == head(dz=n) == head(out=p[0]) == head(dz=p[0]) == head(dz=p[6]) == -1
    assert head(rout=p[1]) == head(rec=n) == -1
    assert [L.dsspk_stride2_step_records(*a) for a in ((1, 32, 16), (32, 16, 32), (32, 32, 16), (33, 16, 32), (0, 32, 16), (1, 32, 32), (1, 8, 64))] == [16, 128, 512, 0, 0, 0, 0]

    def stride2(dy=p[0], sc=p[2], dx=p[3], partial=p[4], x=p[5], xc=p[6], rec=p[8], N=4, H=32, C=16, chunks=ctypes.byref(ch)):
        return L.dsspk_stride2_step_bwd(n, dy, p[1], sc, dx, partial, x, xc, p[7], rec, N, H, C, chunks)

    assert stride2(dy=n) == stride2(sc=p[3]) == stride2(dx=p[0]) == stride2(x=p[3]) == stride2(xc=p[3]) == stride2(partial=p[3]) == stride2(rec=p[4]) == -1
    assert stride2(N=33) == stride2(H=31) == stride2(C=32) == stride2(chunks=None) == stride2(rec=n) == -1


HEAD_OUT = ("out", "stats", "pooled", "logits", "dlogits", "row_loss", "dz", "records")


def head_inputs(N, classes, half, kind="ordinary", parts=None):
    g = np.random.default_rng(N + classes)
    f = lambda *sh: g.standard_normal(sh).astype(np.float32)
    x, w, bias, gamma, sc = f(N, 64, 64) + 0.3, 0.3 * f(64, classes), f(classes), 1 + 0.1 * f(64), f(N, 16, 16, 32) if half else f(N, 64, 64)
    r = x.astype(np.float64).reshape(parts or N, -1, 64)
    m = r.mean(1)
    rec = np.stack([m, ((r - m[:, None]) ** 2).sum(1)], axis=2).astype(np.float32)
    sc.reshape(-1)[7] = {"inf": np.inf, "nan": np.nan, "far": 3e38}.get(kind, sc.reshape(-1)[7])
    if kind.startswith("weight"):
        w[5, classes - 1] = {"weight inf": np.inf, "weight nan": np.nan, "weight far": 3e38}[kind]
    if kind == "class out":                         # of the question: probability 0
        bias[0] = -np.inf
    if kind == "gamma nan":
        gamma[63] = np.nan
    if kind == "records inf":
        rec[0, 9, 1] = np.inf
    label = (1 + g.integers(0, classes - 1, N)).astype(np.int32) if kind == "class out" else g.integers(0, classes, N).astype(np.int32)
    return dict(x=dev(x), rec=dev(rec), gb=dev(np.concatenate([gamma, 0.1 * f(64)])), sc=dev(sc), wb=dev(np.concatenate([w.ravel(), bias])), label=dev(label))


def head_outputs(N, classes):
    return dict(out=empty((N, 64, 64)), stats=empty(128), pooled=empty((N, 64)), logits=empty((N, classes)), dlogits=empty((N, classes)), row_loss=empty(N),
                dz=empty((N, 64, 64)), records=empty((N, 64, 2)))


def head(t, N, classes, half, parts=None):
    o, L, P = head_outputs(N, classes), B.lib(), {k: v.data_ptr() for k, v in t.items()}
    assert L.dsspk_head_step(stream_ptr(), P["x"], P["rec"], parts or N, P["gb"], P["sc"], int(half), P["wb"], P["label"], 1e-5, *(o[k].data_ptr() for k in HEAD_OUT), N, classes) == 0
    return o


def one_by_one(t, N, classes, half, parts=None):
    o, L, s, P = head_outputs(N, classes), B.lib(), stream_ptr(), {k: v.data_ptr() for k, v in t.items()}
    O = {k: v.data_ptr() for k, v in o.items()}
    w, bias, dp, dw, db = P["wb"], P["wb"] + 4 * 64 * classes, empty((N, 64)), empty((64, classes)), empty(classes)
    assert L.dsspk_bn_fwd_gap(s, P["x"], P["gb"], P["gb"] + 256, O["out"], O["stats"], P["rec"], parts or N, P["sc"], int(half), O["pooled"], N, 8, 64, 1e-5) == 0
    assert L.dsspk_fc_softmax_xent(s, O["pooled"], w, bias, P["label"], O["logits"], O["dlogits"], O["row_loss"], N, 64, classes) == 0
    assert L.dsspk_fc_bwd(s, O["pooled"], O["dlogits"], w, dw.data_ptr(), db.data_ptr(), dp.data_ptr(), 0, None, None, N, 64, classes) == 0
    assert L.dsspk_gap_bwd_bn_reduce(s, dp.data_ptr(), P["x"], O["stats"], O["out"], O["dz"], O["records"], N, 8, 64) == 0
    return o


HEADS = [(1, 2, False, 1), (13, 7, True, 13), (5, 64, False, 5), (3, 65, True, 3), (37, 127, False, 37), (128, 100, True, 128), (128, 128, False, 128),
         (6, 10, False, 1), (4, 10, True, 128), (200, 10, False, 100)]          # the last three: records of several images, of a part of one


@pytest.mark.gpu
@pytest.mark.parametrize("N,classes,half,parts", HEADS)
def test_head(N, classes, half, parts):
    """Bounds: a sum of n terms is off by at most n roundings of the sum of their magnitudes; e carries one stage's bound into the next."""
    t = head_inputs(N, classes, half, parts=parts)
    o, one = head(t, N, classes, half, parts), one_by_one(t, N, classes, half, parts)
    same(o["out"], one["out"], "output")
    same(o["stats"], one["stats"], "mean, invstd")
    out, stats, wb, label = f64(o["out"]), f64(o["stats"]), f64(t["wb"]), host(t["label"])
    w, bias, rows = wb[:64 * classes].reshape(64, classes), wb[64 * classes:], np.arange(N)
    pooled = out.mean(1)
    e = 64 * U * pooled                             # nothing is negative
    within(o["pooled"], pooled, e, "pooled")
    logits = pooled @ w + bias
    e = e @ np.abs(w) + 66 * U * (pooled @ np.abs(w) + np.abs(bias))
    within(o["logits"], logits, e, "logits")
    top = logits.max(1, keepdims=True)
    lse = top + np.log(np.exp(logits - top).sum(1, keepdims=True))
    prob, hot, e = np.exp(logits - lse), np.eye(classes)[label], e.max(1, keepdims=True)
    within(o["row_loss"], (lse[:, 0] - logits[rows, label]), 2 * e[:, 0] + 2 * classes * U + 4 * U * (np.abs(logits).max(1) + np.abs(lse[:, 0])), "loss of a row")
    # probabilities: exp of a difference (rounded), and two units of expf and of the division each
    d = (prob - hot) / N
    e = (prob * (2 * e + 2 * U * np.abs(logits - top) + (classes + 8) * U) + 4 * U * (prob + hot)) / N
    within(o["dlogits"], d, e, "gradient of the logits")
    g = (d @ w.T) / 64
    e = (e @ np.abs(w.T) + (classes + 2) * U * (np.abs(d) @ np.abs(w.T))) / 64
    mask = out > 0
    dz = np.where(mask, g[:, None], 0)
    within(o["dz"], dz, np.where(mask, e[:, None], 0), "gradient in front of the ReLU")
    hat = (f64(t["x"]) - stats[:64]) * stats[64:]
    sums = np.stack([dz.sum(1), (dz * hat).sum(1)], axis=2)
    size = np.stack([mask.sum(1), (mask * np.abs(hat)).sum(1)], axis=2)
    within(o["records"], sums, size * (e + 68 * U * np.abs(g))[..., None], "sums")


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["inf", "nan", "far", "weight inf", "weight nan", "weight far", "class out", "gamma nan", "records inf"])
@pytest.mark.parametrize("N,classes,half", [(3, 10, True), (5, 100, False)])
def test_head_beyond_the_finite(N, classes, half, kind):
    t = head_inputs(N, classes, half, kind)
    o, one = head(t, N, classes, half), one_by_one(t, N, classes, half)
    same(o["out"], one["out"], "output")
    same(o["stats"], one["stats"], "mean, invstd")
    for k in HEAD_OUT[2:]:
        not_finite_alike(o[k], one[k], k)


SHAPES = [(32, 16), (16, 32)]


def stride2(N, H, C, kind="ordinary"):
    """(gradient, records, partial filter gradients) of the one kernel and, records aside, of the launches it replaces; the inputs."""
    g = np.random.default_rng(N + C)
    f = lambda *sh: g.standard_normal(sh).astype(np.float32)
    dy, w, sc, x, xc = f(N, H // 2, H // 2, 2 * C), 0.2 * f(3, 3, C, 2 * C), f(N, H // 2, H // 2, 2 * C), f(N, H, H, C), f(N, H, H, C)
    stats = np.concatenate([f(C), np.abs(f(C)) + 0.5])
    at = (0, 5, 3, 2)
    what, _, value = kind.rpartition(" ")
    if what:
        {"dy": dy, "shortcut": sc, "x": x, "xc": xc}.get(what, w)[at if what != "w" else (1, 2, 5, 7)] = float(value)
    t = {k: dev(v) for k, v in dict(dy=dy, w=w, sc=sc, x=x, xc=xc, stats=stats).items()}
    P, L, s, E, ch = {k: v.data_ptr() for k, v in t.items()}, B.lib(), stream_ptr(), 18 * C * C, ctypes.c_int(0)
    room = L.dsspk_conv_wgrad_scratch_floats(N, H, H, C, 2 * C, 3, 3, 2, 1) // E
    dx, rec, part = empty((N, H, H, C)), empty((L.dsspk_stride2_step_records(N, H, C), C, 2)), empty((room, E))
    assert L.dsspk_stride2_step_bwd(s, P["dy"], P["w"], P["sc"], dx.data_ptr(), part.data_ptr(), P["x"], P["xc"], P["stats"], rec.data_ptr(), N, H, C, ctypes.byref(ch)) == 0
    dx1, part1, ch1 = empty((N, H, H, C)), empty((room, E)), ctypes.c_int(0)
    assert L.dsspk_conv_bwd_data_shortcut(s, P["dy"], P["w"], P["sc"], dx1.data_ptr(), N, H, H, C, 2 * C, 3, 3, 1) == 0
    assert L.dsspk_conv_bwd_weight_parts(s, P["x"], P["dy"], part1.data_ptr(), N, H, H, C, 2 * C, 3, 3, 2, 1, None, 0, 0, None, None, None, ctypes.byref(ch1)) == 0
    assert ch.value == ch1.value <= room
    return dx, rec, part[:ch.value], torch.where(t["x"] > 0, dx1, torch.zeros_like(dx1)), part1[:ch.value], {k: f64(v) for k, v in t.items()}


def tiles(a, N, H, C):
    """Rows of a tensor in the order of the records: the four classes of pixels (h mod 2, w mod 2) one after the other, 64 of a class to a record."""
    return np.concatenate([a.reshape(N, H, H, C)[:, h::2, v::2].reshape(-1, 64, C) for h in (0, 1) for v in (0, 1)])


@pytest.mark.gpu
@pytest.mark.parametrize("N", [1, 2, 15, 16, 31, 32])
@pytest.mark.parametrize("H,C", SHAPES)
def test_stride2(N, H, C):
    """The gradients have the bits of the launches one by one; a record's sums of 64 terms are off by at most 64 roundings of their magnitudes (and xhat's
    own three)."""
    dx, rec, part, dx1, part1, t = stride2(N, H, C)
    same(dx, dx1, "gradient w.r.t. the input")
    same(part, part1, "partial filter gradients")
    d, hat = tiles(f64(dx), N, H, C), tiles((t["xc"] - t["stats"][:C]) * t["stats"][C:], N, H, C)
    want = np.stack([d.sum(1), (d * hat).sum(1)], axis=2)
    size = np.stack([np.abs(d).sum(1), np.abs(d * hat).sum(1)], axis=2)
    within(rec, want, 67 * U * size, "records")


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["%s %s" % (a, v) for a in ("dy", "w", "shortcut", "x") for v in ("inf", "nan", "3.395e38")] + ["x -inf", "xc inf", "xc nan"])
@pytest.mark.parametrize("H,C", SHAPES)
def test_stride2_beyond_the_finite(H, C, kind):
    """Also a masked element: an infinite or undefined gradient where the input is not positive is 0."""
    N = 3
    dx, rec, part, dx1, part1, t = stride2(N, H, C, kind)
    same(dx, dx1, "gradient w.r.t. the input")
    same(part, part1, "partial filter gradients")
    with np.errstate(all="ignore"):
        d = tiles(host(dx), N, H, C).astype(np.float64)
        hat = tiles(((t["xc"] - t["stats"][:C]) * t["stats"][C:]).astype(np.float32), N, H, C).astype(np.float64)
        want = np.stack([d.sum(1), (d * hat).sum(1)], axis=2)
        size = np.stack([np.abs(d).sum(1), np.abs(d * hat).sum(1)], axis=2)
    r = host(rec).astype(np.float64)
    ok = np.isfinite(want) & (size < 1e38)          # beyond that a sum may overflow on the way
    assert np.all(np.abs(r[ok] - want[ok]) <= 67 * U * size[ok])
    assert not np.isfinite(r[~np.isfinite(want)]).any()
