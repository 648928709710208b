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
