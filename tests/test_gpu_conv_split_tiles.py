"""Wide convolutions with more tiles of the largest kind than compute units (a workgroup walks several tiles): forward and d-input against the
oracle's loops in float64, where the number of workgroups is odd, the last tile or workgroup is partly filled, several images share a tile, and the
channels come in several blocks.  Tolerances as in test_gpu_conv_split.py, relative to the result's largest value; with an operand
beyond the range of the scaled terms its tile is computed in fp32."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr     # noqa: E402

# N, H, W, Cin, Cout, k, pad
CASES = [(129, 15, 15, 64, 64, 5, 2), (515, 7, 7, 64, 64, 3, 1), (140, 9, 14, 128, 128, 3, 1), (260, 3, 40, 64, 64, 3, 1)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("large", [False, True])
def test_walked_tiles(oracle_nn, case, large):
    N, H, W, Cin, Cout, k, pad = case
    g = np.random.default_rng(N + H)
    x = g.standard_normal((N, H, W, Cin)).astype(np.float32)
    w = (np.sqrt(2.0 / (k * k * Cin)) * g.standard_normal((k, k, Cin, Cout))).astype(np.float32)
    b = g.standard_normal(Cout).astype(np.float32)
    OH, OW = H + 2 * pad - k + 1, W + 2 * pad - k + 1
    dy = g.standard_normal((N, OH, OW, Cout)).astype(np.float32)
    add = g.standard_normal((N, H, W, Cin)).astype(np.float32)
    if large:
        x[N - 1, 1, 2, 3], dy[N // 2, 0, 0, 1] = 3e31, 2e32
    L, s = B.lib(), stream_ptr()
    X, Wd, Bd, DY, ADD = dev(x), dev(w), dev(b), dev(dy), dev(add)
    n_planes = L.dsspk_conv_split_filter_bytes(Cin, Cout, k) // 4
    pf, pb = empty(n_planes), empty(n_planes)
    assert L.dsspk_conv_split_filters(s, Wd.data_ptr(), pf.data_ptr(), pb.data_ptr(), Cin, Cout, k) == 0
    y, dx = empty((N, OH, OW, Cout)), empty((N, H, W, Cin))
    assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), Bd.data_ptr(), y.data_ptr(), N, H, W, Cin, Cout, k, pad, 1) == 0
    assert L.dsspk_conv_split_bwd_data(s, DY.data_ptr(), pb.data_ptr(), ADD.data_ptr(), dx.data_ptr(), N, H, W, Cin, Cout, k, pad) == 0
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    dxo, _, _ = oracle_nn.conv2d_bwd(x64, w64, dy64, 1, pad, True)
    yo = np.maximum(oracle_nn.conv2d_fwd(x64, w64, b.astype(np.float64), 1, pad), 0)
    for got, want in ((host(y), yo), (host(dx), dxo + add.astype(np.float64))):
        assert rel_l2(got, want) < 2e-6 and max_abs(got, want) < 2e-5 * max(1.0, np.abs(want).max() / 4)
        ordinary = np.abs(want) < 1e6           # where the large operand does not reach
        assert rel_l2(got[ordinary], want[ordinary]) < 2e-6


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("kind", ["relu", "offset"])
def test_no_less_exact_than_on_the_fp32_cores(oracle_nn, case, kind):
    """Forward against the implicit GEMM on the fp32 matrix cores, both against float64 (measured: 2.2e-7 to 3.9e-7 against 2.8e-7 to 6.8e-7)."""
    N, H, W, Cin, Cout, k, pad = case
    g = np.random.default_rng(N + H)
    x = g.standard_normal((N, H, W, Cin))
    x = (np.maximum(x, 0) if kind == "relu" else x + 4).astype(np.float32)
    w = (np.sqrt(2.0 / (k * k * Cin)) * g.standard_normal((k, k, Cin, Cout))).astype(np.float32)
    OH, OW = H + 2 * pad - k + 1, W + 2 * pad - k + 1
    L, s = B.lib(), stream_ptr()
    X, Wd, y, y32, pf = dev(x), dev(w), empty((N, OH, OW, Cout)), empty((N, OH, OW, Cout)), empty(L.dsspk_conv_split_filter_bytes(Cin, Cout, k) // 4)
    pb = empty(pf.shape)
    assert L.dsspk_conv_split_filters(s, Wd.data_ptr(), pf.data_ptr(), pb.data_ptr(), Cin, Cout, k) == 0
    assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), None, y.data_ptr(), N, H, W, Cin, Cout, k, pad, 0) == 0
    assert L.dsspk_conv_fwd(s, X.data_ptr(), Wd.data_ptr(), None, y32.data_ptr(), N, H, W, Cin, Cout, k, k, 1, pad, 0, None) == 0
    want = oracle_nn.conv2d_fwd(x.astype(np.float64), w.astype(np.float64), None, 1, pad)
    split, fp32 = rel_l2(host(y), want), rel_l2(host(y32), want)
    assert split <= fp32, (split, fp32)
