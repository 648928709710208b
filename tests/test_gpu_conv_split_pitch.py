"""Wide convolutions where the LDS layout of their tile changes: rows too long for padding (5x5 on 61 to 64 columns, the widest there are), groups of tiny
images of which padding would admit fewer, rows shorter and longer than the 16 pixels of a matrix-core tile, and walked tiles of several images.
Against the oracle's loops in float64; tolerances as in test_gpu_conv_split.py (an fp32 accumulation of K <= 1600 products)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr     # noqa: E402

# N, H, W, k, pad
CASES = [(1, 4, 64, 5, 2), (100, 2, 63, 5, 2), (97, 5, 61, 5, 2), (130, 3, 64, 3, 1), (31, 2, 2, 3, 1), (27, 1, 3, 5, 2), (3, 11, 13, 5, 2), (2, 5, 31, 3, 1),
         (1030, 5, 5, 3, 1), (300, 13, 1, 3, 1)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_tile_layouts(oracle_nn, case):
    N, H, W, k, pad = case
    C = 64
    g = np.random.default_rng(N + 7 * W)
    x = g.standard_normal((N, H, W, C)).astype(np.float32)
    w = (0.05 * g.standard_normal((k, k, C, C))).astype(np.float32)
    dy = g.standard_normal((N, H, W, C)).astype(np.float32)
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_conv_split_covers(N, H, W, C, C, k, pad) == 1
    X, Wd, DY = dev(x), dev(w), dev(dy)
    planes = L.dsspk_conv_split_filter_bytes(C, C, k) // 4
    pf, pb, y, dx = empty(planes), empty(planes), empty((N, H, W, C)), empty((N, H, W, C))
    assert L.dsspk_conv_split_filters(s, Wd.data_ptr(), pf.data_ptr(), pb.data_ptr(), C, C, k) == 0
    assert L.dsspk_conv_split_fwd(s, X.data_ptr(), pf.data_ptr(), None, y.data_ptr(), N, H, W, C, C, k, pad, 0) == 0
    assert L.dsspk_conv_split_bwd_data(s, DY.data_ptr(), pb.data_ptr(), None, dx.data_ptr(), N, H, W, C, C, k, pad) == 0
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    dxo, _, _ = oracle_nn.conv2d_bwd(x64, w64, dy64, 1, pad, False)
    for got, want in ((host(y), oracle_nn.conv2d_fwd(x64, w64, None, 1, pad)), (host(dx), dxo)):
        assert rel_l2(got, want) < 2e-6 and max_abs(got, want) < 2e-5
