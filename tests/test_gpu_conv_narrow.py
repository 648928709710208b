"""Generic convolutions whose grid leaves half the chip idle: channel tiles narrower than the layer, several k-chunks to a stage.  Forward and
d-input against the oracle's loops in float64, at one tile of rows (16 channels wide), at 64 to 127 of them (32 wide), with ragged last tiles, and
every number of reduction channels that chooses another stage.  Tolerance as for the other generic convolutions: fp32 sums of at most 1152
products, 2e-6 / 2e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr     # noqa: E402

# N, H, Cin, Cout, stride
CASES = [(N, H, C, 64, stride) for N, H, stride in ((1, 9, 1), (1, 16, 2), (17, 32, 2)) for C in (16, 32, 128)] + [(19, 16, 16, 64, 1), (5, 16, 32, 32, 2)]
CASES += [(N, H, 64, C, stride) for N, H, stride, C in ((1, 9, 1, 16), (1, 16, 2, 32), (3, 16, 2, 128), (17, 16, 1, 32), (20, 16, 2, 128), (20, 16, 2, 16))]


@pytest.mark.parametrize("N,H,Cin,Cout,stride", CASES)
def test_forward_and_d_input(oracle_nn, N, H, Cin, Cout, stride):
    g = np.random.default_rng(N * 100 + H + Cin)
    x = g.standard_normal((N, H, H, Cin)).astype(np.float32)
    w = (np.sqrt(2.0 / (9 * Cin)) * g.standard_normal((3, 3, Cin, Cout))).astype(np.float32)
    OH = (H - 1) // stride + 1
    dy = g.standard_normal((N, OH, OH, Cout)).astype(np.float32)
    L, s = B.lib(), stream_ptr()
    X, W, DY, y, dx = dev(x), dev(w), dev(dy), empty((N, OH, OH, Cout)), empty((N, H, H, Cin))
    assert L.dsspk_conv_fwd(s, X.data_ptr(), W.data_ptr(), None, y.data_ptr(), N, H, H, Cin, Cout, 3, 3, stride, 1, 0, None) == 0
    assert L.dsspk_conv_bwd_data(s, DY.data_ptr(), W.data_ptr(), None, dx.data_ptr(), N, H, H, Cin, Cout, 3, 3, stride, 1) == 0
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    dxo, _, _ = oracle_nn.conv2d_bwd(x64, w64, dy64, stride, 1, True)
    for got, want in ((host(y), oracle_nn.conv2d_fwd(x64, w64, None, stride, 1)), (host(dx), dxo)):
        assert rel_l2(got, want) < 2e-6 and max_abs(got, want) < 2e-5 * max(1.0, np.abs(want).max() / 4)
