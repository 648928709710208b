"""The 3x3 / stride 1 convolutions of the residual networks (fp32 arithmetic on the bf16 matrix cores, leading and small
products summed apart) against the oracle's direct loops in float64.

Tolerance: the sum of the leading products is rounded once per instruction, 9 C / 32 (at least 9) times, each time by up to
6e-8 of the running sum, which is below the final one for most of the way; errors of random sign add up to
sqrt(9 .. 18) * 6e-8 * 0.6 = 1.1e-7 .. 1.6e-7 of the result.  Bound 2e-7 (measured at most 1.2e-7; the fp32 matrix-core
form of the same convolution shows up to 2.1e-7)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr     # noqa: E402


@pytest.mark.parametrize("N,H,C", [(1, 32, 16), (7, 32, 16), (1, 16, 32), (5, 16, 32), (1, 8, 64), (9, 8, 64)])
@pytest.mark.parametrize("offset", [0.0, 8.0])
def test_error_of_forward_and_input_gradient(oracle_nn, N, H, C, offset):
    g = np.random.default_rng(100 * N + C)
    x = (offset + g.standard_normal((N, H, H, C))).astype(np.float32)
    w = (np.sqrt(2.0 / (9 * C)) * g.standard_normal((3, 3, C, C))).astype(np.float32)
    dy = (1e-3 * g.standard_normal((N, H, H, C))).astype(np.float32)
    X, W, DY, y, dx = dev(x), dev(w), dev(dy), empty((N, H, H, C)), empty((N, H, H, C))
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_conv_fwd(s, X.data_ptr(), W.data_ptr(), None, y.data_ptr(), N, H, H, C, C, 3, 3, 1, 1, 0, None) == 0
    assert L.dsspk_conv_bwd_data(s, DY.data_ptr(), W.data_ptr(), None, dx.data_ptr(), N, H, H, C, C, 3, 3, 1, 1) == 0
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    yo = oracle_nn.conv2d_fwd(x64, w64, None, 1, 1)
    dxo, _, _ = oracle_nn.conv2d_bwd(x64, w64, dy64, 1, 1, True)
    assert rel_l2(host(y), yo) < 2e-7 and max_abs(host(y), yo) < 2e-6
    assert rel_l2(host(dx), dxo) < 2e-7 and max_abs(host(dx), dxo) < 2e-6
