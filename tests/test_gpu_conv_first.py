"""First layer of the AlexNet-style networks (convolution, bias, ReLU and max-pool in one pass; filter and bias gradients from the
pooled gradient) against the oracle's layers in float64.

Tolerance: 75 products per output (leading products rounded five times, below 1.5e-7 of the result); the gradients sum up to
N * 1024 of them, most of them zero, sqrt(count) * 6e-8 against sqrt(count).  2e-6 / 2e-5 as for the other convolution kernels.
Pooling decisions are taken on the kernel's own activations, so they are checked on those, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr     # noqa: E402
import torch                                                 # noqa: E402


# one image, several, more bands than one round of workgroups takes (two and three bands each, the last chunk not full)
@pytest.mark.parametrize("N", [1, 3, 37, 128, 130, 300])
@pytest.mark.parametrize("offset", [0.0, 4.0])
def test_conv_first(oracle_nn, N, offset):
    if offset and N > 128:
        pytest.skip("the offset is about sums within an output")
    g = np.random.default_rng(N)
    x = (offset + g.standard_normal((N, 32, 32, 3))).astype(np.float32)
    w = (np.sqrt(2.0 / 75) * g.standard_normal((5, 5, 3, 64))).astype(np.float32)
    b = g.standard_normal(64).astype(np.float32)
    dp = (1e-2 * g.standard_normal((N, 15, 15, 64))).astype(np.float32)
    X, W, Bd, DP = dev(x), dev(w), dev(b), dev(dp)
    a, p, arg = empty((N, 32, 32, 64)), empty((N, 15, 15, 64)), torch.empty(N * 225 * 64, dtype=torch.uint8, device="cuda")
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_conv_first_pool_fwd(s, X.data_ptr(), W.data_ptr(), Bd.data_ptr(), a.data_ptr(), p.data_ptr(), arg.data_ptr(), N) == 0
    x64, w64 = x.astype(np.float64), w.astype(np.float64)
    ao = np.maximum(oracle_nn.conv2d_fwd(x64, w64, b.astype(np.float64), 1, 2), 0)
    got = host(a)
    assert rel_l2(got, ao) < 2e-7 and max_abs(got, ao) < 2e-6
    # pooling: that of the stand-alone kernels on these activations
    p1, arg1 = empty((N, 15, 15, 64)), torch.empty_like(arg)
    assert L.dsspk_maxpool_fwd(s, a.data_ptr(), p1.data_ptr(), arg1.data_ptr(), N, 32, 32, 64) == 0
    assert np.array_equal(host(p), host(p1)) and np.array_equal(arg.cpu().numpy(), arg1.cpu().numpy())
    # gradients: those of the stand-alone pooling backward pass, in float64 from there
    da = empty((N, 32, 32, 64))
    assert L.dsspk_maxpool_bwd_relu(s, DP.data_ptr(), arg.data_ptr(), a.data_ptr(), da.data_ptr(), N, 32, 32, 64) == 0
    da64 = host(da).astype(np.float64).reshape(N, 32, 32, 64)
    _, dwo, dbo = oracle_nn.conv2d_bwd(x64, w64, da64, 1, 2, True, need_dx=False)
    dw, scr = empty(4864), empty(L.dsspk_conv_first_scratch_floats(N))
    assert L.dsspk_conv_first_pool_bwd_weight(s, X.data_ptr(), DP.data_ptr(), p.data_ptr(), arg.data_ptr(), dw.data_ptr(), scr.data_ptr(), N) == 0
    out = host(dw)
    assert rel_l2(out[:4800], dwo) < 2e-6 and max_abs(out[:4800], dwo) < 2e-5
    assert np.max(np.abs(out[4800:] - dbo)) < 2e-6 * 1e-2 * max(1.0, np.sqrt(N * 225)) * 4


@pytest.mark.parametrize("N", [1, 37, 128, 300])
def test_error_no_larger_than_the_fp32_matrix_cores(oracle_nn, N):
    """Output and filter gradient against the general kernels' (implicit matrix product on the fp32 cores) on the same operands."""
    g = np.random.default_rng(N)
    x, b = g.standard_normal((N, 32, 32, 3)).astype(np.float32), g.standard_normal(64).astype(np.float32)
    w = (np.sqrt(2.0 / 75) * g.standard_normal((5, 5, 3, 64))).astype(np.float32)
    dp = (1e-3 * g.standard_normal((N, 15, 15, 64))).astype(np.float32)
    X, W, Bd, DP = dev(x), dev(w), dev(b), dev(dp)
    a, a32, p, arg, da = empty((N, 32, 32, 64)), empty((N, 32, 32, 64)), empty((N, 15, 15, 64)), torch.empty(N * 225 * 64, dtype=torch.uint8, device="cuda"), empty((N, 32, 32, 64))
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_conv_first_pool_fwd(s, X.data_ptr(), W.data_ptr(), Bd.data_ptr(), a.data_ptr(), p.data_ptr(), arg.data_ptr(), N) == 0
    general = (N, 32, 32, 3, 64, 5, 5, 1, 2)
    assert L.dsspk_conv_fwd(s, X.data_ptr(), W.data_ptr(), Bd.data_ptr(), a32.data_ptr(), *general, 1, None) == 0
    assert L.dsspk_maxpool_bwd_relu(s, DP.data_ptr(), arg.data_ptr(), a.data_ptr(), da.data_ptr(), N, 32, 32, 64) == 0
    dw, dw32 = empty(4864), empty(4800)
    scr, scr32 = empty(L.dsspk_conv_first_scratch_floats(N)), empty(L.dsspk_conv_wgrad_scratch_floats(*general))
    assert L.dsspk_conv_first_pool_bwd_weight(s, X.data_ptr(), DP.data_ptr(), p.data_ptr(), arg.data_ptr(), dw.data_ptr(), scr.data_ptr(), N) == 0
    assert L.dsspk_conv_bwd_weight(s, X.data_ptr(), da.data_ptr(), dw32.data_ptr(), scr32.data_ptr(), *general) == 0
    x64, w64 = x.astype(np.float64), w.astype(np.float64)
    ao = np.maximum(oracle_nn.conv2d_fwd(x64, w64, b.astype(np.float64), 1, 2), 0)
    _, dwo, _ = oracle_nn.conv2d_bwd(x64, w64, host(da).astype(np.float64).reshape(N, 32, 32, 64), 1, 2, True, need_dx=False)
    for got, got32, want in ((host(a), host(a32), ao), (host(dw)[:4800], host(dw32), dwo)):
        split, fp32 = rel_l2(got, want), rel_l2(got32, want)
        assert split <= fp32, (split, fp32)
