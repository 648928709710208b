"""Fully connected layers: the products that split their reduction over the wavefronts of a workgroup, the backward pass of a
layer in one launch, and the last layer with its softmax cross-entropy, against the oracle's layer functions.

Tolerances: fp32 accumulation of K products of O(1) terms is off by about sqrt(K) * 6e-8 relative to the sum's scale (3.4e-6
at K = 3136, measured 5e-7); 2e-6 relative L2 and 2e-5 of the largest entry hold for every case, as for the other kernels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1908_11848_amd import binding as B               # noqa: E402
from gpu_util import dev, empty, host, max_abs, rel_l2, stream_ptr     # noqa: E402


def close(got, want):
    got = host(got)
    assert np.isfinite(got).all()
    assert rel_l2(got, want) < 2e-6 and max_abs(got, want) < 2e-5


# (m, n_in, n_out): one sample; edges of the 16-, 32- and 64-wide tiles; K around the 16-wide chunks and not a multiple of 4;
# shapes on both sides of the tile-shape rule
SHAPES = [(1, 1, 1), (1, 3072, 256), (15, 17, 18), (16, 16, 16), (17, 33, 65), (33, 50, 7), (37, 3136, 384), (64, 500, 130),
          (128, 192, 100), (130, 1030, 34), (512, 384, 192), (512, 3136, 384), (1000, 64, 10)]


@pytest.mark.parametrize("m,n_in,n_out", SHAPES)
def test_fc_backward_in_one_launch(oracle_nn, m, n_in, n_out):
    g = np.random.default_rng(m + 7 * n_in + 131 * n_out)
    x = np.maximum(g.standard_normal((m, n_in)), 0).astype(np.float32)
    w = (0.1 * g.standard_normal((n_in, n_out))).astype(np.float32)
    dy = g.standard_normal((m, n_out)).astype(np.float32)
    rl = g.standard_normal(m).astype(np.float32)
    X, W, DY, RL = dev(x), dev(w), dev(dy), dev(rl)
    dxo, dwo, dbo = oracle_nn.fc_bwd(x.astype(np.float64), w.astype(np.float64), dy.astype(np.float64))
    L, s = B.lib(), stream_ptr()
    for mask in (0, 1):
        dx, dw, db, loss = empty((m, n_in)), empty((n_in, n_out)), empty(n_out), empty(1)
        assert L.dsspk_fc_bwd(s, X.data_ptr(), DY.data_ptr(), W.data_ptr(), dw.data_ptr(), db.data_ptr(), dx.data_ptr(), mask,
                              RL.data_ptr(), loss.data_ptr(), m, n_in, n_out) == 0
        close(dx, dxo * (x > 0) if mask else dxo)
        close(dw, dwo)
        close(db, dbo)
        assert abs(host(loss)[0] - rl.astype(np.float64).mean()) < 1e-6
    dw, db = empty((n_in, n_out)), empty(n_out)              # without dx and loss: the other outputs alone
    assert L.dsspk_fc_bwd(s, X.data_ptr(), DY.data_ptr(), None, dw.data_ptr(), db.data_ptr(), None, 0, None, None, m, n_in, n_out) == 0
    close(dw, dwo)
    close(db, dbo)
    assert L.dsspk_fc_bwd(s, X.data_ptr(), DY.data_ptr(), None, dw.data_ptr(), db.data_ptr(), dx.data_ptr(), 0, None, None, m, n_in, n_out) == -1


@pytest.mark.parametrize("m,n_in,n_out", SHAPES)
def test_fc_forward_shapes(oracle_nn, m, n_in, n_out):
    g = np.random.default_rng(m + 3 * n_in + 17 * n_out)
    x, w, b = (g.standard_normal(s).astype(np.float32) for s in ((m, n_in), (n_in, n_out), (n_out,)))
    y = empty((m, n_out))
    X, W, Bv = dev(x), dev(w), dev(b)
    assert B.lib().dsspk_gemm(stream_ptr(), X.data_ptr(), n_in, 1, W.data_ptr(), n_out, 1, y.data_ptr(), n_out, m, n_out, n_in,
                              Bv.data_ptr(), 1) == 0
    close(y, np.maximum(oracle_nn.fc_fwd(x.astype(np.float64), w.astype(np.float64), b.astype(np.float64)), 0))


@pytest.mark.parametrize("m,n_in,C", [(1, 256, 2), (7, 30, 3), (16, 64, 16), (17, 192, 17), (32, 256, 10), (128, 64, 100), (130, 384, 128)])
def test_last_layer_with_softmax(oracle_nn, m, n_in, C):
    g = np.random.default_rng(m * 3 + C)
    x, b = g.standard_normal((m, n_in)).astype(np.float32), g.standard_normal(C).astype(np.float32)
    w = (g.standard_normal((n_in, C)) / np.sqrt(n_in) * 4).astype(np.float32)
    lab = g.integers(0, C, m).astype(np.int32)
    X, W, Bv, Y = dev(x), dev(w), dev(b), dev(lab)
    z, dz, rl = empty((m, C)), empty((m, C)), empty(m)
    L, s = B.lib(), stream_ptr()
    assert L.dsspk_fc_softmax_xent(s, X.data_ptr(), W.data_ptr(), Bv.data_ptr(), Y.data_ptr(), z.data_ptr(), dz.data_ptr(),
                                   rl.data_ptr(), m, n_in, C) == 0
    zo = oracle_nn.fc_fwd(x.astype(np.float64), w.astype(np.float64), b.astype(np.float64))
    close(z, zo)
    lo, dzo = oracle_nn.softmax_xent(zo, lab)
    assert abs(host(rl).astype(np.float64).mean() - lo) < 2e-6 * max(1, abs(lo))
    # an error of 2e-6 in a logit moves a probability by at most that much, relatively; ten times that for the sum of C of them
    assert rel_l2(host(dz), dzo) < 1e-5 and max_abs(host(dz), dzo) < 2e-5
    assert L.dsspk_fc_softmax_xent(s, X.data_ptr(), W.data_ptr(), Bv.data_ptr(), Y.data_ptr(), z.data_ptr(), dz.data_ptr(),
                                   rl.data_ptr(), m, n_in, 129) == -1


# both sides of the line from which a product takes its operands through LDS (1024 tiles of 64x64), remainders in every direction, every
# order of the operands, a row pitch of the result
@pytest.mark.parametrize("M,N,K", [(1985, 2000, 70), (2050, 2000, 70), (65500, 33, 17), (64, 65473, 1), (2048, 2048, 129)])
@pytest.mark.parametrize("a_rows,b_rows", [(True, True), (False, True), (True, False), (False, False)])
def test_gemm_large(M, N, K, a_rows, b_rows):
    g = np.random.default_rng(M + K)
    a, b, bias = (g.standard_normal(sh).astype(np.float32) for sh in ((M, K), (K, N), (N,)))
    A, Bm, Bv = dev(a if a_rows else a.T), dev(b if b_rows else b.T), dev(bias)
    ldc = N + 3
    C = empty((M, ldc))
    assert B.lib().dsspk_gemm(stream_ptr(), A.data_ptr(), *((K, 1) if a_rows else (1, M)), Bm.data_ptr(), *((N, 1) if b_rows else (1, K)), C.data_ptr(),
                              ldc, M, N, K, Bv.data_ptr(), 1) == 0
    got, want = host(C), np.maximum(a.astype(np.float64) @ b.astype(np.float64) + bias, 0)
    assert np.isnan(got[:, N:]).all()                   # the pitch's gap is left alone
    assert rel_l2(got[:, :N], want) < 1e-6 and max_abs(got[:, :N], want) < 1e-5         # sqrt(K) * 6e-8 of the sum's scale
