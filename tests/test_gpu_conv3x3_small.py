"""The 3x3 kernels with two pixel tiles to a wavefront (dsspk_conv3x3_small_*): what test_gpu_conv3x3_large.py holds the larger workgroups to,
at one image, a few, an odd number of records and the largest batch they cover."""
import pytest

import test_gpu_conv3x3_large as large
from paper_1908_11848_amd import binding as B

SIZES = [(N, H, C) for N in (1, 3, 13, 32) for H, C in large.SHAPES]


def test_what_is_covered():
    L = B.lib()
    for (H, C), per_image in zip(large.SHAPES, (8, 4, 1)):
        assert [L.dsspk_conv3x3_small_parts(N, H, C) for N in (0, 1, 32, 33)] == [0, per_image, 32 * per_image, 0]
        assert L.dsspk_conv3x3_small_parts(4, H + 1, C) == 0 and L.dsspk_conv3x3_small_parts(4, H, C + 16) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,C", SIZES)
@pytest.mark.parametrize("form", ["plain", "bn", "bn+shortcut"])
def test_forward(oracle_nn, N, H, C, form):
    large.forward(oracle_nn, "small", N, H, C, form)


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,C", SIZES)
@pytest.mark.parametrize("big", [False, True])
def test_backward(N, H, C, big):
    large.backward("small", N, H, C, big)
