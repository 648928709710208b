"""What the library lays out and refuses before anything is launched; no GPU needed."""
import ctypes
import os
import re
import subprocess

import pytest

from paper_1908_11848_amd import binding as B, buildlib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("batch", [1, 37, 128, 512])
@pytest.mark.parametrize("model", ["alexnet_ds", "alexnet_3c"])
def test_alexnet_style_workspace_holds_what_the_step_uses(model, batch):
    """Activations, their gradients, converted filters and one buffer of partial sums for each convolution's filter gradient, sized by that
    convolution: every buffer begins on a 256-byte boundary (at most 40 of them), a few more hold 4 bytes to 2 KB."""
    L, m = B.lib(), batch
    a1, p1, p2 = m * 32 * 32 * 64, m * 15 * 15 * 64, m * 7 * 7 * 64
    wide = [(15, 5, 2)] + ([(7, 3, 1)] if model == "alexnet_3c" else [])
    rows = 384 * 2 if model == "alexnet_3c" else 384 * 2 + 192 * 2
    floats = a1 + 4 * p1 + (2 if model == "alexnet_ds" else 4) * p2 + rows * m + 21 * m       # two rows of 10 classes, one of losses
    floats += L.dsspk_conv_first_scratch_floats(m) + sum(L.dsspk_conv_split_wgrad_scratch_floats(m, H, H, 64, 64, k, p) for H, k, p in wide)
    nbytes = 4 * floats + p1 + p2 + sum(2 * L.dsspk_conv_split_filter_bytes(64, 64, k) for _, k, _ in wide)
    assert 0 <= B.dssp_workspace_bytes(B.model_id(model), batch, 10, 1) - nbytes < 40 * 256 + 4096


class Partials(ctypes.Structure):           # jobs::Partials
    _fields_ = [("partial", ctypes.c_void_p), ("dw", ctypes.c_void_p), ("E", ctypes.c_int), ("chunks", ctypes.c_int), ("quads", ctypes.c_bool)]


def test_a_step_reduces_no_more_filter_gradients_than_one_launch_holds():
    """The library's own reduction launcher, which the networks' steps call: it fills an array of DSSPK_WGRAD_REDUCE_MAX jobs."""
    text = open(os.path.join(ROOT, "include", "dssp_kernels.h")).read()
    most = int(re.search(r"#define DSSPK_WGRAD_REDUCE_MAX (\d+)", text).group(1))
    many = B.lib()._Z17wgrad_reduce_manyP12ihipStream_tiPKN4jobs8PartialsE
    many.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    jobs = (Partials * (most + 1))(*[Partials(4096, 4096, 4, 1, False)] * (most + 1))
    assert many(None, 0, jobs) == -1
    assert many(None, most + 1, jobs) == -1


def test_small_steps_ask_the_small_kernels_how_many_records_they_add_up():
    """A step leaves a stride-2 convolution's sums to the kernel behind as long as that one takes so many: the number is the kernels' own, one
    record more is refused (before anything is launched), and 16 images with 16 channels and 32 with 32 are what just fits."""
    L, p, q, r, n = B.lib(), 4096, 8192, 12288, None
    most, left = L._Z21conv3x3_small_recordsi, L._Z24conv_stride2_bwd_recordsiii
    for N, H, C in ((16, 32, 16), (32, 16, 32)):
        assert left(N, H, C) == most(C)
        assert L.dsspk_conv3x3_small_bwd(n, p, p, p, p, q, most(C) + 1, p, p, n, r, p, n, r, p, p, p, p, n, n, 0, 0, N, H, C) == -1
    assert left(17, 32, 16) > most(16) and left(33, 16, 32) == 0


def test_what_goes_between_source_files_is_one_type():
    """SplitFilterJob is passed by value from models.hip to k_conv_first.hip; its member type must be the same in both."""
    names = subprocess.run(["nm", "-C", buildlib.LIB], capture_output=True, text=True, check=True).stdout
    assert "SplitFilterJob" in names and "Frag" in names
    assert "(anonymous namespace)::Frag" not in names


def test_converted_filters_only_where_a_step_takes_them():
    """conv3x3_kernel<C, HW, R, NSPLIT, WAVES, TRANSPOSED, PRE, POST, WG, PL, REPEAT>: a step's backward pass takes d-input and d-filter from one kernel
    with 16 and 32 channels at every batch, and recomputes (REPEAT) only with converted filters (PL)."""
    names = subprocess.run(["nm", "-C", buildlib.LIB], capture_output=True, text=True, check=True).stdout
    forms = set(re.findall(r" void \(anonymous namespace\)::conv3x3_kernel<([^>]*)>", names))
    assert len(forms) > 60
    for form in forms:
        C, _, _, _, _, T, PRE, _, WG, PL, REPEAT = form.split(", ")
        assert PL == "false" or T == "false" or (PRE == "3" and (WG == "true" or C == "64")), form
        assert REPEAT == "false" or PL == "true" and T == "true", form


# pixels of LDS without padding: 400 bytes each, 160 KB a compute unit.  Two workgroups: 64 result pixels of a row and 3x3's halo, 3 x 66; 5x5's around
# two rows of 29 or 30, 6 x 33, 6 x 34; around a row of 36, 5 x 40; a 5x5 filter on a single row of 9, 5 x 3 x 13 (three images of 1x9).
@pytest.mark.parametrize("shape,resident", [((5, 64, 64, 64, 64, 3, 1), 2), ((18, 29, 29, 64, 64, 5, 2), 2), ((20, 30, 30, 64, 64, 5, 2), 2),
                                            ((10, 36, 36, 64, 64, 5, 2), 2), ((8, 1, 9, 64, 64, 5, 2), 2), ((37, 15, 15, 64, 64, 5, 2), 2),
                                            ((128, 15, 15, 64, 64, 5, 2), 1), ((6, 64, 64, 64, 64, 3, 1), 1), ((1, 8, 200, 64, 64, 3, 1), 0)])
def test_wide_tiles_are_not_padded_out_of_a_compute_unit(shape, resident):
    assert B.lib().dsspk_conv_split_resident(*shape) == resident
