"""What the convolution calls answer before they launch anything, without a GPU."""
import ctypes

import pytest

import paper_2103_03936_amd as pf


def _desc(N, C, H, W, Cout, r, k, stride=1, dtype=pf.PF_F32):
    return pf.pf_conv_desc(N, C, H, W, Cout, r, k, stride, k // 2, pf.PF_NCHW, dtype, pf.PF_F32)


def _saved(*shape, **opt):
    return pf.lib.pf_lowrank_conv_saved_weights_bytes(ctypes.byref(_desc(*shape, **opt)))


@pytest.mark.parametrize("shape, el", [((226, 64, 14, 14, 64, 16, 1), 4), ((12, 96, 14, 14, 96, 24, 1), 4), ((128, 128, 16, 16, 256, 32, 1), 4),
                                       ((128, 128, 16, 16, 128, 32, 3), 2)])
def test_saved_filters_have_the_size_that_is_written(shape, el):
    """Where the pixel-major kernels take both directions the forward call keeps the thin filters for the backward one: every tap of
    every channel with the ranks padded to 32, in either type, in whole 256 bytes."""
    N, C, H, W, Cout, r, k = shape
    assert _saved(*shape, dtype=pf.PF_F32 if el == 4 else pf.PF_BF16) == (k * k * C * 32 * el + 255) // 256 * 256
