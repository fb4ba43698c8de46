"""Where the pixel-major convolution kernels find their pixels (pf_conv_px_index.h), without a GPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not found")
    out = str(tmp_path_factory.mktemp("emu") / "libconv_px_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "paper_2103_03936_amd", "csrc"),
                    os.path.join(ROOT, "tests", "emulation", "conv_px_host.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("S", [2, 3])
@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("P", [32, 64, 128])
def test_tiles(emu, S, k, P):
    """Every tap of every pixel of every tile is the pixel it should be, or a slot that nothing is stored to; loads stay in their planes."""
    for H, W, N in [(4, 4, 40), (8, 8, 5), (7, 7, 11), (16, 16, 2), (32, 32, 1), (5, 5, 40), (4, 32, 3), (32, 4, 3), (31, 29, 2), (2, 4, 9),
                    (13, 17, 3), (10, 10, 7), (9, 1, 30), (14, 14, 3), (3, 11, 9), (1, 8, 40)]:
        assert emu.emu_px(S, N, H, W, k, 1, P, 100000, 100000) == 0, (H, W, N)
        for stride in (2, 3):
            if ((H - 1) // stride + 1) * ((W - 1) // stride + 1) >= 1 << S:
                assert emu.emu_px(S, N, H, W, k, stride, P, 100000, 100000) == 0, (H, W, N, stride)


@pytest.mark.parametrize("S,groups", [(2, 64), (3, 32)])
@pytest.mark.parametrize("P,rows", [(32, 160), (64, 192), (128, 256)])
def test_common_planes_fit(emu, P, rows, S, groups):
    """Planes of 4 x 4 to 32 x 32 pixels fit the LDS that a tile has."""
    for H in range(4, 33):
        for W in {4, 5, 7, 8, H, 32}:
            assert emu.emu_px(S, max(2, 300 // (H * W)), H, W, 3, 1, P, rows, groups if P > 32 else groups // 2) == 0, (H, W)
            if P == 32 and H >= 8 and W >= 8: # with stride
                assert emu.emu_px(S, max(2, 600 // (H * W)), H, W, 3, 2, P, 256, groups) == 0, (H, W)


def test_banks(emu):
    assert max(emu.emu_px_banks(s, 1, o) for s in range(64) for o in range(8)) <= 2   # fragments of eight neighbouring slots
    assert max(emu.emu_px_banks(s, 8, o) for s in range(64) for o in range(8)) <= 2   # stores of groups of eight
