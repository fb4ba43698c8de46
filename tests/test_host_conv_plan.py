"""What the convolution calls answer before they launch anything, without a GPU."""
import ctypes
import os
import random
import shutil
import subprocess
import time

import pytest

import paper_2103_03936_amd as pf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2103_03936_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _desc(N, C, H, W, Cout, r, k, stride=1, dtype=pf.PF_F32):
    return pf.pf_conv_desc(N, C, H, W, Cout, r, k, stride, k // 2, pf.PF_NCHW, dtype, pf.PF_F32)


def _saved(*shape, **opt):
    return pf.lib.pf_lowrank_conv_saved_weights_bytes(ctypes.byref(_desc(*shape, **opt)))


@pytest.mark.parametrize("shape, el", [((88, 64, 13, 10, 64, 16, 1), 4), ((12, 96, 14, 14, 96, 24, 1), 4), ((128, 128, 16, 16, 256, 32, 1), 4),
                                       ((128, 128, 16, 16, 128, 32, 3), 2)])
def test_saved_filters_have_the_size_that_is_written(shape, el):
    """Where the pixel-major kernels take both directions the forward call keeps the thin filters for the backward one: every tap of
    every channel with the ranks padded to 32, in either type, in whole 256 bytes."""
    N, C, H, W, Cout, r, k = shape
    assert _saved(*shape, dtype=pf.PF_F32 if el == 4 else pf.PF_BF16) == (k * k * C * 32 * el + 255) // 256 * 256


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not found")
    out = str(tmp_path_factory.mktemp("emu") / "libconv_plan_host.so")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(PACKAGE, "csrc"),
           os.path.join(ROOT, "tests", "emulation", "conv_plan_host.cpp"), "-o", out, "-L" + PACKAGE, "-lpufferfish", "-Wl,-rpath," + PACKAGE]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE)
    return ctypes.CDLL(out)


def test_tiles_that_fit(emu):
    """The plan's answer (bounds, the tiles that stand for others) is that of every tile: no tile too large where it says yes, and the same yes
    for small planes, few images and planes whose tiles start everywhere; only a plane of odd size with few images may be refused where
    its tiles would just fit."""
    rng, refused, asked = random.Random(1), 0, 0
    planes = [(H, W) for H in range(1, 34, 2) for W in (1, 2, 3, 4, 7, 8, 13, 14, 16, 28, 31, 32, 33)]
    planes += [(56, 56), (112, 112), (49, 47), (97, 101), (101, 97), (120, 56), (56, 120), (225, 105), (105, 225), (64, 64), (60, 50), (301, 17)]
    for H, W in planes:
        for N in (1, 2, 5, 40, 300):
            for f32 in (0, 1):
                for k, st in ((1, 1), (3, 1), (1, 2), (3, 2)):
                    if ((H - 1) // st + 1) * ((W - 1) // st + 1) < (4 if f32 else 8):
                        continue
                    for P in (32, 64, 128):
                        r = emu.emu_fits(f32, N, H, W, k, st, P)
                        assert r & 1 <= r >> 1 & 1 and r >> 2 & 1 <= r >> 3 & 1, (H, W, N, f32, k, st, P)
                        refused += (r & 3 == 2) + (r & 12 == 8)
                        asked += 1
                        assert not (r & 3 == 2 or r & 12 == 8) or (N < P and N * H * W > 256 * P), (H, W, N, f32, k, st, P)
    assert refused <= asked // 1000, (refused, asked)


def test_arrays_within_32_bit_offsets(emu):
    """Every array that the kernels index is below 2^31 bytes, the re-ordered thin filters (ranks padded to 32) with it."""
    for f32, el in ((0, 2), (1, 4)):
        for k in (1, 3):
            most = (1 << 31) // (k * k * 32 * el) // 8 * 8  # channels whose filters fill that
            assert emu.emu_takes(f32, 1, most - 8, 2, 4, 8, 1, k) == 1
            for C in (most, most + 8):
                assert emu.emu_takes(f32, 1, C, 2, 4, 8, 1, k) == (k * k * C * 32 * el < 1 << 31), (f32, k, C)


def test_groups_of_the_filter_gradients(emu):
    """The bounded search finds what the search over every number of tiles does."""
    rng = random.Random(2)
    for _ in range(400):
        npx, k, f32 = int(2 ** rng.uniform(3, 19)), rng.choice([1, 3]), rng.random() < 0.3
        k = 1 if f32 else k
        C1, C2, r = rng.choice([8, 64, 72, 256, 512, 2048, 20000]), rng.choice([8, 64, 136, 512, 2048, 40000]), rng.randint(1, 32 if f32 else 128)
        out = (ctypes.c_int * 8)()
        emu.emu_wgrad_plan(int(f32), npx, r, C1, k, C2, out)
        assert list(out[:4]) == list(out[4:]), (f32, npx, r, C1, k, C2)


RESNET50 = [(256, 3, 56, 56, 64, 3, 1)] + [s for H, mid in ((56, 64), (28, 128), (14, 256), (7, 512)) for s in (
    (256, mid, H, H, mid, mid // 4, 3), (256, mid, H, H, 4 * mid, mid // 4, 1), (256, 4 * mid, H, H, mid, mid // 4, 1))]
RESNET50 += [s for H, mid in ((56, 128), (28, 256), (14, 512)) for s in ((256, mid, H, H, mid, mid // 4, 3, 2), (256, 2 * mid, H, H, 4 * mid, mid // 4, 1, 2),
                                                                        (256, 2 * mid, H, H, mid, mid // 4, 1))]


def _seconds(shape, dtype=pf.PF_BF16):
    d = _desc(*shape, dtype=dtype)
    t = time.perf_counter()
    pf.lib.pf_lowrank_conv_bwd_workspace_bytes(ctypes.byref(d))
    return time.perf_counter() - t


def test_time_of_a_plan():
    """A plan takes microseconds, and the layers of a model keep theirs.  (Times are of other batch sizes each, so that none is known;
    the median of nine, bounds some ten times what was measured.)"""
    _seconds((2, 8, 8, 8, 8, 4, 3))
    worst = {}
    for s in RESNET50 + [(64, 64, 112, 112, 64, 16, 3), (64, 16, 224, 224, 64, 4, 1), (64, 16, 225, 225, 64, 4, 1), (64, 48, 101, 97, 64, 16, 3)]:
        for dtype in (pf.PF_BF16, pf.PF_F32):
            worst[s, dtype] = sorted(_seconds((s[0] - i,) + s[1:], dtype) for i in range(9))[4]
    assert max(worst.values()) < 100e-6, max(worst, key=worst.get)
    rounds = [[_seconds(s) for s in RESNET50] for _ in range(6)][1:]
    assert max(min(t) for t in zip(*rounds)) < 10e-6


@pytest.mark.parametrize("shape", [(7, 816, 3, 3, 168, 14, 3), (2, 1040, 13, 10, 40, 18, 3), (3, 1024, 10, 10, 64, 16, 3), (1, 640, 8, 8, 128, 32, 3),
                                   (3, 576, 25, 4, 80, 20, 3)])
def test_few_tiles_with_many_channels_are_dealt_out(shape):
    """Shapes that the tiled products ran in half to four fifths of the time that the pixel-major kernels take: nothing is kept for those."""
    assert _saved(*shape, dtype=pf.PF_BF16) == 0


@pytest.mark.parametrize("shape", [(128, 128, 16, 16, 128, 32, 3), (256, 64, 32, 32, 64, 16, 3), (32, 256, 14, 14, 256, 64, 3)])
def test_layers_of_the_pixel_major_kernels(shape):
    """... and shapes that they run 1.3 to 2.9 times as fast in both directions."""
    assert _saved(*shape, dtype=pf.PF_BF16) > 0
