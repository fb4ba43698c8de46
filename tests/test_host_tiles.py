"""The host side of the tiled products without a GPU (tests/emulation/tile_host.cpp, linked against the library)."""
import ctypes
import os
import shutil
import subprocess

import pytest
import torch  # noqa: F401  (its HIP runtime is the one that the library uses)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2103_03936_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
F32, BF16 = 0, 1
TS_32, TS_64, TS_128x64, TS_128, TS_32x64, TS_32x128, TS_32D = range(7)
UNSUPPORTED = 3


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not found")
    import paper_2103_03936_amd  # noqa: F401  (the library is built)
    out = str(tmp_path_factory.mktemp("emu") / "libtile_host.so")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(PACKAGE, "csrc"),
           os.path.join(ROOT, "tests", "emulation", "tile_host.cpp"), "-o", out, "-L" + PACKAGE, "-lpufferfish", "-Wl,-rpath," + PACKAGE]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE)
    return ctypes.CDLL(out)


@pytest.mark.skipif(torch.cuda.is_available(), reason="asks for launches without operands: only where none can take place")
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("shape", [TS_32x64, TS_128x64])
def test_paired_pixels_have_one_tile_shape(emu, dtype, shape):
    """The kernel that stores even and odd pixels together deals 64 x 64 tiles to its threads; other shapes are refused before a launch."""
    assert emu.emu_pair(dtype, shape, TS_64) == UNSUPPORTED


def _plan(emu, dtype, M, N, K):
    split = ctypes.c_int()
    i64 = ctypes.c_longlong
    return emu.emu_plan(dtype, i64(M), i64(N), i64(K), 16, ctypes.byref(split)), split.value


def _gradients(emu, dtype, M, n_in, n_out, r):
    split = (ctypes.c_int * 3)()
    i64 = ctypes.c_longlong
    return emu.emu_gradients(dtype, i64(M), i64(n_in), i64(n_out), i64(r), split), list(split)


def test_plans_that_the_gpu_tests_count_on(emu):
    """Shapes of test_gpu_tiles.LINEAR that stand for a tile shape reach it: 32 x 32 by eight wavefronts with and without a split, also for
    gradients, and 128 x 128 gradients."""
    for dtype in (F32, BF16):
        assert _plan(emu, dtype, 96, 218, 4093) == (TS_32D, 8)
    assert _plan(emu, F32, 282, 86, 3492) == (TS_32D, 7)
    assert _plan(emu, F32, 160, 37, 260) == _plan(emu, BF16, 160, 37, 517) == (TS_32D, 1)
    assert _gradients(emu, F32, 300, 256, 256, 250)[0] == _gradients(emu, BF16, 515, 160, 150, 514)[0] == TS_32D
    shape, split = _gradients(emu, BF16, 6500, 489, 985, 128)
    assert shape == TS_128 and split[1] == split[2] > 1


@pytest.mark.parametrize("M,n_in,n_out", [(10183, 576, 1344), (7740, 832, 176), (7474, 784, 738), (6337, 484, 1030), (6337, 500, 264)])
def test_padded_gradients_stay_on_smaller_tiles(emu, M, n_in, n_out):
    """128 x 128 tiles, of which padding took more than a seventeenth, were the slower ones (the first 47.5 -> 56.8 us)."""
    assert _gradients(emu, BF16, M, n_in, n_out, 128)[0] == TS_64


@pytest.mark.parametrize("dtype,shape,forward,backward", [
    (F32, (1, 1030, 517, 97), 4, 4), (F32, (31, 2047, 1021, 181), 1, 4), (F32, (33, 640, 1280, 8), 4, 4),
    (F32, (65, 1000, 1064, 250), 4, 4), (F32, (128, 1152, 256, 116), 4, 4), (F32, (250, 704, 832, 181), 4, 4),
    (BF16, (1, 1030, 517, 97), 3, 3), (BF16, (31, 2047, 1021, 181), 4, 2), (BF16, (33, 640, 1280, 8), 4, 4),
    (BF16, (65, 1000, 1064, 250), 2, 2), (BF16, (128, 1152, 256, 116), 3, 1), (BF16, (250, 704, 832, 181), 2, 1)])
def test_slices_that_the_gpu_tests_count_on(emu, dtype, shape, forward, backward):
    M, n_in, n_out, r = (ctypes.c_longlong(v) for v in shape)
    assert (emu.emu_slices(dtype, M, n_in, n_out, r, 0), emu.emu_slices(dtype, M, n_in, n_out, r, 1)) == (forward, backward)


@pytest.mark.parametrize("shape,groups,forward,backward,one,streaming", [
    ((1, 515, 260, 65), 1, 3, 4, 1, 0), ((1, 515, 260, 65), 4, 3, 3, 1, 0), ((20, 700, 516, 129), 1, 4, 1, 1, 0), ((20, 700, 516, 129), 4, 4, 3, 1, 0),
    ((33, 1030, 900, 225), 1, 3, 1, 1, 0), ((33, 1030, 900, 225), 4, 2, 2, 1, 0), ((3, 1302, 1360, 341), 4, 2, 1, 0, 1),
    ((64, 70, 1500, 375), 4, 2, 1, 0, 0)])
def test_cell_slices_that_the_gpu_tests_count_on(emu, shape, groups, forward, backward, one, streaming):
    """test_gpu_tiles.test_lstm_cell_slices: slices of T and dT, dx and dh_prev beside the gradients or not, streaming kernels backward."""
    B, d, h, r = (ctypes.c_longlong(v) for v in shape)
    a, b = ctypes.c_int(), ctypes.c_int()
    assert emu.emu_cell_slices(B, d, h, r, groups, 0, ctypes.byref(a), ctypes.byref(b)) == forward
    assert emu.emu_cell_slices(B, d, h, r, groups, 1, ctypes.byref(a), ctypes.byref(b)) == backward
    assert (a.value, b.value) == (one, streaming)


@pytest.mark.parametrize("rows,d,h,r,groups,slices", [(1, 260, 9, 4, 1, 2), (2, 1030, 70, 33, 4, 1), (15, 36, 40, 10, 4, 2), (35, 515, 129, 31, 1, 4)])
def test_stack_slices_that_the_gpu_tests_count_on(emu, rows, d, h, r, groups, slices):
    """test_gpu_lstm.test_layer_stack_few_rows"""
    i64 = ctypes.c_longlong
    assert emu.emu_tall_slices(i64(rows), i64(d), i64(h), i64(r), groups) == slices


@pytest.mark.parametrize("shape,groups,one", [((7, 768, 768, 192), 1, 1), ((23, 640, 640, 160), 1, 1), ((200, 448, 384, 96), 4, 1),
                                              ((64, 1500, 1500, 375), 4, 0), ((87, 576, 1280, 320), 4, 0), ((188, 448, 448, 168), 4, 0)])
def test_cells_whose_gradients_go_with_dx(emu, shape, groups, one):
    """The faster of one launch and two, by a twentieth and more of the call."""
    B, d, h, r = (ctypes.c_longlong(v) for v in shape)
    got, streaming = ctypes.c_int(), ctypes.c_int()
    emu.emu_cell_slices(B, d, h, r, groups, 1, ctypes.byref(got), ctypes.byref(streaming))
    assert got.value == one


@pytest.mark.parametrize("shape,groups,streaming", [((2, 1024, 1024, 256), 4, 1), ((4, 1296, 1296, 324), 4, 1), ((2, 448, 1152, 288), 4, 1), ((4, 1024, 1024, 453), 1, 1),
                                                    ((22, 960, 960, 240), 4, 0), ((24, 1216, 1216, 304), 1, 0), ((10, 512, 512, 128), 1, 0),
                                                    ((1, 515, 1400, 402), 1, 1), ((3, 130, 1033, 290), 4, 1), ((17, 1100, 1499, 391), 4, 1),
                                                    ((33, 1500, 1500, 375), 4, 0), ((1, 3, 1500, 375), 4, 0)])
def test_cells_whose_factors_are_streamed(emu, shape, groups, streaming):
    """Backward, the faster of the streaming kernels and the tiled products by a tenth and more of the call, factors in the caches or not;
    those of test_gpu_tiles.test_lstm_cell_streamed; neither more rows than the streaming kernels take nor rows shorter than a 16-byte load."""
    B, d, h, r = (ctypes.c_longlong(v) for v in shape)
    one, got = ctypes.c_int(), ctypes.c_int()
    emu.emu_cell_slices(B, d, h, r, groups, 1, ctypes.byref(one), ctypes.byref(got))
    assert got.value == streaming


@pytest.mark.parametrize("shape,streamed", [((9, 2224, 2816, 970), 3), ((14, 2848, 4000, 712), 2), ((1, 4000, 4000, 500), 2),
                                            ((8, 2816, 3696, 704), 2), ((1, 2048, 2048, 512), 0), ((6, 2432, 3136, 608), 0), ((16, 2048, 2048, 512), 0),
                                            ((1, 2051, 1030, 515), 1), ((32, 4001, 4098, 1029), 2),
                                            ((32, 4096, 4096, 512), 0), ((33, 4096, 4096, 2000), 0), ((1, 448, 768, 112), 0), ((1, 3, 4096, 1000), 0)])
def test_layers_whose_factors_are_streamed(emu, shape, streamed):
    """Forward (1) and backward (2), the faster of the streaming kernels and the tiled products by a twentieth and more, factors in the caches or
    not; neither more rows than the streaming kernels take nor rows shorter than a 16-byte load."""
    assert emu.emu_streamed(*(ctypes.c_longlong(v) for v in shape)) == streamed
