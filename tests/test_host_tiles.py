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
