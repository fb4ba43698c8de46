"""Which shapes the bf16 factor gradients take (tests/emulation/linear_host.cpp, linked against the library), without a GPU."""
import ctypes
import os
import shutil
import subprocess

import pytest
import torch  # noqa: F401  (its HIP runtime is the one that the library uses)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2103_03936_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not found")
    import paper_2103_03936_amd  # noqa: F401  (the library is built)
    out = str(tmp_path_factory.mktemp("emu") / "liblinear_host.so")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(PACKAGE, "csrc"),
           os.path.join(ROOT, "tests", "emulation", "linear_host.cpp"), "-o", out, "-L" + PACKAGE, "-lpufferfish", "-Wl,-rpath," + PACKAGE]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE)
    return ctypes.CDLL(out)


def test_arrays_that_a_descriptor_holds(emu):
    """Every array is less than 2^31 bytes of bf16: both matrices of a gradient, also where the rank is above the width."""
    i64 = ctypes.c_longlong
    takes = lambda *s: (emu.emu_grad_takes(*map(i64, s)), emu.emu_grad_splits(*map(i64, s)) > 0)
    assert takes(8192, 512, 512, 128) == (1, True)
    assert takes((1 << 23) - 1, 104, 104, 128) == (1, True)
    for M, n_in, n_out, r in [(1 << 23, 104, 104, 128), (10300000, 104, 104, 128), (1 << 21, 512, 104, 128), (1 << 21, 104, 512, 128)]:
        assert takes(M, n_in, n_out, r) == (0, False), (M, n_in, n_out, r)
