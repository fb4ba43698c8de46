"""Decisions of the Jacobi SVD without a GPU (tests/emulation/svd_host.cpp)."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not found")
    out = str(tmp_path_factory.mktemp("emu") / "libsvd_host.so")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
           "-I", os.path.join(ROOT, "paper_2103_03936_amd", "csrc"),
           os.path.join(ROOT, "tests", "emulation", "svd_host.cpp"), "-o", out]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE)
    return ctypes.CDLL(out)


def test_a_wait_that_gave_up_is_never_reported_as_converged(emu):
    out = (ctypes.c_int * 3)()
    for sweeps, last in ((0, 0), (5, 0), (24, 3)):
        for nc in (1, 2, 300):
            emu.emu_outcome(1, sweeps, last, nc, out)
            assert out[1] != 0 and out[2] == 1
            emu.emu_outcome(0, sweeps, last, nc, out)
            assert list(out) == ([sweeps, last, 0] if nc > 1 else [0, 0, 0])
