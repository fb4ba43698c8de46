"""Index arithmetic of the one-launch LSTM recurrence without a GPU (tests/emulation/lstm_persist_host.cpp)."""
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
    out = str(tmp_path_factory.mktemp("emu") / "liblstm_persist_host.so")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
           "-I", os.path.join(ROOT, "paper_2103_03936_amd", "csrc"),
           os.path.join(ROOT, "tests", "emulation", "lstm_persist_host.cpp"), "-o", out]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("n,workgroups,rows", [
    (4 * 384 * 20, 256, 69906),   # forward, a pair per gate: 32 bits end inside
    (384 * 32, 24, 5 * 34953),    # backward, three layers, sums over slices
    (384 * 32, 24, 5 * 34952),
    (32 * 4, 8, 3 * 7),           # a step is many rows
    (128, 1, 1),
])
def test_walk_visits_every_element_once(emu, n, workgroups, rows):
    """Thread `first` of `step` visits first, first + step, ... below rows * n, also beyond 32 bits."""
    step, total = 512 * workgroups, rows * n
    count, last = ctypes.c_longlong(), ctypes.c_longlong()
    for first in {0, 1, step // 2 + 5, step - 1}:
        assert emu.emu_walk(n, first, step, rows, ctypes.byref(count), ctypes.byref(last))
        want = len(range(first, total, step))
        assert (count.value, last.value) == (want, first + (want - 1) * step if want else -1)


@pytest.mark.parametrize("T,B,h,r,groups,layers", [
    (4, 3, 40, 12, 1, 2), (3, 20, 260, 65, 1, 3), (5, 7, 33, 9, 4, 2), (3, 20, 500, 125, 4, 1), (4, 32, 640, 33, 1, 1),
    (3, 9, 1500, 375, 1, 2),
])
@pytest.mark.parametrize("bwd", [0, 1])
def test_workgroups_that_give_up_leave_nan(emu, T, B, h, r, groups, layers, bwd):
    """A wait that gives up returns no status: what its workgroups have not written yet is NaN, whatever the slot, and what
    they wrote before stays."""
    for slot in {0, 1, layers, T - 1, T + layers - 2}:
        assert emu.emu_void(T, B, h, r, groups, layers, bwd, slot) == 0, slot


@pytest.mark.parametrize("groups", [1, 4])
@pytest.mark.parametrize("bwd", [0, 1])
def test_wavefronts_wait_for_what_they_read(emu, groups, bwd):
    """The flags that a wavefront polls are those of the tasks that write its part of the exchanged matrix, over all widths."""
    ran = 0
    for h in [4, 33, 96, 130, 260, 500, 777, 1216, 1500, 1536]:
        for B in (1, 12, 20, 32):
            for layers in (1, 2, 3):
                for r in {h // 4, min(h, 33), min(h, 384)}:
                    wrong = emu.emu_watch(3, B, h, r, groups, layers, bwd)
                    assert wrong <= 0, (h, B, layers, r)
                    ran += wrong == 0
    assert ran > 30
