"""Index arithmetic of the one-launch LSTM recurrence without a GPU (tests/emulation/lstm_persist_host.cpp, linked against the library)."""
import ctypes
import os
import shutil
import subprocess

import pytest
import torch  # noqa: F401  (its HIP runtime is the one that the library uses)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not found")
    import paper_2103_03936_amd  # noqa: F401  (the library is built)
    package = os.path.join(ROOT, "paper_2103_03936_amd")
    out = str(tmp_path_factory.mktemp("emu") / "liblstm_persist_host.so")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
           "-I", os.path.join(ROOT, "paper_2103_03936_amd", "csrc"),
           os.path.join(ROOT, "tests", "emulation", "lstm_persist_host.cpp"), "-o", out, "-L" + package, "-lpufferfish",
           "-Wl,-rpath," + package]
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


@pytest.mark.parametrize("T,B,h,r,groups,layers", [(4, 21, 40, 12, 1, 2), (3, 23, 260, 65, 4, 3), (5, 31, 70, 9, 4, 2), (3, 29, 300, 75, 1, 3)])
@pytest.mark.parametrize("bwd", [0, 1])
def test_workgroups_of_half_the_rows_leave_the_others(emu, T, B, h, r, groups, layers, bwd):
    """A launch of some of the rows that gives up writes NaN over those alone: the other half's results stay, and nothing past them goes."""
    half = (B + 1) // 2
    for b0, rows in ((0, half), (half, B - half)):
        for slot in {0, layers, T + layers - 2}:
            assert emu.emu_void_rows(T, rows, h, r, groups, layers, bwd, slot, b0, B) == 0, (b0, slot)


# T, B, d, h, r, layers, groups; rows at once forward and backward (test_gpu_lstm.test_layer_stack_halves)
HALVES = [((9, 23, 12, 1100, 30, 3, 1), 12, 23), ((30, 21, 8, 1400, 20, 3, 1), 11, 11), ((6, 23, 40, 70, 12, 2, 4), 12, 12),
          ((24, 30, 20, 640, 160, 1, 4), 15, 0), ((9, 25, 12, 700, 40, 3, 4), 13, 13), ((9, 29, 12, 1200, 40, 3, 4), 15, 15),
          ((14, 31, 20, 260, 30, 2, 4), 16, 0)]


@pytest.mark.parametrize("shape,forward,backward", HALVES)
def test_rows_at_once_that_the_gpu_tests_count_on(emu, shape, forward, backward):
    """Calls that take half their rows at a time, and whose workspace holds the exchange buffers; 0: the launches of a slot."""
    T, B, d, h, r, L, G = shape
    fits = ctypes.c_int()
    for bwd, want in ((0, forward), (1, backward)):
        rows = emu.emu_rows(T, B, d, h, r, G, L, bwd, ctypes.byref(fits))
        assert (rows if fits.value else 0) == want


@pytest.mark.parametrize("shape,bwd,rows", [((34, 24, 704, 704, 176, 3, 1), 0, 12), ((4, 30, 1152, 1152, 288, 2, 1), 0, 0), ((4, 29, 1378, 1378, 344, 3, 1), 1, 0),
                                            ((37, 23, 1365, 1365, 341, 3, 1), 1, 12), ((57, 27, 128, 128, 32, 3, 4), 0, 14), ((55, 27, 960, 960, 240, 3, 4), 1, 14),
                                            ((51, 22, 1392, 1392, 348, 2, 4), 0, 11), ((51, 26, 1216, 1216, 304, 1, 4), 0, 0), ((8, 32, 832, 832, 208, 1, 4), 1, 0)])
def test_rows_at_once_are_the_faster_way(emu, shape, bwd, rows):
    """Half the rows at a time against the launches of a slot, where one is faster by a twentieth and more (whatever room there is)."""
    T, B, d, h, r, L, G = shape
    fits = ctypes.c_int()
    assert emu.emu_rows(T, B, d, h, r, G, L, bwd, ctypes.byref(fits)) == rows
