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
    lib, d = ctypes.CDLL(out), ctypes.c_double
    lib.emu_orthogonal.argtypes = [d, d, d, d]
    lib.emu_orthogonal_short.argtypes = [d, d, d, d, d, ctypes.c_int]
    lib.emu_rotation.argtypes = [d, d, d, ctypes.c_void_p]
    lib.emu_polls.restype = lib.emu_polls_then_stuck.restype = ctypes.c_longlong
    lib.emu_polls_then_stuck.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
    lib.emu_before.argtypes = [d, ctypes.c_int, d, ctypes.c_int]
    return lib


def test_a_wait_that_gave_up_is_never_reported_as_converged(emu):
    out = (ctypes.c_int * 3)()
    for sweeps, last in ((0, 0), (5, 0), (24, 3)):
        for nc in (1, 2, 300):
            emu.emu_outcome(1, 0, sweeps, last, nc, out)
            assert out[1] != 0 and out[2] == 1
            emu.emu_outcome(0, 0, sweeps, last, nc, out)
            assert list(out) == ([sweeps, last, 0] if nc > 1 else [0, 0, 0])


def test_not_finite_is_not_orthogonal(emu):
    inf, nan = float("inf"), float("nan")
    for a, b, g in ((nan, 1, 1e-20), (1, nan, 0), (1, 1, nan), (nan, nan, nan), (inf, 1, inf), (inf, inf, inf), (1, 1, -inf),
                    (inf, 0, 0)):
        assert not emu.emu_orthogonal(a, b, g, 1e-13), (a, b, g)
    for a, b, g in ((1, 1, 0), (0, 0, 0), (1e80, 1e-80, 1e-14), (2.0, 0.0, 0.0)):
        assert emu.emu_orthogonal(a, b, g, 1e-13), (a, b, g)
    assert not emu.emu_orthogonal(4, 4, 1e-12, 1e-13)


def test_rounding_noise_is_orthogonal(emu):
    """Columns 2^-280 of the longest and shorter, or with a norm that rounding left below zero, count as zero, two of 2^-100 as orthogonal
    to each other while they are held back; longer ones and what is not finite do not."""
    inf, nan, tiny, low = float("inf"), float("nan"), 2.0 ** -561, 2.0 ** -201
    for a, b, g, longest, want in ((tiny, tiny, tiny, 1, 3), (-tiny, 1, 2 ** -281, 1, 3), (1, 0.0, 1e-300, 1, 3), (4 * tiny, 1, 2 ** -280, 1, 0),
                                   (4 * tiny, 1, 2 ** -280, 16, 3), (low, low, low, 1, 1), (low, 4 * low, low, 1, 0), (low, 1, 2 ** -101, 1, 0),
                                   (1, 1, 1e-12, 1, 0), (nan, tiny, nan, 1, 0), (tiny, nan, nan, nan, 0), (tiny, inf, inf, inf, 0),
                                   (low, low, low, inf, 0)):
        for hold in (1, 0):
            got = emu.emu_orthogonal_short(a, b, g, 1e-13, longest, hold)
            assert bool(got) == bool(want & (1 if hold else 2)), (a, b, g, longest, hold)


def test_a_singular_value_that_is_not_finite_is_never_reported_as_converged(emu):
    out = (ctypes.c_int * 3)()
    for nc, want in ((1, [0, 1, 0]), (300, [3, 1, 0])):
        emu.emu_outcome(0, 1, 3, 0, nc, out)
        assert list(out) == want


def test_every_column_has_a_place(emu):
    """The order of the singular values is total, NaN included: no two columns share a place, none is left unwritten."""
    nan = float("nan")
    for v in ([3.0, nan, 5.0, nan, 5.0, 0.0, float("inf")], [nan] * 4, [1.0, 1.0, 0.0, 0.0]):
        rank = [sum(emu.emu_before(v[i], i, v[j], j) for i in range(len(v))) for j in range(len(v))]
        assert sorted(rank) == list(range(len(v)))
        finite = [v[rank.index(k)] for k in range(len(v)) if v[rank.index(k)] == v[rank.index(k)]]
        assert finite == sorted(finite, reverse=True)


def test_rotation_is_exact_to_double(emu):
    """(c, s) takes gamma out to the rounding of doubles, also between columns whose norms are 1e30 apart or equal."""
    from fractions import Fraction as F
    cs = (ctypes.c_double * 2)()
    for alpha, beta, rel in ((3.0, 2.0, 0.5), (2.0, 3.0, -0.5), (1.0, 1.0, 1e-13), (1.0, 1.0 + 2 ** -40, -1e-12), (1.0, 1e-60, 1e-13),
                             (1e-60, 1e60, 0.9), (5e70, 4e70, -1e-9), (1.0, 1.0, -1.0 + 2 ** -50)):
        gamma = rel * alpha ** 0.5 * beta ** 0.5
        emu.emu_rotation(alpha, beta, gamma, cs)
        c, s, a, b, g = (F(v) for v in (cs[0], cs[1], alpha, beta, gamma))
        assert abs(float(c * c + s * s - 1)) <= 8 * 2.0 ** -53
        # columns p, q -> c p - s q, s p + c q: their inner product, relative to what it was
        assert abs(float((c * s * (a - b) + (c * c - s * s) * g) / g)) <= 16 * 2.0 ** -53, (alpha, beta, gamma)


def test_rotation_of_cancelled_columns(emu):
    """Norms that rounding left zero, opposite or negative, with an inner product between them: still a rotation, by 45 degrees at most."""
    cs = (ctypes.c_double * 2)()
    for alpha, beta, gamma in ((0.0, 0.0, 1e-40), (-1e-30, 1e-30, 1e-31), (1e-30, -1e-30, -1e-29), (-2e-33, 1e-33, 0.0), (-1e-320, 1e-310, 1e-315),
                               (1e-30, -1e-30 * (1 - 2 ** -50), 1e-50), (0.0, 4e300, 1e-10), (0.0, 0.0, 5e-324)):
        emu.emu_rotation(alpha, beta, gamma, cs)
        assert abs(cs[0] ** 2 + cs[1] ** 2 - 1) <= 8 * 2.0 ** -53 and abs(cs[1]) <= 0.5 ** 0.5 * (1 + 2.0 ** -50), (alpha, beta, gamma)


def test_workgroups_that_wait_for_one_another_are_all_resident(emu):
    """The tridiagonal route is taken by devices with a compute unit for each of its workgroups, the Jacobi iteration by others."""
    for n, workgroups in ((17, 0), (128, 0), (129, 33), (512, 128), (513, 65), (1537, 193), (2048, 256)):
        assert emu.emu_takes_eigenvectors(n, workgroups) and emu.emu_takes_eigenvectors(n, 304)
        assert workgroups == 0 or not emu.emu_takes_eigenvectors(n, workgroups - 1)
    assert not emu.emu_takes_eigenvectors(16, 256) and not emu.emu_takes_eigenvectors(2049, 304)


@pytest.mark.parametrize("rounds,each", [(280, 60000), (2, 3999999), (40, 1000000), (280, 40)])
def test_who_waits_for_sweeps_outlasts_them(emu, rounds, each):
    """A stage of sweeps is many rounds (ten sweeps of 64 columns: 70 and more), each of them well within the limit of a wait but not all
    together: 70 rounds of 30 ms at two polls a microsecond are 4.2 million polls."""
    assert emu.emu_polls(rounds, each) == rounds * each


@pytest.mark.parametrize("rounds", [0, 1, 3])
def test_a_wait_ends_without_progress(emu, rounds):
    """Rounds of a thousand polls, then nothing: given up within the limit, counted from the last round seen."""
    limit = 4000000
    got = emu.emu_polls_then_stuck(rounds, 1000, 2 * limit)
    assert abs(got - limit - rounds * 1000) <= 1256


def test_workgroups_that_have_no_pair_wait(emu):
    """Of eight workgroups the preconditioner has all; B of 64 columns has four pairs of blocks, of 112 seven, of 113 eight."""
    for nc, crew in ((1, 1), (16, 1), (17, 2), (64, 4), (112, 7), (113, 8), (128, 8), (129, 9)):
        sweepers = max(8, crew)
        assert emu.emu_crew(0, nc, sweepers) == sweepers
        assert emu.emu_crew(1, nc, sweepers) == emu.emu_crew(2, nc, sweepers) == crew
