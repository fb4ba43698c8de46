"""GPU parity of the two-stage kernel (pf_linear_two.h) with every number of rows per workgroup, against torch in float32: widths
and ranks beside their tiles, one row, layers that share their input, outputs shared by several workgroups, masks; of the factor
gradients (pf_linear_grad.h) with columns, ranks and runs of rows beside their tiles; and of the backward call on both."""
import ctypes
import os
import subprocess

import pytest
import torch

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2103_03936_amd")


@pytest.fixture(scope="module")
def two(tmp_path_factory):
    import paper_2103_03936_amd  # noqa: F401  (the library is loaded)
    out = str(tmp_path_factory.mktemp("two") / "liblinear_two.so")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(PACKAGE, "csrc"),
                    os.path.join(ROOT, "tests", "emulation", "linear_two_launch.cpp"), "-o", out, "-L" + PACKAGE, "-lpufferfish",
                    "-Wl,-rpath," + PACKAGE], check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("M,K,N,r,G", [(1, 8, 8, 8, 1), (33, 136, 264, 19, 2), (300, 72, 40, 128, 1), (129, 1032, 520, 65, 3), (200, 264, 1048, 100, 1),
                                       (97, 128, 128, 32, 1), (31, 384, 136, 40, 2), (260, 520, 392, 61, 1)])
def test_parity(two, M, K, N, r, G):
    """An output is rounded to bf16 once, a share of 2^-8 = 3.9e-3 at most; the intermediate before the second stage, here and in the reference."""
    g = torch.Generator(device="cuda").manual_seed(3)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X, V, U = n(M, K).bfloat16(), (n(G, K, r) * K ** -0.5).bfloat16(), (n(G, N, r) * r ** -0.5).bfloat16()
    bias, add = n(G, N).bfloat16(), n(M, N).bfloat16()
    for rows in (32, 64, 128):
        chunks = (N + 127) // 128
        for osplit in {1, min(2, chunks), chunks}:
            for ep in (False, True):
                Y, T = (torch.full((G, M, w), float("nan"), dtype=torch.bfloat16, device="cuda") for w in (N, r))
                args = [X, V, U, bias if ep else None, add if ep and G == 1 else None]
                p = lambda t: ctypes.c_void_p(None if t is None else t.data_ptr())
                st = two.linear_two(ctypes.c_longlong(M), K, N, r, G, rows, osplit, *map(p, args), int(ep), p(Y), p(T), None,
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
                assert st == 0
                want = T.float() @ U.float().transpose(1, 2).contiguous()
                if ep:
                    want = (want + bias.float()[:, None] + (add.float() if G == 1 else 0)).clamp_min(0)
                for got, ref in ((T, X.float() @ V.float()), (Y, want)):
                    err = (got.double() - ref.double()).norm() / ref.double().norm().clamp_min(1e-30)
                    assert err <= 4e-3, (rows, osplit, ep, err)


@pytest.mark.parametrize("M,K,N,r", [(1, 8, 8, 8), (70, 136, 264, 24), (300, 72, 136, 64), (129, 264, 648, 128)])
def test_mask(two, M, K, N, r):
    """An output stays where the mask is above zero: not at zeros of either sign, negative values or NaN."""
    g = torch.Generator(device="cuda").manual_seed(4)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X, V, U, add = n(M, K).bfloat16(), (n(K, r) * K ** -0.5).bfloat16(), (n(N, r) * r ** -0.5).bfloat16(), n(M, N).bfloat16()
    special = torch.tensor([0.0, -0.0, float("nan"), float("inf"), float("-inf"), 1e-37, -1e-37, 3e38], device="cuda").bfloat16()
    mask = torch.where(n(M, N) > 0.5, special[torch.arange(M * N, device="cuda") % 8].reshape(M, N), n(M, N).bfloat16())
    kept = mask.float() > 0
    p = lambda t: ctypes.c_void_p(None if t is None else t.data_ptr())
    for rows in (32, 64, 128):
        for a in (None, add):
            for osplit in {1, (N + 127) // 128}:
                Y, T = (torch.full((M, w), float("nan"), dtype=torch.bfloat16, device="cuda") for w in (N, r))
                assert two.linear_two(ctypes.c_longlong(M), K, N, r, 1, rows, osplit, p(X), p(V), p(U), None, p(a), 0, p(Y), p(T), p(mask),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
                want = T.float() @ U.float().t().contiguous() + (0 if a is None else a.float())
                assert bool((Y[~kept] == 0).all())
                assert float((Y[kept].double() - want[kept].double()).norm()) <= 4e-3 * float(want.double().norm())  # one rounding to bf16


@pytest.mark.parametrize("M,K,N,r,G", [(1, 136, 136, 136, 1), (33, 264, 392, 160, 2), (130, 1032, 648, 168, 1), (70, 192, 128, 192, 3), (97, 520, 264, 200, 1),
                                       (200, 256, 1048, 256, 2)])
def test_wide_ranks(two, M, K, N, r, G):
    """Ranks above 128, first and last of five, six and eight blocks; tolerances as above (and nothing of LDS beyond the rank is seen)."""
    g = torch.Generator(device="cuda").manual_seed(6)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X, V, U = n(M, K).bfloat16(), (n(G, K, r) * K ** -0.5).bfloat16(), (n(G, N, r) * r ** -0.5).bfloat16()
    bias, add, mask = n(G, N).bfloat16(), n(M, N).bfloat16(), n(M, N).bfloat16()
    p = lambda t: ctypes.c_void_p(None if t is None else t.data_ptr())
    for rows in (32, 64, 128):
        for osplit in {1, (N + 127) // 128}:
            for ep in (False, True):
                Y, T = (torch.full((G, M, w), float("nan"), dtype=torch.bfloat16, device="cuda") for w in (N, r))
                one = ep and G == 1
                args = [X, V, U, bias if ep else None, add if one else None]
                st = two.linear_two(ctypes.c_longlong(M), K, N, r, G, rows, osplit, *map(p, args), int(ep and not one), p(Y), p(T), p(mask if one else None),
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
                assert (st == 0) == (rows <= (64 if r <= 192 else 32))
                if st != 0:
                    continue
                want = T.float() @ U.float().transpose(1, 2).contiguous()
                if ep:
                    want = want + bias.float()[:, None]
                    want = (want[0] + add.float())[None] * (mask.float() > 0) if one else want.clamp_min(0)
                for got, ref in ((T, X.float() @ V.float()), (Y, want)):
                    err = (got.double() - ref.double()).norm() / ref.double().norm().clamp_min(1e-30)
                    assert err <= 4e-3, (rows, osplit, ep, err)


@pytest.mark.parametrize("M,cols,r", [(64, (136, 264), 136), (333, (392, 160), 192), (1030, (200, 640), 200), (577, (256, 256), 256)])
def test_wide_gradients(two, M, cols, r):
    test_gradients(two, M, cols, r)


@pytest.mark.parametrize("M,cols,r", [(64, (8, 8), 8), (65, (136, 120), 40), (1000, (264, 72), 64), (700, (128, 640), 128), (1030, (1032, 8), 24),
                                      (577, (256, 128), 96)])
def test_gradients(two, M, cols, r):
    """Sums over M products that float32 holds exactly: 2^-24 each on the way, in a random direction (twice that is allowed)."""
    g = torch.Generator(device="cuda").manual_seed(5)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    A, B, chunks = [n(M, c) for c in cols], [n(M, r) for _ in cols], (M + 63) // 64
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    for per in {1, 2, 3, chunks}:
        splits = (chunks + per - 1) // per
        out = [torch.full((splits, c, r), float("nan"), device="cuda") for c in cols]
        sums = torch.full((splits, cols[0]), float("nan"), device="cuda")
        assert two.linear_grad(ctypes.c_longlong(M), r, splits, per, 2, cols[0], p(A[0]), p(B[0]), p(out[0]), p(sums), cols[1], p(A[1]), p(B[1]), p(out[1]),
                               ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        for got, ref in [(o.double().sum(0), a.double().t() @ b.double()) for o, a, b in zip(out, A, B)] + [(sums.double().sum(0), A[0].double().sum(0))]:
            assert float((got - ref).norm() / ref.norm()) <= M ** 0.5 * 2 ** -23, per


@pytest.mark.parametrize("shape", [(5000, 1536, 384, 96), (6001, 1032, 264, 64), (8192, 512, 512, 128)])
def test_backward(shape):
    """The public call where it takes both kernels (more rows than the oracle's tests have): T kept or not, mask and skip gradient."""
    import paper_2103_03936_amd as pf
    got = None
    M, K, N, r = shape
    g = torch.Generator(device="cuda").manual_seed(6)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X, V, U = n(M, K).bfloat16(), (n(K, r) * K ** -0.5).bfloat16(), (n(N, r) * r ** -0.5).bfloat16()
    dY, add = n(M, N).bfloat16(), n(M, K).bfloat16()
    T = (X.float() @ V.float()).bfloat16()
    dT = (dY.float() @ U.float()).bfloat16().float()
    dX, grads = dT @ V.float().t().contiguous(), (dY.float().t() @ T.float(), X.float().t() @ dT, dY.float().sum(0))
    for a, relu, kept in ((None, False, True), (add, False, False), (None, True, True), (add, True, True)):
        want = dX + (0 if a is None else a.float())
        want = torch.where(X.float() > 0, want, torch.zeros_like(want)) if relu else want

        def call():
            nonlocal got
            got = pf.pf_lowrank_linear_bwd_ep(X, V, U, dY, T_saved=T if kept else None, dX_add=a, x_is_relu=relu, has_bias=True)

        assert {"linear_bwd_data_two", "linear_grads"} <= _launches(pf, call)
        for x, ref in zip(got, (want,) + grads):  # (a share of 2^-8 per rounding to bf16; dT and T may round either way here)
            assert float((x.double() - ref.double()).norm() / ref.double().norm()) <= 4e-3


@pytest.mark.parametrize("shape", [(8192, 640, 640, 160), (8000, 2048, 320, 200)])
def test_wide_backward(shape):
    test_backward(shape)


@pytest.mark.parametrize("wanted", [(1, 1, 1), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1), (0, 1, 1), (0, 0, 0)])
def test_backward_in_parts(wanted):
    """Gradients that are wanted, added to what a flat buffer holds at an odd element, dX beside them; the others are not formed and the
    buffer's other elements stay as they are.  Bounds as above."""
    import paper_2103_03936_amd as pf
    M, K, N, r = 6001, 1032, 264, 64
    g = torch.Generator(device="cuda").manual_seed(7)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X, V, U, dY = n(M, K).bfloat16(), (n(K, r) * K ** -0.5).bfloat16(), (n(N, r) * r ** -0.5).bfloat16(), n(M, N).bfloat16()
    T = (X.float() @ V.float()).bfloat16()
    dT = (dY.float() @ U.float()).bfloat16().float()
    want = [dT @ V.float().t().contiguous(), dY.float().t() @ T.float(), X.float().t() @ dT, dY.float().sum(0)]
    shapes, flat = ((N, r), (K, r), (N,)), n(1 + N * r + K * r + N + 3) * 30
    held, at, out = flat.clone(), 1, []
    for s in shapes:
        size = torch.Size(s).numel()
        out.append(flat[at:at + size].view(s))
        at += size
    grads = tuple(o if w else None for o, w in zip(out, wanted))
    got = None

    def call():
        nonlocal got
        got = pf.pf_lowrank_linear_bwd(X, V, U, dY, T_saved=T, has_bias=True, grads=grads)

    names = _launches(pf, call)
    assert ("linear_bwd_data_two" in names) and ("linear_grads" in names) == any(wanted)
    assert float((got[0].double() - want[0].double()).norm() / want[0].double().norm()) <= 4e-3
    before, at = held[1:], 0
    for o, w, ref in zip(out, wanted, want[1:]):
        was = before[at:at + ref.numel()].view(ref.shape)
        at += ref.numel()
        if w:
            assert float((o.double() - was.double() - ref.double()).norm() / ref.double().norm()) <= 4e-3
        else:
            assert torch.equal(o, was)
    assert flat[0] == held[0] and torch.equal(flat[-3:], held[-3:])


def _launches(pf, call):
    """What a call launches, by the library's own records."""
    pf.timing_reset()
    pf.timing_enable(True)
    call()
    pf.timing_enable(False)
    return set(pf.timing_collect())


@pytest.mark.parametrize("M,K,r,N,forward,two", [(2000, 256, 64, 1024, True, True), (3001, 640, 96, 640, True, True), (7, 576, 67, 2824, True, False),
                                                 (1313, 1104, 83, 2016, True, False), (8192, 512, 128, 2048, False, True), (6001, 1032, 64, 264, False, True),
                                                 (4891, 480, 72, 496, False, False), (4246, 768, 64, 256, False, False)])
def test_where_it_is_the_faster_one(M, K, r, N, forward, two):
    """Shapes on both sides of the rule: 1.2 to 1.5 times as fast on these kernels, or on the tiled products."""
    import paper_2103_03936_amd as pf
    b = lambda *s: torch.randn(*s, device="cuda").bfloat16()
    X, V, U, T, dY = b(M, K), b(K, r), b(N, r), b(M, r), b(M, N)
    names = _launches(pf, (lambda: pf.pf_lowrank_linear_fwd(X, V, U)) if forward else (lambda: pf.pf_lowrank_linear_bwd(X, V, U, dY, T_saved=T)))
    assert (("linear_fwd_two" if forward else "linear_bwd_data_two") in names) == two, names


@pytest.mark.parametrize("M,K,N", [(8192, 512, 512), (6001, 256, 256), (8193, 512, 256)])
def test_plain_calls_and_epilogues(M, K, N):
    """Calls without residual input and ReLU may run on another kernel than those with them.  Bounds as above."""
    import paper_2103_03936_amd as pf
    g = torch.Generator(device="cuda").manual_seed(6)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X, V, U, bias = n(M, K).bfloat16(), (n(K, 128) * K ** -0.5).bfloat16(), (n(N, 128) * 128 ** -0.5).bfloat16(), n(N).bfloat16()
    for Y, T in (pf.pf_lowrank_linear_fwd(X, V, U, bias), pf.pf_lowrank_linear_fwd_ep(X, V, U, bias, residual=X.new_zeros(M, N))):
        for got, ref in ((T, X.float() @ V.float()), (Y, T.float() @ U.float().t() + bias.float())):
            assert (got.double() - ref.double()).norm() <= 4e-3 * ref.double().norm()
