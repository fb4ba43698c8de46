"""GPU parity of the pixel-major convolution kernels (pf_conv_px.h), every tile size with every rank block, against torch in 64 bits:
planes that are whole 16-byte pieces and not, tiles over several images, a last tile that is not full, ranks and channels beside their blocks."""
import ctypes
import os
import subprocess

import pytest
import torch
import torch.nn.functional as F

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2103_03936_amd")
TILES = [(128, 512), (64, 512), (32, 512), (128, 256), (64, 256), (32, 256)]
SHAPES = [
    # N, C, H, W, Cout, r, k
    (2, 64, 16, 16, 96, 32, 3),
    (9, 72, 5, 5, 40, 13, 3),      # planes of three pieces and a pixel, several to a tile
    (3, 136, 9, 11, 264, 64, 3),   # more than one chunk of channels, of output channels
    (1, 24, 4, 2, 8, 1, 3),        # one piece per plane, one rank
    (2, 40, 31, 29, 24, 33, 3),
    (5, 200, 7, 7, 80, 100, 3),
    (1, 520, 6, 10, 16, 128, 3),
    (4, 64, 32, 32, 64, 16, 1),
    (7, 264, 3, 5, 136, 37, 1),
    (3, 24, 13, 3, 520, 65, 1),
]
SHAPES_F32 = [s for s in SHAPES if s[5] <= 64] + [(2, 44, 5, 5, 36, 7, 3), (40, 12, 2, 3, 4, 40, 3), (3, 68, 13, 3, 100, 30, 1),
                                                 (9, 12, 5, 5, 76, 1, 1), (2, 264, 10, 6, 4, 32, 1)]  # (whole pieces: four)


@pytest.fixture(scope="module")
def px(tmp_path_factory):
    import paper_2103_03936_amd  # noqa: F401  (the library is loaded)
    out = str(tmp_path_factory.mktemp("px") / "libconv_px.so")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(PACKAGE, "csrc"),
                    os.path.join(ROOT, "tests", "emulation", "conv_px_launch.cpp"), "-o", out, "-L" + PACKAGE, "-lpufferfish",
                    "-Wl,-rpath," + PACKAGE], check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE)
    lib = ctypes.CDLL(out)
    lib.px_pack_size.restype = ctypes.c_size_t
    return lib


def _entry(px, name, dtype):
    return getattr(px, f"px_{name}_{'f32' if dtype == torch.float32 else 'bf16'}")


def _call(f, *args):
    conv = [ctypes.c_void_p(a.data_ptr()) if torch.is_tensor(a) else ctypes.c_void_p(None) if a is None else a for a in args]
    return f(*conv, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))


def _close(got, want, rel, what):
    err = (got.double() - want.double()).norm() / want.double().norm().clamp_min(1e-30)
    assert torch.isfinite(got.float()).all() and err <= rel, f"{what}: {err:.2e} > {rel:.0e}"


@pytest.mark.parametrize("dtype, shape", [(torch.bfloat16, s) for s in SHAPES] + [(torch.float32, s) for s in SHAPES_F32])
def test_parity(px, dtype, shape):
    """Rounding to bf16 changes an output by a share of 2^-8 = 3.9e-3 at most (1.7e-3 rms over many; the smallest shape has 64 outputs);
    sums of some thousand float products have errors of 2^-24 each.  T and dT are rounded before the second stage, here and in the
    reference; filter gradients add products of bf16 in float."""
    N, C, H, W, Cout, r, k = shape
    f32 = dtype == torch.float32
    tol, V = (1e-6, 4) if f32 else (4e-3, 8)
    g = torch.Generator(device="cuda").manual_seed(7)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    b = lambda t: t.to(dtype)
    X, dZ = b(n(N, C, H, W).clamp_min(0)), b(n(N, Cout, H, W))
    Uk, Vp = b(n(r, C, k, k) * (C * k * k) ** -0.5), b(n(Cout, r) * r ** -0.5)
    scale, shift = torch.rand(Cout, generator=g, device="cuda") + 0.5, n(Cout) * 0.2
    res, add = b(n(N, Cout, H, W)), b(n(N, C, H, W))
    h, out = lambda t: t.cpu().double(), lambda t: t.cuda()
    T = out(F.conv2d(h(X), h(Uk), padding=k // 2))
    col = lambda v: v[None, :, None, None]
    Vs = b(Vp.float() * scale[:, None])
    dT = out(F.conv2d(h(dZ), h(Vs).t()[:, :, None, None]))
    dX = out(torch.nn.grad.conv2d_input(X.shape, h(Uk), h(b(dT)), padding=k // 2))
    rv, taken, back = (r + V - 1) // V * V, 0, not f32 or (k == 1 and r <= 32)
    for P, threads in TILES:
        pack = torch.zeros(px.px_pack_size(C, r, k), dtype=dtype, device="cuda")
        for ep in (False, True):
            Y, T1 = torch.full_like(res, float("nan")), torch.full((N, r, H, W), float("nan"), dtype=dtype, device="cuda")
            st = _call(_entry(px, "fwd", dtype), N, C, H, W, Cout, r, k, 1, P, threads, X, Uk, Vp, scale if ep else None, shift if ep else None,
                       res if ep else None, int(ep), Y, T1, pack)
            if st:
                assert st == 100 or (threads == 256 and (f32 or r > 64)), st
                break
            taken += 1
            what = f"{shape} {P} pixels, {threads} threads"
            _close(T1, T, tol, what + " T")
            want = out(F.conv2d(h(T1), h(Vp)[:, :, None, None]))
            _close(Y, (want * col(scale) + col(shift) + res).clamp_min(0) if ep else want, tol, what + " Y")
            if not back:
                continue
            dX1, dT1 = torch.full_like(X, float("nan")), torch.full((N, rv, H, W), float("nan"), dtype=dtype, device="cuda")
            assert _call(_entry(px, "bwd", dtype), N, C, H, W, Cout, r, k, P, threads, dZ, Vp, pack, scale, add if ep else None, X if ep else None,
                         dX1, dT1) == 0
            _close(dT1[:, :r], dT, tol, what + " dT")
            assert not dT1[:, r:].any()
            _close(dX1, (dX + add) * (X > 0) if ep else dX, tol, what + " dX")
    assert taken >= (3 if f32 else 6), "most tile sizes take the shape"
    if not back:
        return
    Tb, dTb = b(T).contiguous(), torch.zeros(N, rv, H, W, dtype=dtype, device="cuda")
    dTb[:, :r] = b(dT)
    tiles = (N * H * W + 127) // 128
    want_U = out(torch.nn.grad.conv2d_weight(h(X), Uk.shape, h(dTb[:, :r]), padding=k // 2))
    want_V = torch.einsum("nop,nrp->or", dZ.flatten(2).double(), Tb.flatten(2).double())
    for per in {1, 3, tiles}:
        groups = (tiles + per - 1) // per
        pU, pV, ps = (torch.full((groups, m), float("nan"), device="cuda") for m in (r * C * k * k, r * Cout, Cout))
        assert _call(_entry(px, "wgrad", dtype), N, C, H, W, Cout, r, k, per, dTb, X, Tb, dZ, pU, pV, ps) == 0
        _close(pU.sum(0).view(r, C, k, k), want_U, 1e-5, f"{shape} dUk")
        _close(pV.sum(0).view(r, Cout).t(), want_V, 1e-5, f"{shape} dVp")
        _close(ps.sum(0), dZ.double().sum((0, 2, 3)), 1e-5, f"{shape} sums")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("shape", [
    # N, C, H, W, Cout, r, k, stride
    (3, 136, 16, 16, 264, 64, 3, 2),
    (9, 72, 9, 11, 40, 13, 3, 2),   # output planes of 5 x 6
    (2, 24, 8, 33, 16, 32, 3, 2),
    (40, 8, 7, 7, 72, 40, 1, 2),
    (3, 264, 16, 16, 136, 37, 1, 2),
    (5, 16, 7, 21, 24, 8, 1, 3),
])
def test_strided_forward(px, dtype, shape):
    """Bounds as above."""
    N, C, H, W, Cout, r, k, stride = shape
    tol = 1e-6 if dtype == torch.float32 else 4e-3
    g = torch.Generator(device="cuda").manual_seed(9)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X, Uk, Vp = n(N, C, H, W).to(dtype), (n(r, C, k, k) * (C * k * k) ** -0.5).to(dtype), (n(Cout, r) * r ** -0.5).to(dtype)
    h, out = lambda t: t.cpu().double(), lambda t: t.cuda()
    T = out(F.conv2d(h(X), h(Uk), stride=stride, padding=k // 2))
    res, taken = n(N, Cout, *T.shape[2:]).to(dtype), 0
    for P, threads in TILES:
        Y, T1 = torch.full_like(res, float("nan")), torch.full(T.shape, float("nan"), dtype=dtype, device="cuda")
        st = _call(_entry(px, "fwd", dtype), N, C, H, W, Cout, r, k, stride, P, threads, X, Uk, Vp, None, None, res, 0, Y, T1, None)
        if st:
            assert st == 100 or threads == 256 or P == 128 or (P == 64 and k == 3), st
            continue
        taken += 1
        _close(T1, T, tol, f"{shape} {P} T")
        _close(Y, out(F.conv2d(h(T1), h(Vp)[:, :, None, None])) + res, tol, f"{shape} {P} Y")
    assert taken >= 1


def test_infinite_input(px):
    """An infinite input pixel gives infinities and NaN where its taps reach and nowhere else; ranks beside the blocks stay out of it."""
    N, C, H, W, Cout, r, k = 1, 64, 12, 12, 32, 20, 3
    g = torch.Generator(device="cuda").manual_seed(8)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    X, Uk, Vp = n(N, C, H, W), n(r, C, k, k), n(Cout, r).abs()
    X[0, 5, 4, 4] = float("inf")
    Uk[:, 5] = Uk[:, 5].abs()
    for P, threads in TILES:
        Y, T = torch.empty(N, Cout, H, W, dtype=torch.bfloat16, device="cuda"), torch.empty(N, r, H, W, dtype=torch.bfloat16, device="cuda")
        assert _call(px.px_fwd_bf16, N, C, H, W, Cout, r, k, 1, P, threads, X, Uk, Vp, None, None, None, 0, Y, T, None) == 0
        want = torch.zeros(H, W, dtype=torch.bool, device="cuda")
        want[3:6, 3:6] = True
        assert (torch.isposinf(Y) == want).all() and torch.isfinite(Y[:, :, ~want]).all(), (P, threads)


@pytest.mark.parametrize("shape", [(3, 72, 12, 12, 24, 20, 3), (5, 64, 5, 7, 16, 33, 3), (4, 40, 16, 16, 8, 128, 3), (2, 136, 9, 11, 8, 64, 3)])
def test_infinite_edges_in_gradients(px, shape):
    """An infinite (or NaN) pixel at the edge of its plane is in the gradients of the taps that see it and in no others, as a sum over the
    terms that exist has it; what is finite is within float rounding of it (M terms of 2^-24 in a random direction, twice that is allowed)."""
    N, C, H, W, Cout, r, k = shape
    g = torch.Generator(device="cuda").manual_seed(13)
    b = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    dT, mid, dZ, rv, tiles = torch.zeros(N, (r + 7) // 8 * 8, H, W, device="cuda").bfloat16(), b(N, r, H, W), b(N, Cout, H, W), (r + 7) // 8 * 8, (N * H * W + 127) // 128
    dT[:, :r] = b(N, r, H, W).abs() + 0.1
    for places in ([(0, 5, 0, 0, "inf")], [(N - 1, C - 1, H - 1, 2, "-inf"), (1, 7, 3, W - 1, "inf")], [(0, 3, 2, 0, "nan"), (1, 4, 2, 2, "inf")]):
        X = b(N, C, H, W)
        for n, c, y, x, v in places:
            X[n, c, y, x] = float(v)
        want = torch.empty(r, C, 3, 3, dtype=torch.float64)
        A, B = dT[:, :r].cpu().double(), X.cpu().double()
        for i in range(3):
            for j in range(3):
                ys, xs, yo, xo = slice(max(0, i - 1), H + min(0, i - 1)), slice(max(0, j - 1), W + min(0, j - 1)), slice(max(0, 1 - i), H + min(0, 1 - i)), slice(max(0, 1 - j), W + min(0, 1 - j))
                want[:, :, i, j] = (A[:, :, None, yo, xo] * B[:, None, :, ys, xs]).sum((0, 3, 4))
        for per in {1, 3, tiles}:
            groups = (tiles + per - 1) // per
            pU, pV, ps = (torch.full((groups, m), float("nan"), device="cuda") for m in (r * C * 9, r * Cout, Cout))
            assert _call(px.px_wgrad_bf16, N, C, H, W, Cout, r, k, per, dT, X, mid, dZ, pU, pV, ps) == 0
            got, ok = pU.cpu().double().sum(0).view(r, C, 3, 3), torch.isfinite(want)
            assert (torch.isfinite(got) == ok).all() and (torch.isposinf(got) == torch.isposinf(want)).all() and (torch.isnan(got) == torch.isnan(want)).all(), (places, per)
            assert float((got - want)[ok].norm() / want[ok].norm()) <= (N * H * W) ** 0.5 * 2 ** -23
            assert torch.isfinite(pV).all()


@pytest.mark.parametrize("dtype, shape", [(torch.float32, (88, 64, 13, 10, 64, 16, 1)), (torch.float32, (12, 96, 14, 14, 96, 24, 1)),
                                          (torch.float32, (2, 44, 5, 5, 36, 7, 3)), (torch.bfloat16, (12, 128, 16, 16, 128, 32, 3))])
def test_saved_filters_stay_in_their_buffer(dtype, shape):
    """A forward call writes as many bytes of W_save as the query states and none beyond, and the backward call gives the same with and
    without them."""
    import paper_2103_03936_amd as pf
    N, C, H, W, Cout, r, k = shape
    g = torch.Generator(device="cuda").manual_seed(12)
    b = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dtype)
    X, Uk, Vp, dY = b(N, C, H, W), b(r, C, k, k) * (C * k * k) ** -0.5, b(Cout, r) * r ** -0.5, b(N, Cout, H, W)
    d = pf.pf_conv_desc(N, C, H, W, Cout, r, k, 1, k // 2, pf.PF_NCHW, pf.PF_F32 if dtype == torch.float32 else pf.PF_BF16, pf.PF_F32)
    size, guard = pf.lib.pf_lowrank_conv_saved_weights_bytes(ctypes.byref(d)), 1 << 20
    kept = torch.full((size + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = torch.empty(pf.lib.pf_lowrank_conv_fwd_workspace_bytes(ctypes.byref(d)), dtype=torch.uint8, device="cuda")
    Y, T = torch.empty_like(dY), torch.empty(N, r, H, W, dtype=dtype, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert pf.lib.pf_lowrank_conv_fwd(ctypes.byref(d), p(X), p(Uk), p(Vp), p(Y), p(T), p(kept), p(ws), ctypes.c_size_t(ws.numel()),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert bool((kept[size:] == 0xA5).all()) and (size == 0) == (k == 3 and dtype == torch.float32)
    one = pf.pf_lowrank_conv_bwd(X, Uk, Vp, dY, T_saved=T, pad=k // 2)
    other = pf.pf_lowrank_conv_bwd(X, Uk, Vp, dY, T_saved=T, pad=k // 2, W_saved=kept[:size] if size else None)
    assert all(torch.equal(x, y) for x, y in zip(one, other))


@pytest.mark.parametrize("dtype, shape", [(torch.float32, (88, 64, 13, 10, 64, 16, 1)), (torch.bfloat16, (12, 128, 16, 16, 128, 32, 3)),
                                          (torch.bfloat16, (30, 96, 9, 11, 128, 20, 1))])
def test_gradients_are_added(dtype, shape):
    """The public backward call with batch norm adds to what a flat buffer holds at an odd element, on these kernels, and to nothing else."""
    import paper_2103_03936_amd as pf
    N, C, H, W, Cout, r, k = shape
    g = torch.Generator(device="cuda").manual_seed(15)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    b = lambda *s: n(*s).to(dtype)
    X, Uk, Vp, dZ = b(N, C, H, W), b(r, C, k, k) * (C * k * k) ** -0.5, b(Cout, r) * r ** -0.5, b(N, Cout, H, W)
    scale = torch.rand(Cout, generator=g, device="cuda") + 0.5
    Y, T, kept = pf.pf_lowrank_conv_fwd_ep(X, Uk, Vp, scale, pad=k // 2, save_W=True)
    plain = pf.pf_lowrank_conv_bwd_ep(X, Uk, Vp, scale, dZ, T_saved=T, pad=k // 2, W_saved=kept)
    shapes, flat = ((r, C, k, k), (Cout, r), (Cout,)), n(1 + r * C * k * k + Cout * r + Cout + 3)
    held, at, out = flat.clone(), 1, []
    for s in shapes:
        size = torch.Size(s).numel()
        out.append(flat[at:at + size].view(s))
        at += size
    pf.timing_reset()
    pf.timing_enable(True)
    dX = pf.pf_lowrank_conv_bwd_ep(X, Uk, Vp, scale, dZ, T_saved=T, pad=k // 2, W_saved=kept, grads=tuple(out))[0]
    pf.timing_enable(False)
    assert {"conv_bwd_px", "conv_wgrad_px", "split_sums"} == set(pf.timing_collect())
    assert torch.equal(dX, plain[0]) and flat[0] == held[0] and torch.equal(flat[-3:], held[-3:])
    at = 1
    for o, p in zip(out, plain[1:]):
        was = held[at:at + p.numel()].view(p.shape)
        at += p.numel()
        assert torch.equal(o, was + p) or float((o - was - p).abs().max()) <= 2 ** -22 * float((was.abs() + p.abs()).max())  # (one addition)
    _close(plain[3], dZ.double().sum((0, 2, 3)), 1e-5, "dshift")


@pytest.mark.parametrize("shape", [(2, 256, 4, 12, 256, 64, 3), (3, 256, 6, 10, 512, 128, 1)])
def test_batch_norm_in_the_backward_kernels(shape):
    """Planes that the chain kernel takes forward and not the gradients of its filters: the pixel-major kernels fold the scale in and form the
    shift gradient, in three launches; without a T that was kept other kernels do, to the same results (dT and dVp in bf16 and float,
    the scaled filters are rounded in either case: a share of 2^-8 per rounding)."""
    import paper_2103_03936_amd as pf
    N, C, H, W, Cout, r, k = shape
    g = torch.Generator(device="cuda").manual_seed(14)
    b = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    X, Uk, Vp, dZ = b(N, C, H, W), b(r, C, k, k) * (C * k * k) ** -0.5, b(Cout, r) * r ** -0.5, b(N, Cout, H, W)
    scale = torch.rand(Cout, generator=g, device="cuda") + 0.5
    Y, T, kept = pf.pf_lowrank_conv_fwd_ep(X, Uk, Vp, scale, pad=k // 2, save_W=True)
    pf.timing_reset()
    pf.timing_enable(True)
    one = pf.pf_lowrank_conv_bwd_ep(X, Uk, Vp, scale, dZ, T_saved=T, pad=k // 2, W_saved=kept)
    pf.timing_enable(False)
    assert sorted(n for n in pf.timing_collect()) == ["conv_bwd_px", "conv_wgrad_px", "split_sums"]
    other = pf.pf_lowrank_conv_bwd_ep(X, Uk, Vp, scale, dZ, pad=k // 2)
    h, Vs = lambda t: t.cpu().double(), (Vp.float() * scale[:, None]).bfloat16()
    dT = F.conv2d(h(dZ), h(Vs).t()[:, :, None, None]).bfloat16().double()
    P = (h(dZ) * scale.cpu().double()[:, None, None]).flatten(2)
    want = (torch.nn.grad.conv2d_input(X.shape, h(Uk), dT, padding=k // 2), torch.nn.grad.conv2d_weight(h(X), Uk.shape, dT, padding=k // 2),
            (P @ h(T).flatten(2).transpose(1, 2)).sum(0), h(dZ).sum((0, 2, 3)))
    for got in (one, other):
        for x, ref, what in zip(got, want, ("dX", "dUk", "dVp", "dshift")):
            _close(x.cpu(), ref, 4e-3, f"{shape} {what}")


@pytest.mark.parametrize("shape", [(4, 256, 8, 8, 256, 64, 3), (3, 256, 8, 8, 1024, 128, 1), (28, 512, 8, 8, 256, 128, 1), (33, 512, 5, 9, 2048, 128, 1)])
def test_plain_calls_and_epilogues(shape):
    """Calls without an epilogue may run on another kernel than those with one: the same output, to two roundings of T and Y (2^-9 of a
    value at most each, on either side), and the same factors kept for the backward direction."""
    import paper_2103_03936_amd as pf
    N, C, H, W, Cout, r, k = shape
    g = torch.Generator(device="cuda").manual_seed(11)
    b = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    X, Uk, Vp = b(N, C, H, W), b(r, C, k, k) * (C * k * k) ** -0.5, b(Cout, r) * r ** -0.5
    Y, T, kept = pf.pf_lowrank_conv_fwd(X, Uk, Vp, pad=k // 2, save_W=True)
    Ye, Te, kept_e = pf.pf_lowrank_conv_fwd_ep(X, Uk, Vp, residual=torch.zeros_like(Y), pad=k // 2, save_W=True)
    mid = F.conv2d(X.cpu().float(), Uk.cpu().float(), padding=k // 2)
    ref = F.conv2d(mid.bfloat16().float(), Vp.cpu().float()[:, :, None, None])
    for y, t in ((Y, T), (Ye, Te)):
        _close(t.cpu().float().reshape(mid.shape), mid, 4e-3, "T")
        _close(y.cpu().float(), ref, 4e-3, "Y")
    assert (kept is None) == (kept_e is None) and (kept is None or torch.equal(kept, kept_e))
    dY = b(N, Cout, H, W)
    one = pf.pf_lowrank_conv_bwd(X, Uk, Vp, dY, T_saved=T, pad=k // 2, W_saved=kept)
    other = pf.pf_lowrank_conv_bwd(X, Uk, Vp, dY, T_saved=T, pad=k // 2, W_saved=kept_e)
    assert all(torch.equal(x, y) for x, y in zip(one, other))
