"""GPU parity of the pixel-major convolution kernels (pf_conv_px.h), every tile size with every rank block, against torch in float32:
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


def _call(f, *args):
    conv = [ctypes.c_void_p(a.data_ptr()) if torch.is_tensor(a) else ctypes.c_void_p(None) if a is None else a for a in args]
    return f(*conv, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))


def _close(got, want, rel, what):
    err = (got.double() - want.double()).norm() / want.double().norm().clamp_min(1e-30)
    assert torch.isfinite(got.float()).all() and err <= rel, f"{what}: {err:.2e} > {rel:.0e}"


@pytest.mark.parametrize("shape", SHAPES)
def test_parity(px, shape):
    """Rounding to bf16 changes an output by a share of 2^-8 = 3.9e-3 at most (1.7e-3 rms over many; the smallest shape has 64 outputs).
    T and dT are rounded before the second stage, here and in the reference; filter gradients add bf16 products in float."""
    N, C, H, W, Cout, r, k = shape
    g = torch.Generator(device="cuda").manual_seed(7)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    b = lambda t: t.bfloat16()
    X, dZ = b(n(N, C, H, W).clamp_min(0)), b(n(N, Cout, H, W))
    Uk, Vp = b(n(r, C, k, k) * (C * k * k) ** -0.5), b(n(Cout, r) * r ** -0.5)
    scale, shift = torch.rand(Cout, generator=g, device="cuda") + 0.5, n(Cout) * 0.2
    res, add = b(n(N, Cout, H, W)), b(n(N, C, H, W))
    T = F.conv2d(X.float(), Uk.float(), padding=k // 2)
    col = lambda v: v[None, :, None, None]
    Vs = b(Vp.float() * scale[:, None]).float()
    dT = F.conv2d(dZ.float(), Vs.t()[:, :, None, None].contiguous())
    dX = torch.nn.grad.conv2d_input(X.shape, Uk.float(), b(dT).float(), padding=k // 2)
    r8, taken = (r + 7) // 8 * 8, 0
    for P, threads in TILES:
        pack = torch.zeros(px.px_pack_size(C, r, k), dtype=torch.bfloat16, device="cuda")
        for ep in (False, True):
            Y, T1 = torch.full_like(res, float("nan")), torch.full((N, r, H, W), float("nan"), dtype=torch.bfloat16, device="cuda")
            st = _call(px.px_fwd, N, C, H, W, Cout, r, k, P, threads, X, Uk, Vp, scale if ep else None, shift if ep else None,
                       res if ep else None, int(ep), Y, T1, pack)
            if st:
                assert st == 100 or (threads == 256 and r > 64), st
                break
            taken += 1
            what = f"{shape} {P} pixels, {threads} threads"
            _close(T1, T, 4e-3, what + " T")
            want = F.conv2d(T1.float(), Vp.float()[:, :, None, None])
            _close(Y, (want * col(scale) + col(shift) + res.float()).clamp_min(0) if ep else want, 4e-3, what + " Y")
            dX1, dT1 = torch.full_like(X, float("nan")), torch.full((N, r8, H, W), float("nan"), dtype=torch.bfloat16, device="cuda")
            assert _call(px.px_bwd, N, C, H, W, Cout, r, k, P, threads, dZ, Vp, pack, scale, add if ep else None, X if ep else None, dX1, dT1) == 0
            _close(dT1[:, :r], dT, 4e-3, what + " dT")
            assert not dT1[:, r:].any()
            _close(dX1, (dX + add.float()) * (X > 0) if ep else dX, 4e-3, what + " dX")
    assert taken >= 6, "most tile sizes take the shape"
    Tb, dTb = b(T).contiguous(), torch.zeros(N, r8, H, W, dtype=torch.bfloat16, device="cuda")
    dTb[:, :r] = b(dT)
    tiles = (N * H * W + 127) // 128
    for per in {1, 3, tiles}:
        groups = (tiles + per - 1) // per
        pU, pV, ps = (torch.full((groups, m), float("nan"), device="cuda") for m in (r * C * k * k, r * Cout, Cout))
        assert _call(px.px_wgrad, N, C, H, W, Cout, r, k, per, dTb, X, Tb, dZ, pU, pV, ps) == 0
        # (sums of some thousand float products at 2^-24 each)
        _close(pU.sum(0).view(r, C, k, k), torch.nn.grad.conv2d_weight(X.double(), Uk.shape, dTb[:, :r].double(), padding=k // 2), 1e-5, f"{shape} dUk")
        _close(pV.sum(0).view(r, Cout).t(), torch.einsum("nop,nrp->or", dZ.flatten(2).double(), Tb.flatten(2).double()), 1e-5, f"{shape} dVp")
        _close(ps.sum(0), dZ.double().sum((0, 2, 3)), 1e-5, f"{shape} sums")


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
        assert _call(px.px_fwd, N, C, H, W, Cout, r, k, P, threads, X, Uk, Vp, None, None, None, 0, Y, T, None) == 0
        want = torch.zeros(H, W, dtype=torch.bool, device="cuda")
        want[3:6, 3:6] = True
        assert (torch.isposinf(Y) == want).all() and torch.isfinite(Y[:, :, ~want]).all(), (P, threads)
