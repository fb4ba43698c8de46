"""GPU parity of the two-stage forward kernel (pf_linear_two.h) with every number of rows per workgroup, against torch in float32: widths
and ranks beside their tiles, one row, layers that share their input, outputs shared by several workgroups."""
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
    return ctypes.CDLL(out).linear_two


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
                st = two(ctypes.c_longlong(M), K, N, r, G, rows, osplit, *map(p, args), int(ep), p(Y), p(T),
                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
                assert st == 0
                want = T.float() @ U.float().transpose(1, 2).contiguous()
                if ep:
                    want = (want + bias.float()[:, None] + (add.float() if G == 1 else 0)).clamp_min(0)
                for got, ref in ((T, X.float() @ V.float()), (Y, want)):
                    err = (got.double() - ref.double()).norm() / ref.double().norm().clamp_min(1e-30)
                    assert err <= 4e-3, (rows, osplit, ep, err)
