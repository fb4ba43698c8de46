"""GPU parity of the tiled products (pf_tile.h) at the sizes where they can go wrong: dimensions of one 16-byte piece, tile
edges, rows of odd length (unaligned pieces, the last piece of a row pulled back), contractions split over workgroups,
every tile shape; convolutions whose pixels do not fill their pieces, planes smaller than a piece, stride."""
import pytest

import test_gpu_conv
import test_gpu_linear
import test_gpu_linear_shared
import test_gpu_lstm

pytestmark = pytest.mark.gpu

LINEAR = [
    # M, n_in, n_out, r
    (1, 8, 8, 8),
    (129, 9, 8, 15),
    (200, 333, 100, 70),
    (257, 65, 127, 33),
    (1500, 129, 72, 17),     # gradients split over the rows
    (2050, 1032, 1160, 264),  # large tiles with ragged edges
    (160, 517, 260, 37),      # one workgroup per compute unit: chunks of twice the length, the last one nearly empty or not whole
    (130, 2047, 40, 64),
    (300, 255, 1030, 96),
    (282, 3492, 400, 86),     # ... with the contraction split as well (float), into slices of 15 chunks or 7 1/2 long ones
    (96, 4093, 300, 218),     # (both types)
    (300, 256, 256, 250),     # ... and all gradients, with the bias's (float)
    (515, 160, 150, 514),     # (bf16)
    (6337, 500, 264, 128),    # many rows, but too little for the larger tiles of
    (6337, 484, 1030, 128),   # (too much padding for them)
    (6500, 489, 985, 128),    # bf16 gradients on 128 x 128 tiles, two workgroups per compute unit
]

CONV = [
    # N, C, H, W, Cout, r, k, stride, pad
    (3, 9, 7, 5, 17, 10, 3, 2, 1),
    (5, 24, 7, 7, 20, 8, 1, 2, 0),    # three of the four phases of dX are reached by no tap
    (9, 40, 2, 2, 33, 12, 3, 1, 1),
    (5, 16, 1, 1, 16, 8, 3, 1, 1),
    (2, 10, 17, 16, 21, 9, 5, 1, 2),
    (3, 130, 14, 14, 136, 40, 3, 1, 1),
    (70, 64, 8, 8, 200, 36, 3, 2, 1),  # image groups of the filter gradients of unequal length
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", LINEAR)
def test_linear(shape, dtype):
    test_gpu_linear._run(*shape, dtype=dtype, bias=True, saved_T=shape[0] != 257, seed=21)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", CONV)
def test_conv(shape, dtype):
    test_gpu_conv._run(shape, dtype, saved_T=shape[0] != 5, seed=22)


@pytest.mark.parametrize("groups", [1, 4])
@pytest.mark.parametrize("shape", [(33, 9, 5, 4), (70, 41, 38, 9), (130, 700, 644, 161)])
def test_lstm_cell(shape, groups):
    test_gpu_lstm._cell(*shape, groups, seed=23)


@pytest.mark.parametrize("shape", [(9, 2224, 2816, 970), (1, 2051, 1030, 515), (32, 4001, 4098, 1029)])
def test_linear_streamed(shape):
    """Few rows in float whose factors are streamed in one direction or both (tests/test_host_tiles.py: these are)."""
    test_gpu_linear._run(*shape, dtype="f32", bias=True, saved_T=shape[0] != 1, seed=29)


@pytest.mark.parametrize("groups", [1, 4])
@pytest.mark.parametrize("shape", [(1, 515, 260, 65), (20, 700, 516, 129), (33, 1030, 900, 225), (3, 1302, 1360, 341), (64, 70, 1500, 375)])
def test_lstm_cell_slices(shape, groups):
    """Slices of T and dT that their readers add, dx and dh_prev beside the gradients and in a launch of their own; the fourth one's
    backward direction with a pair per gate is on the streaming kernels."""
    test_gpu_lstm._cell(*shape, groups, seed=27)


@pytest.mark.parametrize("shape,groups", [((4, 1024, 1024, 453), 1), ((1, 515, 1400, 402), 1), ((3, 130, 1033, 290), 4), ((17, 1100, 1499, 391), 4)])
def test_lstm_cell_streamed(shape, groups):
    """Few rows whose factors backward are streamed, one pair and a pair per gate (tests/test_host_tiles.py: these are)."""
    test_gpu_lstm._cell(*shape, groups, seed=28)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(33, 9, 10, 8, 2), (20, 24, 1500, 16, 3), (700, 130, 41, 24, 4), (6100, 264, 130, 128, 3),
                                   (6100, 264, 330, 128, 3), (6100, 380, 378, 128, 3)])
def test_linear_shared(shape, dtype):
    """The second one splits the contraction of dT, whose layers then lie one after the other instead of side by side; the last one's
    bf16 gradients are on 128 x 128 tiles, of which none is shared by two layers."""
    test_gpu_linear_shared._run(*shape, dtype=dtype, saved_T=shape[0] != 700, seed=24)


# Intermediates in slices that their readers add up (tests/test_host_tiles.py: which of these have them, and how many): one row to
# just past a tile of them, ranks of one piece to several chunks, rows of slices that no piece divides.
SLICED = [(1, 1030, 517, 97), (31, 2047, 1021, 181), (33, 640, 1280, 8), (65, 1000, 1064, 250), (128, 1152, 256, 116), (250, 704, 832, 181)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("saved_T", [True, False])
@pytest.mark.parametrize("shape", SLICED)
def test_linear_slices(shape, saved_T, dtype):
    test_gpu_linear._run(*shape, dtype=dtype, bias=True, saved_T=saved_T, seed=25)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(33, 1000, 1064, 40, 3), (20, 1500, 1504, 16, 2)])
def test_linear_shared_slices(shape, dtype):
    test_gpu_linear_shared._run(*shape, dtype=dtype, saved_T=True, seed=26)


def test_bias_gradient_of_many_rows():
    """Float sums over 16384 rows of zero mean, unsplit.  Chains of n additions of such terms are off by about 2^-24 sqrt(n / 6)
    of the sum, rms: 2^-22 for runs of at most 96 rows, which the thousands of one thread's single chain would miss."""
    import torch
    import paper_2103_03936_amd as pf
    g = torch.Generator(device="cuda").manual_seed(5)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    X, V, U, dY = n(16384, 1024), n(1024, 250) * 0.05, n(1000, 250) * 0.05, n(16384, 1000)
    db = pf.pf_lowrank_linear_bwd(X, V, U, dY, has_bias=True)[3].double()
    want = dY.double().sum(0)
    assert float((db - want).norm() / want.norm()) <= 2.0 ** -22


def _rel(got, want):
    return float((got.double() - want).norm() / want.norm())


# Where one layer or several go from the chain kernel to the tiled products or back.  bf16: the rank-r intermediate and the
# output are rounded (2^-9 / sqrt(3) rms each, and what the first carries into the second): 2^-9 sqrt(3) bounds them together.
ROUNDED = 2.0 ** -9 * 3 ** 0.5


@pytest.mark.parametrize("M,n_in,n_out,r", [
    (4095, 512, 2048, 128), (4096, 512, 2048, 128), (8192, 512, 256, 128), (8193, 512, 256, 128), (8193, 768, 256, 128),
    (4096, 1024, 512, 128), (4999, 256, 256, 128), (5000, 256, 256, 128), (10001, 256, 256, 128), (10000, 256, 256, 64),
    (16385, 256, 256, 64), (24001, 512, 256, 64),
    # the kernel for few rows, one row to the last that it takes and one more: both sides of every contraction length
    (1, 256, 256, 128), (32, 512, 512, 128), (65, 768, 256, 128), (129, 1024, 512, 128), (2048, 512, 512, 128), (2049, 512, 512, 128),
    (31, 1280, 256, 128), (256, 1024, 4096, 128),
    # the chain kernel's loops: a ragged last row tile, one to eight pairs of output blocks, any number of them, ten chunks
    (33, 256, 256, 128), (4129, 768, 1024, 128), (4129, 1024, 768, 128), (5003, 1280, 1280, 128), (4129, 2048, 512, 128)])
@pytest.mark.parametrize("saved_T", [True, False])
def test_linear_routes(M, n_in, n_out, r, saved_T):
    import torch
    import paper_2103_03936_amd as pf
    g = torch.Generator(device="cuda").manual_seed(M)
    n = lambda *s, std=1.0: (torch.randn(s, generator=g, device="cuda") * std).to(torch.bfloat16)
    X, V, U, dY, b = n(M, n_in), n(n_in, r, std=n_in ** -0.5), n(n_out, r, std=r ** -0.5), n(M, n_out), n(n_out)
    Y, T = pf.pf_lowrank_linear_fwd(X, V, U, b)
    dX, dU, dV, db = pf.pf_lowrank_linear_bwd(X, V, U, dY, T_saved=T if saved_T else None, has_bias=True)
    x, v, u, dy = (t.double() for t in (X, V, U, dY))
    t, dt = x @ v, dy @ u
    for name, got, want in (("Y", Y, t @ u.t() + b.double()), ("T", T, t), ("dX", dX, dt @ v.t()), ("dU", dU, dy.t() @ t),
                            ("dV", dV, x.t() @ dt), ("db", db, dy.sum(0))):
        assert _rel(got, want) <= ROUNDED, name


@pytest.mark.parametrize("G,M,n_in,n_out", [(3, 8192, 256, 512), (3, 8193, 256, 512), (2, 4096, 1024, 256), (2, 4097, 1024, 256),
                                            (8, 33, 512, 256), (9, 33, 512, 256), (3, 682, 768, 512), (3, 704, 512, 512)])
def test_linear_shared_routes(G, M, n_in, n_out):
    import torch
    import paper_2103_03936_amd as pf
    r, g = 128, torch.Generator(device="cuda").manual_seed(M + G)
    n = lambda *s, std=1.0: (torch.randn(s, generator=g, device="cuda") * std).to(torch.bfloat16)
    X, V, U, dY, b = n(M, n_in), n(G, n_in, r, std=n_in ** -0.5), n(G, n_out, r, std=r ** -0.5), n(G, M, n_out), n(G, n_out)
    Y, T = pf.pf_lowrank_linear_shared_fwd(X, V, U, b)
    dX, dU, dV, db = pf.pf_lowrank_linear_shared_bwd(X, V, U, dY, T_saved=T, has_bias=True)
    x, total = X.double(), 0
    for k in range(G):
        v, u, dy = (t[k].double() for t in (V, U, dY))
        t, dt = x @ v, dy @ u
        total = total + dt @ v.t()
        for name, got, want in (("Y", Y, t @ u.t() + b[k].double()), ("T", T, t), ("dU", dU, dy.t() @ t), ("dV", dV, x.t() @ dt),
                                ("db", db, dy.sum(0))):
            assert _rel(got[k], want) <= ROUNDED, name
    assert _rel(dX, total) <= ROUNDED


@pytest.mark.parametrize("M,n_in,n_out", [(33, 256, 512), (47, 1024, 256), (4129, 1024, 512), (4129, 1024, 768), (5003, 1280, 1280), (4129, 512, 2048)])
def test_linear_routes_epilogue(M, n_in, n_out):
    """Residual and ReLU forward, skip gradient and mask backward, where the chain kernel applies them and where tiles do; an
    output that the chain kernel adds to is rounded twice."""
    import torch
    import paper_2103_03936_amd as pf
    r, g = 128, torch.Generator(device="cuda").manual_seed(M)
    n = lambda *s, std=1.0: (torch.randn(s, generator=g, device="cuda") * std).to(torch.bfloat16)
    X, V, U, dZ, b = n(M, n_in).clamp_(min=0), n(n_in, r, std=n_in ** -0.5), n(n_out, r, std=r ** -0.5), n(M, n_out), n(n_out)
    R, skip = n(M, n_out), n(M, n_in)
    Y, T = pf.pf_lowrank_linear_fwd_ep(X, V, U, b, residual=R, act="relu")
    dX = pf.pf_lowrank_linear_bwd_ep(X, V, U, dZ, T_saved=T, dX_add=skip, x_is_relu=True, has_bias=True)[0]
    x, v, u, dz = (t.double() for t in (X, V, U, dZ))
    assert _rel(Y, (x @ v @ u.t() + b.double() + R.double()).clamp(min=0)) <= ROUNDED
    assert _rel(dX, (dz @ u @ v.t() + skip.double()) * (x > 0)) <= ROUNDED


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(3, 20, 16, 16, 24, 12, 3), (5, 9, 8, 24, 12, 8, 3), (2, 70, 12, 8, 16, 40, 3), (3, 12, 7, 9, 16, 8, 3),
                                   (2, 16, 10, 6, 16, 8, 5), (1, 12, 2, 8, 12, 8, 3), (2, 16, 32, 4, 16, 8, 1),
                                   (3, 20, 16, 16, 24, 12, 2, 0), (5, 9, 6, 8, 12, 8, 2, 0), (2, 70, 10, 24, 16, 40, 4, 1), (3, 12, 9, 17, 16, 8, 2, 0)])
def test_strided_conv_epilogue(shape, dtype):
    """Stride 2, input read by pairs of loads and the even and odd pixels of dX in one workgroup where rows hold whole pieces, and
    where they do not; even filters, whose padding is no half of them; skip gradient and mask against the plain gradient: the same sums, added to and masked before one rounding."""
    import torch
    import paper_2103_03936_amd as pf
    N, C, H, W, Cout, r, k, *p = shape
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    g = torch.Generator(device="cuda").manual_seed(H * W + k)
    n = lambda *s, std=1.0: (torch.randn(s, generator=g, device="cuda") * std).to(dt)
    pad = p[0] if p else k // 2
    Ho, Wo = (H + 2 * pad - k) // 2 + 1, (W + 2 * pad - k) // 2 + 1
    X, Uk, Vp, dY, add = n(N, C, H, W).clamp_(min=0), n(r, C, k, k, std=(C * k * k) ** -0.5), n(Cout, r, std=r ** -0.5), n(N, Cout, Ho, Wo), n(N, C, H, W)
    Y, T = pf.pf_lowrank_conv_fwd(X, Uk, Vp, 2, pad)
    want_T = torch.nn.functional.conv2d(X.double().cpu(), Uk.double().cpu(), stride=2, padding=pad)
    # T: float sums of C k k terms, or rounded to bf16
    assert _rel(T.cpu(), want_T) <= (2.0 ** -20 if dtype == "f32" else ROUNDED)
    dX = pf.pf_lowrank_conv_bwd(X, Uk, Vp, dY, T_saved=T, stride=2, pad=pad)[0]
    got = pf.pf_lowrank_conv_bwd_ep(X, Uk, Vp, None, dY, T_saved=T, stride=2, pad=pad, dX_add=add, x_is_relu=True)[0]
    want = torch.where(X > 0, dX.float() + add.float(), torch.zeros((), device="cuda"))
    if dtype == "f32":
        assert torch.equal(got, want)
    else:
        assert _rel(got, want.double()) <= ROUNDED
    ref = torch.nn.grad.conv2d_input((N, C, H, W), Uk.double().cpu(), torch.einsum("or,nohw->nrhw", Vp.double().cpu(), dY.double().cpu()),
                                     stride=2, padding=pad)
    assert _rel(dX.cpu(), ref) <= (2.0 ** -20 if dtype == "f32" else ROUNDED)


@pytest.mark.parametrize("n_in,r,n_out,M,more", [(320, 128, 128, 20000, 24000), (1000, 128, 256, 7500, 7900), (640, 128, 768, 11000, 11500)])
def test_fewer_rows_take_no_longer(n_in, r, n_out, M, more):
    """bf16 backward: large tiles that left compute units waiting took 1.3 to 1.7 times as long for the smaller numbers of rows."""
    import torch
    import paper_2103_03936_amd as pf
    g = torch.Generator(device="cuda").manual_seed(9)
    n = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)

    def best(rows):
        X, V, U, dY, T = n(rows, n_in), n(n_in, r), n(n_out, r), n(rows, n_out), n(rows, r)
        times = []
        for _ in range(6):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            for _ in range(10):
                pf.pf_lowrank_linear_bwd(X, V, U, dY, T_saved=T, has_bias=True)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        return min(times[1:])

    assert best(M) <= 1.1 * best(more)
