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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(33, 9, 10, 8, 2), (20, 24, 1500, 16, 3), (700, 130, 41, 24, 4)])
def test_linear_shared(shape, dtype):
    """The middle one splits the contraction of dT, whose layers then lie one after the other instead of side by side."""
    test_gpu_linear_shared._run(*shape, dtype=dtype, saved_T=shape[0] != 700, seed=24)


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
