"""GPU parity of the tiled products (pf_tile.h) at the sizes where they can go wrong: dimensions of one 16-byte piece, tile
edges, rows of odd length (unaligned pieces, the last piece of a row pulled back), contractions split over workgroups,
every tile shape; convolutions whose pixels do not fill their pieces, planes smaller than a piece, stride."""
import pytest

import test_gpu_linear

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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", LINEAR)
def test_linear(shape, dtype):
    test_gpu_linear._run(*shape, dtype=dtype, bias=True, saved_T=shape[0] != 257, seed=21)
