// The host side of the tiled products (test infrastructure, CPU only).  Built by tests/test_host_tiles.py against the library; nothing
// in the product loads it.
#include "pf_tile_host.h"

using namespace pf;

extern "C" {
// status of a convolution launch, with tiles of the given shape, whose two products are the even and the odd pixels of rows
int emu_pair(int dtype, int shape, int wg)
{
    TileArgs a = {};
    for (int i = 0; i < 2; ++i) {
        TileProb q = tile_prob(TILE_CONV, 32, 64, 64, nullptr, 64, nullptr, 0, nullptr, 0);
        q.pb.ntap = 1;
        tile_add(a, (TileShape)shape, dtype, q, 1);
    }
    tile_pair(a);
    return launch_tiles_conv(nullptr, "pair", dtype, (TileShape)shape, (TileShape)wg, a);
}

// tile shape of a product [M][K] [K][N] of which the plan may split the contraction, and the split
int emu_plan(int dtype, long long M, long long N, long long K, int max_split, int *split)
{
    const TilePlan p = plan_tiles(dtype, M, N, K, max_split);
    *split = p.ksplit;
    return p.shape;
}
// slices of the intermediate T (backward: dT) of a layer [M][in] -> r -> out that its readers add up, 1: none
int emu_slices(int dtype, long long M, long long in, long long out, long long r, int backward)
{
    const TileNeed need[3] = {{M, in, r, false}, {out, r, M, true, true}, {in, r, M, true, true}};
    const TileShape reader = backward ? plan_tile_group(dtype, need, 3).shape : plan_tiles(dtype, M, out, r, 1).shape;
    const long long rows = (M + 31) / 32 * 32, ins = (in + 31) / 32, outs = (out + 31) / 32;
    const MidPlan p = backward ? plan_mid(dtype, M, r, out, 16, reader, 8 * ins * rows * r, 128 * (M > r ? M : r))
                               : plan_mid(dtype, M, r, in, 16, reader, 4 * outs * rows * r, 128 * r);
    return p.sliced ? p.t.ksplit : 1;
}
// the same for the gradients of a layer [M][in] -> r -> out in one launch (dX, dU, dV)
int emu_gradients(int dtype, long long M, long long in, long long out, long long r, int *split)
{
    const TileNeed need[3] = {{M, in, r, false}, {out, r, M, true, true}, {in, r, M, true, true}};
    const TileGroup g = plan_tile_group(dtype, need, 3);
    for (int i = 0; i < 3; ++i) split[i] = g.ksplit[i];
    return g.shape;
}
}
