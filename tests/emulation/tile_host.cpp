// The host side of the tiled products (test infrastructure, CPU only).  Built by tests/test_host_tiles.py against the library; nothing
// in the product loads it.
#include "pf_tile_plans.h"

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
    pf_linear_desc d = {};
    d.M = M, d.in = in, d.out = out, d.r = r, d.dtype = dtype;
    const LinearTiles p = make_linear_tiles(&d, 1);
    return backward ? (p.dT_sliced ? p.dT.ksplit : 1) : p.T_sliced ? p.T.ksplit : 1;
}
// whether the streaming kernels take a layer in float, forward (1) and backward (2)
int emu_streamed(long long M, long long in, long long out, long long r)
{
    pf_linear_desc d = {};
    d.M = M, d.in = in, d.out = out, d.r = r, d.dtype = PF_F32;
    bool fwd, bwd;
    linear_skinny_pays(&d, make_linear_tiles(&d, 1), fwd, bwd);
    return fwd + 2 * bwd;
}
// slices of an LSTM cell's T (backward: dT), and whether dx and dh_prev go with the gradients (*one) or all of it backward is on the streaming
// kernels (*skinny)
int emu_cell_slices(long long B, long long din, long long h, long long r, int groups, int backward, int *one, int *skinny)
{
    pf_lstm_desc d = {};
    d.B = B, d.d_in = din, d.h = h, d.r = r, d.groups = groups;
    const LstmTilePlan p = make_lstm_tile_plan(&d);
    *one = p.one, *skinny = lstm_skinny_pays(&d);
    const MidGroup &m = backward ? p.dT : p.T;
    return m.sliced ? m.g.ksplit[0] : 1;
}
// ... and of dTx over all rows of a stack
int emu_tall_slices(long long rows, long long din, long long h, long long r, int groups)
{
    const StackTall t = make_tall(rows, din, h, r, groups);
    return t.dTx.sliced ? t.dTx.t.ksplit : 1;
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
