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
}
