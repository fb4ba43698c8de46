// The pixel-major convolution kernels by tile size (test infrastructure).  Built by tests/test_gpu_conv_px.py against the library, whose
// own calls choose the tile.
#include "pf_conv_px.h"

using namespace pf;
typedef uint16_t *u16;

// 0: launched; 100: the kernels do not take the shape with this tile
extern "C" int px_fwd(int N, int C, int H, int W, int Cout, int r, int k, int P, int threads, u16 X, u16 Uk, u16 Vp, float *scale, float *shift,
                      u16 residual, int relu, u16 Y, u16 T, u16 pack, hipStream_t s)
{
    if (!px_fits(N, C, H, W, Cout, r, k, 1, k / 2, H, W) || !px_tile_fits(px_plane(N, H, W, k), P)) return 100;
    return launch_px_fwd(s, PxFwdArgs{px_plane(N, H, W, k), C, Cout, r, X, Uk, Vp, Y, T, {scale, shift, residual, nullptr, relu},
                                      {Uk, pack, C, r, k * k}, {}, {}}, k, P, threads);
}
extern "C" int px_bwd(int N, int C, int H, int W, int Cout, int r, int k, int P, int threads, u16 dZ, u16 Vp, u16 pack, float *scale, u16 add, u16 mask,
                      u16 dX, u16 dT, hipStream_t s)
{
    return launch_px_bwd(s, PxBwdArgs{px_plane(N, H, W, k), C, Cout, r, dZ, Vp, pack, dX, dT, scale, {nullptr, nullptr, add, mask, 0}}, k, P, threads);
}
// partial sums [groups][r][C][k k] and [groups][r][Cout] (and of dZ [groups][Cout]) over groups of `per` tiles
extern "C" int px_wgrad(int N, int C, int H, int W, int Cout, int r, int k, int per, u16 dT, u16 X, u16 T, u16 dZ, float *partU, float *partV, float *sums,
                        hipStream_t s)
{
    const PxPlane g = px_plane(N, H, W, k);
    if (!px_wgrad_fits(g)) return 100;
    const int tiles = (N * H * W + 127) / 128, groups = (tiles + per - 1) / per, r8 = (r + 7) / 8 * 8;
    return launch_px_wgrad(s, PxWgradArgs{px_plane(N, H, W, 1), g, r, 2,
                                          {{dT, X, r8, C, k * k, (C + px_slab(k, r) - 1) / px_slab(k, r), groups, per, partU, nullptr},
                                           {T, dZ, r, Cout, 1, (Cout + 127) / 128, groups, per, partV, sums}}});
}
extern "C" size_t px_pack_size(int C, int r, int k) { return px_pack_elems(C, r, k); }
