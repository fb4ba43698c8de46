// The pixel-major convolution kernels by tile size (test infrastructure).  Built by tests/test_gpu_conv_px.py against the library, whose
// own calls choose the tile.
#include "pf_conv_px.h"

using namespace pf;

template <typename T>
static PxPlaneOf<T> plane(int N, int H, int W, int k) { return px_plane<PxEl<T>::S>(N, H, W, k); }

// 0: launched; 100: the kernels do not take the shape with this tile
template <typename T>
static int fwd(int N, int C, int H, int W, int Cout, int r, int k, int st, int P, int threads, T *X, T *Uk, T *Vp, float *scale, float *shift, T *residual,
               int relu, T *Y, T *mid, T *pack, hipStream_t s)
{
    const int Ho = (H - 1) / st + 1, Wo = (W - 1) / st + 1;
    const PxPlaneOf<T> g = plane<T>(N, H, W, k), o = plane<T>(N, Ho, Wo, 1);
    if (!px_fits<T>(N, C, H, W, Cout, r, k, st, k / 2, Ho, Wo) || !px_tile_fits(g, o, st, P)) return 100;
    return launch_px_fwd(s, PxFwdArgs<T>{g, o, st, C, Cout, r, X, Uk, Vp, Y, mid, {scale, shift, residual, nullptr, relu},
                                         {Uk, pack, C, r, k * k}, {}, {}}, k, P, threads);
}
template <typename T>
static int bwd(int N, int C, int H, int W, int Cout, int r, int k, int P, int threads, T *dZ, T *Vp, T *pack, float *scale, T *add, T *mask, T *dX,
               T *dT, hipStream_t s)
{
    return launch_px_bwd(s, PxBwdArgs<T>{plane<T>(N, H, W, k), C, Cout, r, dZ, Vp, pack, dX, dT, scale, {nullptr, nullptr, add, mask, 0}}, k, P, threads);
}
// partial sums [groups][r][C][k k] and [groups][r][Cout] (and of dZ [groups][Cout]) over groups of `per` tiles
template <typename T>
static int wgrad(int N, int C, int H, int W, int Cout, int r, int k, int per, T *dT, T *X, T *mid, T *dZ, float *partU, float *partV, float *sums,
                 hipStream_t s)
{
    const PxPlaneOf<T> g = plane<T>(N, H, W, k);
    if (!px_wgrad_fits(g)) return 100;
    const int tiles = (N * H * W + 127) / 128, groups = (tiles + per - 1) / per, s1 = px_slab<T>(k, r), s2 = px_slab<T>(1, r);
    return launch_px_wgrad(s, PxWgradArgs<T>{plane<T>(N, H, W, 1), g, r, 2,
                                             {{dT, X, px_ranks<T>(r), C, k * k, (C + s1 - 1) / s1, groups, per, partU, nullptr},
                                              {mid, dZ, r, Cout, 1, (Cout + s2 - 1) / s2, groups, per, partV, sums}}});
}

#define ENTRIES(T, name) \
    extern "C" int px_fwd_##name(int N, int C, int H, int W, int Cout, int r, int k, int st, int P, int threads, T *X, T *Uk, T *Vp, float *scale, \
                                 float *shift, T *residual, int relu, T *Y, T *mid, T *pack, hipStream_t s) \
    { return fwd<T>(N, C, H, W, Cout, r, k, st, P, threads, X, Uk, Vp, scale, shift, residual, relu, Y, mid, pack, s); } \
    extern "C" int px_bwd_##name(int N, int C, int H, int W, int Cout, int r, int k, int P, int threads, T *dZ, T *Vp, T *pack, float *scale, \
                                 T *add, T *mask, T *dX, T *dT, hipStream_t s) \
    { return bwd<T>(N, C, H, W, Cout, r, k, P, threads, dZ, Vp, pack, scale, add, mask, dX, dT, s); } \
    extern "C" int px_wgrad_##name(int N, int C, int H, int W, int Cout, int r, int k, int per, T *dT, T *X, T *mid, T *dZ, float *partU, \
                                   float *partV, float *sums, hipStream_t s) \
    { return wgrad<T>(N, C, H, W, Cout, r, k, per, dT, X, mid, dZ, partU, partV, sums, s); }
ENTRIES(uint16_t, bf16)
ENTRIES(float, f32)
extern "C" size_t px_pack_size(int C, int r, int k) { return px_pack_elems(C, r, k); }
