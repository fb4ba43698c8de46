// What the plan of a convolution asks of the pixel-major kernels, and the same by trying everything (test infrastructure, CPU only).
#include "pf_conv_px.h"

using namespace pf;

// every tile
template <typename T>
static bool fit_all(const PxPlaneOf<T> &g, const PxPlaneOf<T> &o, int st, int P, int slots, int groups, bool loose = false)
{
    for (i64 i = 0; i < ((i64)o.N * o.HW + P - 1) / P && i < o.HW; ++i) {
        const PxTile t = px_tile(g, o, st, (int)(i * P), P, loose);
        if (t.slots > slots || px_groups(g, t) > groups) return false;
    }
    return true;
}
// bit 0: the plan's answer, bit 1: by every tile; the filter gradients' in bits 2 and 3
template <typename T>
static int fits(int N, int H, int W, int k, int st, int P)
{
    constexpr int S = PxEl<T>::S, V = PxEl<T>::V;
    const PxPlaneOf<T> g = px_plane<S>(N, H, W, k), o = px_plane<S>(N, (H - 1) / st + 1, (W - 1) / st + 1, 1);
    const int rows = P == 128 || st > 1 ? 256 : P == 64 ? 192 : 160, groups = (P == 32 && st == 1 ? 128 : 256) / V;
    int r = px_tile_fits(g, o, st, P) | fit_all<T>(g, o, st, P, rows - 1, groups) << 1;
    if (st == 1 && P == 128) r |= px_wgrad_fits(g) << 2 | fit_all<T>(g, g, 1, P, 1 << 30, (PX_WG_ROWS - 8) >> S, true) << 3;
    return r;
}
extern "C" int emu_fits(int f32, int N, int H, int W, int k, int st, int P) { return f32 ? fits<float>(N, H, W, k, st, P) : fits<uint16_t>(N, H, W, k, st, P); }

// shapes that the kernels take
extern "C" int emu_takes(int f32, int N, int C, int H, int W, int Cout, int r, int k)
{
    return f32 ? px_fits<float>(N, C, H, W, Cout, r, k, 1, k / 2, H, W) : px_fits<uint16_t>(N, C, H, W, Cout, r, k, 1, k / 2, H, W);
}

// the groups of both filter gradients, and by every number of tiles per group
template <typename T>
static void plan(int npx, int r, int C1, int k, int C2, int *out)
{
    int groups[2], per[2];
    px_wgrad_plan<T>(npx, r, C1, k, C2, groups, per);
    out[0] = groups[0], out[1] = groups[1], out[2] = per[0], out[3] = per[1];
    const int tiles = (npx + 127) / 128, s1 = px_slab<T>(k, r), s2 = px_slab<T>(1, r), u1 = (C1 + s1 - 1) / s1, u2 = (C2 + s2 - 1) / s2;
    const double c1 = px_wgrad_cost<T>(k, r), c2 = px_wgrad_cost<T>(1, r);
    double best = 1e30;
    for (int p1 = 1; p1 <= tiles; ++p1) {
        const int g1 = (tiles + p1 - 1) / p1;
        if (g1 > 1 && u1 * g1 + u2 > 256) continue;
        int p2 = (int)(p1 * c1 / c2);
        p2 = p2 < 1 ? 1 : p2 > tiles ? tiles : p2;
        int g2 = (tiles + p2 - 1) / p2;
        while (g2 > 1 && u1 * g1 + u2 * g2 > 256) p2++, g2 = (tiles + p2 - 1) / p2;
        const double t = (p1 * c1 > p2 * c2 ? p1 * c1 : p2 * c2) + (g1 * (4e-6 * r * C1 * k * k) + g2 * (4e-6 * r * C2)) * 1.5;
        if (t < best) best = t, out[4] = g1, out[5] = g2, out[6] = p1, out[7] = p2;
    }
}
extern "C" void emu_wgrad_plan(int f32, int npx, int r, int C1, int k, int C2, int *out)
{
    if (f32) plan<float>(npx, r, C1, k, C2, out);
    else plan<uint16_t>(npx, r, C1, k, C2, out);
}
