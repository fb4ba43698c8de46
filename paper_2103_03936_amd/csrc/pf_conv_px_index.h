// Index arithmetic of the pixel-major convolution kernels (pf_conv_px.h), for device and host: which pixels a tile needs, where
// they lie in LDS, and which 16-byte pieces of memory hold them.
//
// A tile is a run of pixels of all images laid end to end (pixel = image * H W + y W + x), whatever the plane's size: no column of a
// tile is padding but in the last tile.  In LDS every pixel of the tile and of its halo has a slot (a row of channels); slots follow
// the pixels with a zero column of h slots between rows and h zero rows between images, shared by both neighbours, so that the
// neighbour (dy, dx) of any pixel is always dy (W + h) + dx slots away and a neighbour outside the plane is a zero slot.
#pragma once

#if defined(__HIPCC__)
#define PX_HD __host__ __device__ __forceinline__
#else
#define PX_HD inline
#endif

namespace pf {

// p / d for 0 <= p < 2^31, with m = floor(2^32 / d) (all ones for d = 1): the product is at most one short
inline unsigned px_magic(int d) { return d == 1 ? 0xffffffffu : (unsigned)((1ULL << 32) / (unsigned)d); }
PX_HD int px_div(int p, int d, unsigned m)
{
    const int q = (int)(((unsigned long long)(unsigned)p * m) >> 32);
    return p - q * d >= d ? q + 1 : q;
}

struct PxPlane {
    int N, H, W, HW;
    int h;      // halo: (k - 1) / 2
    int Wp, Hp; // row pitch and rows of an image in slots
    int per;    // groups of eight pixels that a plane needs
    unsigned mW, mHW, mper; // px_div by W, HW, per
    unsigned mwhole, mrest; // ... by HW / 8, the whole groups of a plane, and by HW % 8, the pixels they leave (if any)
};

PX_HD PxPlane px_plane(int N, int H, int W, int k)
{
    PxPlane g;
    g.N = N, g.H = H, g.W = W, g.HW = H * W;
    g.h = (k - 1) / 2;
    g.Wp = W + g.h;
    g.Hp = H + g.h;
    g.per = (g.HW + 7) >> 3;
    g.mW = px_magic(W), g.mHW = px_magic(g.HW), g.mper = px_magic(g.per);
    g.mwhole = px_magic(g.HW >= 8 ? g.HW >> 3 : 1), g.mrest = px_magic(g.HW & 7 ? g.HW & 7 : 1);
    return g;
}

// slot of pixel q of image n (counted from image 0's first zero row)
PX_HD int px_slot(const PxPlane &g, int n, int q)
{
    const int y = px_div(q, g.W, g.mW), x = q - y * g.W;
    return (n * g.Hp + y + g.h) * g.Wp + x + g.h;
}
PX_HD int px_slot(const PxPlane &g, int p)
{
    const int n = px_div(p, g.HW, g.mHW);
    return px_slot(g, n, p - n * g.HW);
}

struct PxTile {
    int p0, p1;      // pixels of the tile
    int pa, pb;      // pixels with the halo
    int base, slots; // first slot, slots
};

PX_HD PxTile px_tile(const PxPlane &g, int p0, int P)
{
    PxTile t;
    t.p0 = p0;
    const int all = g.N * g.HW;
    t.p1 = p0 + P < all ? p0 + P : all;
    const int reach = g.h * (g.Wp + 1), n0 = px_div(p0, g.HW, g.mHW), n1 = px_div(t.p1 - 1, g.HW, g.mHW);
    t.base = px_slot(g, n0, p0 - n0 * g.HW) - reach;
    t.slots = px_slot(g, n1, t.p1 - 1 - n1 * g.HW) + reach - t.base + 1;
    const int back = g.h * (g.W + 1), a = p0 - back, b = t.p1 + back;
    t.pa = a > n0 * g.HW ? a : n0 * g.HW;
    t.pb = b < (n1 + 1) * g.HW ? b : (n1 + 1) * g.HW;
    return t;
}

// Group gi of the tile's pixels: eight neighbours in the plane of image n from q on (whole 16-byte pieces where a plane is a
// multiple of them).  The last group of a plane is pulled back inside it.  False: past the end.
PX_HD bool px_group(const PxPlane &g, const PxTile &t, int gi, int &n, int &q)
{
    if (g.HW % 8 == 0) { // (no group crosses planes)
        const int p = (t.pa & ~7) + 8 * gi;
        n = px_div(p, g.HW, g.mHW);
        q = p - n * g.HW;
        return p < t.pb;
    }
    n = px_div(t.pa, g.HW, g.mHW);
    q = t.pa - n * g.HW;
    const int first = (g.HW - q + 7) >> 3;
    if (gi < first) {
        q += 8 * gi;
    } else {
        const int i = px_div(gi - first, g.per, g.mper);
        n += 1 + i;
        q = 8 * (gi - first - i * g.per);
    }
    if (n * g.HW + q >= t.pb) return false;
    if (q > g.HW - 8) q = g.HW - 8;
    return true;
}
// Where pixel q of image n is when the groups lie in LDS one after the other, eight rows each (any pixel of the tile or its halo).
PX_HD int px_linear(const PxPlane &g, const PxTile &t, int n, int q)
{
    if (g.HW % 8 == 0) return n * g.HW + q - (t.pa & ~7);
    const int n0 = px_div(t.pa, g.HW, g.mHW), q0 = t.pa - n0 * g.HW, first = (g.HW - q0 + 7) >> 3;
    const int qs = n == n0 ? q0 : 0, gi = n == n0 ? 0 : first + (n - n0 - 1) * g.per;
    const int k = (q - qs) >> 3, at = qs + 8 * k, back = at > g.HW - 8 ? at - (g.HW - 8) : 0;
    return (gi + k) * 8 + (q - at) + back;
}
PX_HD int px_groups(const PxPlane &g, const PxTile &t) // how many
{
    if (g.HW % 8 == 0) return (t.pb - (t.pa & ~7) + 7) >> 3;
    const int n0 = px_div(t.pa, g.HW, g.mHW), n1 = px_div(t.pb - 1, g.HW, g.mHW);
    if (n0 == n1) return (t.pb - t.pa + 7) >> 3;
    return ((n0 + 1) * g.HW - t.pa + 7) / 8 + (n1 - n0 - 1) * g.per + (t.pb - n1 * g.HW + 7) / 8;
}

// What leaves a tile: whole groups of eight pixels of one plane, counted from where the tile starts in it, and what is left over of
// every plane.  P / 8 groups and 8 times the planes that a tile touches are upper bounds.
struct PxOut {
    int n0, q0, first, images, last; // first image, its first pixel, pixels of the tile in it, whole images after it, pixels in the one after those
};
PX_HD PxOut px_out(const PxPlane &g, const PxTile &t)
{
    PxOut o;
    o.n0 = px_div(t.p0, g.HW, g.mHW);
    o.q0 = t.p0 - o.n0 * g.HW;
    const int all = t.p1 - t.p0;
    o.first = all < g.HW - o.q0 ? all : g.HW - o.q0;
    o.images = px_div(all - o.first, g.HW, g.mHW);
    o.last = all - o.first - o.images * g.HW;
    return o;
}
PX_HD bool px_out_group(const PxPlane &g, const PxOut &o, int gi, int &n, int &q)
{
    const int f = o.first >> 3;
    if (gi < f) {
        n = o.n0;
        q = o.q0 + 8 * gi;
        return true;
    }
    const int per = g.HW >> 3, i = px_div(gi - f, per, g.mwhole);
    n = o.n0 + 1 + i;
    q = 8 * (gi - f - i * per);
    return i < o.images || (i == o.images && q + 8 <= o.last);
}
PX_HD int px_out_rest(const PxPlane &g, const PxOut &o) { return (o.first & 7) + o.images * (g.HW & 7) + (o.last & 7); }
PX_HD void px_out_pixel(const PxPlane &g, const PxOut &o, int i, int &n, int &q)
{
    const int f = o.first & 7, per = g.HW & 7;
    n = o.n0;
    q = o.q0 + (o.first & ~7) + i;
    if (i < f) return;
    i -= f;
    const int w = per ? px_div(i, per, g.mrest) : o.images;
    if (w < o.images) {
        n += 1 + w;
        q = (g.HW & ~7) + i - w * per;
        return;
    }
    n += 1 + o.images;
    q = (o.last & ~7) + i - o.images * per;
}

// A slot is a row of 64 channels, eight octets of 16 bytes, in an order that keeps apart in the banks: eight consecutive slots read
// at one octet (fragments), four consecutive slots read at two octets (transposing reads) and, in pairs, slots eight apart (stores).
PX_HD int px_swizzle(int slot) { return (((slot & 3) << 1) | (slot >> 2 & 1)) ^ ((slot >> 3 & 3) << 1); }
PX_HD int px_at(int slot, int octet) { return slot * 128 + ((octet ^ px_swizzle(slot)) << 4); } // byte

} // namespace pf
