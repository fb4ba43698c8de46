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

// Planes of N images; pixels come in groups of 2^S, what a 16-byte piece of a plane holds.
template <int S>
struct PxPlane {
    static constexpr int V = 1 << S;
    int N, H, W, HW;
    int h;      // halo: (k - 1) / 2
    int Wp, Hp; // row pitch and rows of an image in slots
    int per;    // groups that a plane needs
    unsigned mW, mHW, mper; // px_div by W, HW, per
    unsigned mwhole, mrest; // ... by HW / V, the whole groups of a plane, and by HW % V, the pixels they leave (if any)
};

template <int S>
PX_HD PxPlane<S> px_plane(int N, int H, int W, int k)
{
    PxPlane<S> g;
    constexpr int V = 1 << S;
    g.N = N, g.H = H, g.W = W, g.HW = H * W;
    g.h = (k - 1) / 2;
    g.Wp = W + g.h;
    g.Hp = H + g.h;
    g.per = (g.HW + V - 1) >> S;
    g.mW = px_magic(W), g.mHW = px_magic(g.HW), g.mper = px_magic(g.per);
    g.mwhole = px_magic(g.HW >= V ? g.HW >> S : 1), g.mrest = px_magic(g.HW & (V - 1) ? g.HW & (V - 1) : 1);
    return g;
}

// slot of pixel q of image n (counted from image 0's first zero row)
template <int S>
PX_HD int px_slot(const PxPlane<S> &g, int n, int q)
{
    const int y = px_div(q, g.W, g.mW), x = q - y * g.W;
    return (n * g.Hp + y + g.h) * g.Wp + x + g.h;
}
template <int S>
PX_HD int px_slot(const PxPlane<S> &g, int p)
{
    const int n = px_div(p, g.HW, g.mHW);
    return px_slot(g, n, p - n * g.HW);
}

struct PxTile {
    int p0, p1;      // pixels of the tile
    int pa, pb;      // pixels with the halo: from the first to the last that a tap reaches, all of which have slots (px_tile: or one more)
    int base, slots; // first slot, slots
};

// P pixels of the output planes `o` of a convolution with stride `st` over planes `g`, and what they need of those.
template <int S>
PX_HD int px_slot(const PxPlane<S> &g, const PxPlane<S> &o, int st, int p)
{
    const int n = px_div(p, o.HW, o.mHW), q = p - n * o.HW, y = px_div(q, o.W, o.mW), x = q - y * o.W;
    return (n * g.Hp + y * st + g.h) * g.Wp + x * st + g.h;
}
// `loose`: where the tile starts or ends a row, one more pixel each that no tap reaches and that has no slot, for kernels that
// keep no slots: they then need no columns (filter gradients, 0.2 of 22.4 us).
template <int S>
PX_HD PxTile px_tile(const PxPlane<S> &g, const PxPlane<S> &o, int st, int p0, int P, bool loose = false)
{
    PxTile t;
    t.p0 = p0;
    const int all = o.N * o.HW;
    t.p1 = p0 + P < all ? p0 + P : all;
    const int reach = g.h * (g.Wp + 1), back = g.h * (g.W + 1);
    const int n0 = px_div(p0, o.HW, o.mHW), q0 = p0 - n0 * o.HW, y0 = px_div(q0, o.W, o.mW), x0 = q0 - y0 * o.W;
    const int n1 = px_div(t.p1 - 1, o.HW, o.mHW), q1 = t.p1 - 1 - n1 * o.HW, y1 = px_div(q1, o.W, o.mW), x1 = q1 - y1 * o.W;
    t.base = (n0 * g.Hp + y0 * st + g.h) * g.Wp + x0 * st + g.h - reach;
    t.slots = (n1 * g.Hp + y1 * st + g.h) * g.Wp + x1 * st + g.h + reach - t.base + 1;
    // (left and right of a row lie zero slots, not the rows beside it)
    const int a = y0 * st * g.W + x0 * st - back + (x0 == 0 && !loose ? g.h : 0), b = y1 * st * g.W + x1 * st + 1 + back - (x1 * st + 1 == g.W && !loose ? g.h : 0);
    t.pa = n0 * g.HW + (a > 0 ? a : 0);
    t.pb = n1 * g.HW + (b < g.HW ? b : g.HW);
    return t;
}
template <int S>
PX_HD PxTile px_tile(const PxPlane<S> &g, int p0, int P, bool loose = false) { return px_tile(g, g, 1, p0, P, loose); }

// Group gi of the tile's pixels: neighbours in the plane of image n from q on (whole 16-byte pieces where a plane is a
// multiple of them).  The last group of a plane is pulled back inside it.  False: past the end.
template <int S>
PX_HD bool px_group(const PxPlane<S> &g, const PxTile &t, int gi, int &n, int &q)
{
    constexpr int V = 1 << S;
    if (g.HW % V == 0) { // (no group crosses planes)
        const int p = (t.pa & ~(V - 1)) + V * gi;
        n = px_div(p, g.HW, g.mHW);
        q = p - n * g.HW;
        return p < t.pb;
    }
    n = px_div(t.pa, g.HW, g.mHW);
    q = t.pa - n * g.HW;
    const int first = (g.HW - q + V - 1) >> S;
    if (gi < first) {
        q += V * gi;
    } else {
        const int i = px_div(gi - first, g.per, g.mper);
        n += 1 + i;
        q = V * (gi - first - i * g.per);
    }
    if (n * g.HW + q >= t.pb) return false;
    if (q > g.HW - V) q = g.HW - V;
    return true;
}
// Where pixel q of image n is when the groups lie in LDS one after the other, V rows each (any pixel of the tile or its halo).
template <int S>
PX_HD int px_linear(const PxPlane<S> &g, const PxTile &t, int n, int q)
{
    constexpr int V = 1 << S;
    if (g.HW % V == 0) return n * g.HW + q - (t.pa & ~(V - 1));
    const int n0 = px_div(t.pa, g.HW, g.mHW), q0 = t.pa - n0 * g.HW, first = (g.HW - q0 + V - 1) >> S;
    const int qs = n == n0 ? q0 : 0, gi = n == n0 ? 0 : first + (n - n0 - 1) * g.per;
    const int k = (q - qs) >> S, at = qs + V * k, back = at > g.HW - V ? at - (g.HW - V) : 0;
    return (gi + k) * V + (q - at) + back;
}
template <int S>
PX_HD int px_groups(const PxPlane<S> &g, const PxTile &t) // how many
{
    constexpr int V = 1 << S;
    if (g.HW % V == 0) return (t.pb - (t.pa & ~(V - 1)) + V - 1) >> S;
    const int n0 = px_div(t.pa, g.HW, g.mHW), n1 = px_div(t.pb - 1, g.HW, g.mHW);
    if (n0 == n1) return (t.pb - t.pa + V - 1) >> S;
    return (((n0 + 1) * g.HW - t.pa + V - 1) >> S) + (n1 - n0 - 1) * g.per + ((t.pb - n1 * g.HW + V - 1) >> S);
}

// What leaves a tile: whole groups of one plane, counted from where the tile starts in it, and what is left over of
// every plane.  P / V groups and V times the planes that a tile touches are upper bounds.
struct PxOut {
    int n0, q0, first, images, last; // first image, its first pixel, pixels of the tile in it, whole images after it, pixels in the one after those
};
template <int S>
PX_HD PxOut px_out(const PxPlane<S> &g, const PxTile &t)
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
template <int S>
PX_HD bool px_out_group(const PxPlane<S> &g, const PxOut &o, int gi, int &n, int &q)
{
    constexpr int V = 1 << S;
    const int f = o.first >> S;
    if (gi < f) {
        n = o.n0;
        q = o.q0 + V * gi;
        return true;
    }
    const int per = g.HW >> S, i = px_div(gi - f, per, g.mwhole);
    n = o.n0 + 1 + i;
    q = V * (gi - f - i * per);
    return i < o.images || (i == o.images && q + V <= o.last);
}
template <int S>
PX_HD int px_out_rest(const PxPlane<S> &g, const PxOut &o)
{
    constexpr int V = 1 << S;
    return (o.first & (V - 1)) + o.images * (g.HW & (V - 1)) + (o.last & (V - 1));
}
template <int S>
PX_HD void px_out_pixel(const PxPlane<S> &g, const PxOut &o, int i, int &n, int &q)
{
    constexpr int V = 1 << S;
    const int f = o.first & (V - 1), per = g.HW & (V - 1);
    n = o.n0;
    q = o.q0 + (o.first & ~(V - 1)) + i;
    if (i < f) return;
    i -= f;
    const int w = per ? px_div(i, per, g.mrest) : o.images;
    if (w < o.images) {
        n += 1 + w;
        q = (g.HW & ~(V - 1)) + i - w * per;
        return;
    }
    n += 1 + o.images;
    q = (o.last & ~(V - 1)) + i - o.images * per;
}

// A slot is a row of 128 bytes, eight pieces of 16 (64 channels in bf16, 32 in float), in an order that keeps apart in the banks: eight
// consecutive slots read at one piece (fragments), four at two pieces (transposing reads) and, in pairs, slots eight apart (stores).
PX_HD int px_swizzle(int slot) { return (((slot & 3) << 1) | (slot >> 2 & 1)) ^ ((slot >> 3 & 3) << 1); }
PX_HD int px_at(int slot, int piece) { return slot * 128 + ((piece ^ px_swizzle(slot)) << 4); } // byte

} // namespace pf
