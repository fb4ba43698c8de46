// The index arithmetic of the pixel-major convolutions (test infrastructure, CPU only; plain C++).
#include "pf_conv_px_index.h"

#include <vector>

using namespace pf;

// Every tile of P output pixels (groups of 2^S) of N planes H x W under k x k taps with stride st, with room for `rows` slots and `groups` groups.  0: right; else what is not.
template <int S>
static int tiles(int N, int H, int W, int k, int st, int P, int rows, int groups)
{
    const PxPlane<S> g = px_plane<S>(N, H, W, k), go = st == 1 ? g : px_plane<S>(N, (H - 1) / st + 1, (W - 1) / st + 1, 1);
    constexpr int V = 1 << S;
    const int all = N * go.HW;
    for (int p0 = 0; p0 < all; p0 += P) {
        const PxTile t = px_tile(g, go, st, p0, P);
        if (t.slots <= 0 || t.slots >= rows) return 1;
        std::vector<int> holds(rows, -1); // pixel in every slot
        int gi = 0, n, q;
        for (; px_group(g, t, gi, n, q); ++gi) {
            if (gi >= groups) return 2;
            if (n < 0 || n >= N || q < 0 || q + V > g.HW) return 3; // a load outside its plane
            if (g.HW % V == 0 && q % V) return 4;
            for (int e = 0; e < V; ++e) {
                const int s = px_slot(g, n, q + e) - t.base;
                if (s < 0 || s >= t.slots) continue;
                const int p = n * g.HW + q + e;
                if (holds[s] >= 0 && holds[s] != p) return 5; // two pixels in one slot
                holds[s] = p;
            }
        }
        if (gi != px_groups(g, t)) return 13;
        for (; gi < groups; ++gi)
            if (px_group(g, t, gi, n, q)) return 6;
        for (int p = t.p0; p < t.p1; ++p)
            for (int dy = -g.h; dy <= g.h; ++dy)
                for (int dx = -g.h; dx <= g.h; ++dx) {
                    const int n1 = p / go.HW, y = p % go.HW / go.W * st + dy, x = p % go.W * st + dx;
                    const int s = px_slot(g, go, st, p) - t.base + dy * g.Wp + dx;
                    if (s < 0 || s >= t.slots) return 7;
                    const int want = y < 0 || y >= H || x < 0 || x >= W ? -1 : n1 * g.HW + y * W + x;
                    if (holds[s] != want) return 8;
                }
        // every pixel of the range has a slot of the tile, which holds it (the backward kernel computes and stores them all)
        for (int p = t.pa; p < t.pb; ++p) {
            const int s = px_slot(g, p) - t.base;
            if (st == 1 && (s < 0 || s >= t.slots)) return 14;
            if (s >= 0 && s < t.slots && holds[s] != p) return 15;
        }
        // the same pixels, and one more at either end for kernels without slots, in rows of V per group
        for (int loose = 0; st == 1 && loose < 2; ++loose) {
            const PxTile l = px_tile(g, p0, P, loose);
            if (l.pa > t.pa || l.pa < t.pa - g.h || l.pb < t.pb || l.pb > t.pb + g.h) return 16;
            int count = 0;
            while (px_group(g, l, count, n, q)) ++count;
            if (count != px_groups(g, l)) return 13;
            for (int p = l.pa; p < l.pb; ++p) {
                const int im = p / g.HW, row = px_linear(g, l, im, p % g.HW);
                if (row < 0 || !px_group(g, l, row / V, n, q) || n != im || q + row % V != p % g.HW) return 12;
            }
        }
        // every pixel leaves once, whole groups within their plane
        std::vector<int> left(t.p1 - t.p0, 0);
        const PxOut o = px_out(go, t);
        int live = 0;
        for (int i = 0; i < groups + 64; ++i)
            if (px_out_group(go, o, i, n, q)) {
                ++live;
                if (i >= P / V || q < 0 || q + V > go.HW || n * go.HW + q < t.p0 || n * go.HW + q + V > t.p1) return 9;
                for (int e = 0; e < V; ++e) ++left[n * go.HW + q + e - t.p0];
            }
        const int rest = px_out_rest(go, o);
        for (int i = 0; i < rest; ++i) {
            px_out_pixel(go, o, i, n, q);
            if (q < 0 || q >= go.HW || n * go.HW + q < t.p0 || n * go.HW + q >= t.p1) return 10;
            ++left[n * go.HW + q - t.p0];
        }
        for (int c : left)
            if (c != 1) return 11;
    }
    return 0;
}

extern "C" int emu_px(int S, int N, int H, int W, int k, int st, int P, int rows, int groups)
{
    return S == 3 ? tiles<3>(N, H, W, k, st, P, rows, groups) : tiles<2>(N, H, W, k, st, P, rows, groups);
}

// Bank conflicts (lanes of eight 16-byte accesses in one group of banks beyond the first) of a read of eight neighbouring slots.
extern "C" int emu_px_banks(int slot, int step, int octet)
{
    int used[8] = {0}, worst = 0;
    for (int i = 0; i < 8; ++i) {
        const int c = ++used[px_at(slot + i * step, octet) / 16 % 8];
        if (c > worst) worst = c;
    }
    return worst;
}
