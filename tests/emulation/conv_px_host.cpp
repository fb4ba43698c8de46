// The index arithmetic of the pixel-major convolutions (test infrastructure, CPU only; plain C++).
#include "pf_conv_px_index.h"

#include <vector>

using namespace pf;

// Every tile of P pixels of N planes H x W under k x k taps, with room for `rows` slots and `groups` groups.  0: right; else what is not.
extern "C" int emu_px(int N, int H, int W, int k, int P, int rows, int groups)
{
    const PxPlane g = px_plane(N, H, W, k);
    const int all = N * H * W;
    for (int p0 = 0; p0 < all; p0 += P) {
        const PxTile t = px_tile(g, p0, P);
        if (t.slots <= 0 || t.slots >= rows) return 1;
        std::vector<int> holds(rows, -1); // pixel in every slot
        int gi = 0, n, q;
        for (; px_group(g, t, gi, n, q); ++gi) {
            if (gi >= groups) return 2;
            if (n < 0 || n >= N || q < 0 || q + 8 > g.HW) return 3; // a load outside its plane
            if (g.HW % 8 == 0 && q % 8) return 4;
            for (int e = 0; e < 8; ++e) {
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
                    const int n1 = p / g.HW, y = p % g.HW / W + dy, x = p % W + dx;
                    const int s = px_slot(g, p) - t.base + dy * g.Wp + dx;
                    if (s < 0 || s >= t.slots) return 7;
                    const int want = y < 0 || y >= H || x < 0 || x >= W ? -1 : n1 * g.HW + y * W + x;
                    if (holds[s] != want) return 8;
                }
        // the same pixels in rows of eight per group
        for (int p = t.pa; p < t.pb; ++p) {
            const int im = p / g.HW, row = px_linear(g, t, im, p % g.HW);
            if (row < 0 || !px_group(g, t, row / 8, n, q) || n != im || q + row % 8 != p % g.HW) return 12;
        }
        // every pixel leaves once, whole groups within their plane
        std::vector<int> left(t.p1 - t.p0, 0);
        const PxOut o = px_out(g, t);
        int live = 0;
        for (int i = 0; i < groups + 64; ++i)
            if (px_out_group(g, o, i, n, q)) {
                ++live;
                if (i >= P / 8 || q < 0 || q + 8 > g.HW || n * g.HW + q < t.p0 || n * g.HW + q + 8 > t.p1) return 9;
                for (int e = 0; e < 8; ++e) ++left[n * g.HW + q + e - t.p0];
            }
        const int rest = px_out_rest(g, o);
        for (int i = 0; i < rest; ++i) {
            px_out_pixel(g, o, i, n, q);
            if (q < 0 || q >= g.HW || n * g.HW + q < t.p0 || n * g.HW + q >= t.p1) return 10;
            ++left[n * g.HW + q - t.p0];
        }
        for (int c : left)
            if (c != 1) return 11;
    }
    return 0;
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
