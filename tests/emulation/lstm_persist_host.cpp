// The index arithmetic of the one-launch LSTM recurrence on the host (test infrastructure, CPU only).  Built by
// tests/test_host_lstm_persist.py; nothing in the product loads it.
#include <cmath>
#include <vector>

#include "pf_lstm_persist_index.h"

using namespace pf;

extern "C" {
// What a walk visits before row `rows`: how many elements, the last of them; 0 if one of them is not first + i * step.
int emu_walk(int n, int first, int step, int rows, long long *count, long long *last)
{
    *count = 0, *last = -1;
    for (LpWalk at(n, first, step); at.row < rows; at.next()) {
        const long long e = (long long)at.row * n + at.o;
        if (at.o < 0 || at.o >= n || e != first + *count * step) return 0;
        *last = e;
        ++*count;
    }
    return 1;
}

// Rows of a launch on a device of 256 compute units (0: not taken); `fits`: and whether the exchange buffers find room in the workspace that
// a call asks for
int emu_rows(int T, int B, int d, int h, int r, int G, int L, int bwd, int *fits)
{
    const LstmGeom g = {T, B, h, r, G, G * r, L};
    pf_lstm_stack_desc s = {};
    s.T = T, s.B = B, s.d_in = d, s.h = h, s.r = r, s.groups = G, s.layers = L;
    const size_t n = lp_floats(g, bwd);
    *fits = n > 0 && n <= lstm_stack_room(&s, bwd);
    return lp_rows_at_once(g, bwd, 256);
}

// Every workgroup of a run of rows b0 .. b0 + B - 1 of BT gives up in slot `slot`: the outputs that are not what they should be (the steps
// that the slot and those after it write are NaN, the ones before and the other rows are untouched, nothing outside is written), or -1: no
// such launch.
int emu_void_rows(int T, int B, int h, int r, int G, int L, int bwd, int slot, int b0, int BT)
{
    const LstmGeom g = {T, B, h, r, G, G * r, L};
    const LpPlan p = lp_plan(g, bwd, 256);
    if (p.NT == 0) return -1;
    const int pad = 4096, TB = T * BT, gr = G * r;
    struct Array {
        std::vector<float> v;
        int rows, width; // elements per step, per row
        bool used;
    };
    std::vector<Array> arrays((size_t)L * 10);
    LstmRunLayer l[LP_MAX_LAYERS] = {};
    for (int q = 0; q < L; ++q) {
        float **out[10] = {&l[q].h_all, &l[q].c_all, &l[q].gates, &l[q].Th, &l[q].Tx, &l[q].dz, &l[q].dTh, &l[q].dTx, &l[q].dh0, &l[q].dc0};
        const int width[10] = {h, h, 4 * h, gr, gr, 4 * h, gr, gr, h, h};
        for (int i = 0; i < 10; ++i) {
            Array &a = arrays[(size_t)q * 10 + i];
            a.width = width[i];
            a.rows = BT * width[i];
            a.v.assign((size_t)(i < 8 ? TB : BT) * width[i] + 2 * pad, 0.f);
            a.used = (i >= 5) == (bwd != 0) && !((i == 4 || i == 7) && q == 0); // (the first layer's Tx is an input, its dTx a later product)
            *out[i] = a.v.data() + pad;
        }
    }
    LpArgs a;
    lp_fill(a, p, g, l, nullptr, nullptr, b0, BT);
    for (int wg = 0; wg < p.nwg; ++wg)
        for (int tid = 0; tid < LP_NT; ++tid) {
            if (bwd)
                lp_void_bwd(a, lp_columns(a, wg, a.n2, a.rp, G == 1 ? 16 : 8, G == 1 ? p.SL : 4), lp_units(a, wg, a.n1, 16 * p.NT), slot, p.SL,
                            p.RB, wg, tid);
            else
                lp_void_fwd(a, lp_columns(a, wg, a.n1, G * a.rp, 8, 1), lp_units(a, wg, a.n2, G == 1 ? 4 * p.NT : 16), slot, tid);
        }
    int wrong = 0;
    for (int q = 0; q < L; ++q)
        for (int i = 0; i < 10; ++i) {
            const Array &b = arrays[(size_t)q * 10 + i];
            const size_t n = b.v.size() - 2 * pad;
            const int left = T - (slot - (L - 1 - q)); // backward: steps below this one
            for (size_t e = 0; e < b.v.size(); ++e) {
                const bool in = e >= (size_t)pad && e < pad + n;
                const int t = in ? (int)((e - pad) / b.rows) : 0, row = in ? (int)((e - pad) % b.rows) / b.width : 0;
                bool want = in && b.used && row >= b0 && row < b0 + B;
                if (i < 5) want = want && t >= slot - q;
                else if (i >= 8) want = want && left >= 0;
                else if (!((i == 6 || i == 7) && p.SL > 1)) want = want && t < left; // (sums over slices are written at the end)
                wrong += std::isnan(b.v[e]) != want;
            }
        }
    return wrong;
}

int emu_void(int T, int B, int h, int r, int G, int L, int bwd, int slot) { return emu_void_rows(T, B, h, r, G, L, bwd, slot, 0, B); }

// The tasks that every wavefront waits for against those whose results it reads: how many wavefronts differ, -1: no such launch.
int emu_watch(int T, int B, int h, int r, int G, int L, int bwd)
{
    const LstmGeom g = {T, B, h, r, G, G * r, L};
    const LpPlan p = lp_plan(g, bwd, 256);
    if (p.NT == 0) return -1;
    std::vector<LstmRunLayer> l(LP_MAX_LAYERS);
    LpArgs a;
    lp_fill(a, p, g, l.data(), nullptr, nullptr);
    const int U = bwd || G != 1 ? 16 * (G != 1 ? 1 : p.NT) : 4 * p.NT, TW = bwd && G == 1 ? 16 : 8;
    const int cols = bwd ? a.rp : G * a.rp, blocks = !bwd ? 1 : G != 1 ? 4 : p.SL;
    auto units = [&](int wg) { return lp_units(a, wg, bwd ? a.n1 : a.n2, U); };
    auto columns = [&](int wg) { return lp_columns(a, wg, bwd ? a.n2 : a.n1, cols, TW, blocks); };
    int wrong = 0;
    for (int wg = 0; wg < p.nwg; ++wg)
        for (int w = 0; w < LP_WAVES; ++w)
            for (int phase = 0; phase < 2; ++phase) {
                const LpUnits z = units(wg);
                const LpColumns c = columns(wg);
                const bool from_units = (phase == 0) == (bwd == 0); // what is read was written by tasks of units
                const LpShare s = from_units ? (bwd ? lp_bwd_share2(a, c, w, p.SL, U) : lp_fwd_share1(a, c, w, U))
                                             : (bwd ? lp_bwd_share1(a, z, w, p.SL) : lp_fwd_share2(a, z, w));
                std::vector<int> want(256), got(256);
                if (s.waits) {
                    for (int i = 0; i < 64; ++i) {
                        const int t = s.on.task(i);
                        if (t < 0 || t >= 256) return 1 << 20;
                        got[t] = 1;
                    }
                    if (s.on.n * s.on.blocks > 64) ++wrong;
                }
                const int k0 = 32 * s.first, k1 = k0 + 32 * (s.n > 0 ? s.n : 0);
                for (int v = 0; v < p.nwg && s.n > 0; ++v) {
                    if (from_units) {
                        const LpUnits y = units(v);
                        const int layer = !bwd && c.path ? c.l - 1 : c.l;
                        for (int k = k0; k < k1 && y.has && y.l == layer; ++k)
                            if (k % a.hp >= y.u0 && k % a.hp < y.u0 + y.n) want[y.task] = 1;
                    } else {
                        const LpColumns y = columns(v);
                        const bool above = bwd ? z.l + 1 < L && w >= 4 : w >= 4;
                        if (!bwd && above && z.l == 0) continue; // (computed beforehand)
                        for (int k = k0; k < k1 && y.has && y.path == (above ? 1 : 0) && y.l == z.l + (bwd && above); ++k) {
                            const int col = bwd ? k % a.rp : k, gate = bwd && G != 1 ? k / a.rp : -1;
                            if (col >= y.col && col < y.col + y.n && (gate < 0 || gate == y.q)) want[y.task] = 1;
                        }
                    }
                }
                if (s.n > 0 && want != got) ++wrong;
            }
    return wrong;
}
}
