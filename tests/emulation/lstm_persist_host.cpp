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

// Every workgroup of a run gives up in slot `slot`: the outputs that are not what they should be (the steps that the slot
// and those after it write are NaN, the ones before are untouched, nothing outside is written), or -1: no such launch.
int emu_void(int T, int B, int h, int r, int G, int L, int bwd, int slot)
{
    const LstmGeom g = {T, B, h, r, G, G * r, L};
    const LpPlan p = lp_plan(g, bwd, 256);
    if (p.NT == 0) return -1;
    const int pad = 4096, TB = T * B, gr = G * r;
    struct Array {
        std::vector<float> v;
        int rows; // per step
        bool used;
    };
    std::vector<Array> arrays((size_t)L * 10);
    LstmRunLayer l[LP_MAX_LAYERS] = {};
    for (int q = 0; q < L; ++q) {
        float **out[10] = {&l[q].h_all, &l[q].c_all, &l[q].gates, &l[q].Th, &l[q].Tx, &l[q].dz, &l[q].dTh, &l[q].dTx, &l[q].dh0, &l[q].dc0};
        const int width[10] = {h, h, 4 * h, gr, gr, 4 * h, gr, gr, h, h};
        for (int i = 0; i < 10; ++i) {
            Array &a = arrays[(size_t)q * 10 + i];
            a.rows = B * width[i];
            a.v.assign((size_t)(i < 8 ? TB : B) * width[i] + 2 * pad, 0.f);
            a.used = (i >= 5) == (bwd != 0) && !((i == 4 || i == 7) && q == 0); // (the first layer's Tx is an input, its dTx a later product)
            *out[i] = a.v.data() + pad;
        }
    }
    LpArgs a;
    lp_fill(a, p, g, l, nullptr, nullptr);
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
                const int t = in ? (int)((e - pad) / b.rows) : 0;
                bool want = in && b.used;
                if (i < 5) want = want && t >= slot - q;
                else if (i >= 8) want = want && left >= 0;
                else if (!((i == 6 || i == 7) && p.SL > 1)) want = want && t < left; // (sums over slices are written at the end)
                wrong += std::isnan(b.v[e]) != want;
            }
        }
    return wrong;
}
}
