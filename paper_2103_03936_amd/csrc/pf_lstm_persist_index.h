// The one-launch LSTM recurrence (pf_lstm_persist.hip): plan, arguments, and which workgroup has what.  Host and device.
#pragma once

#include "pf_lstm_persist.h"

namespace pf {

constexpr int LP_MAX_LAYERS = 4;
constexpr int LP_NT = 512, LP_WAVES = 8; // threads
constexpr int LP_GROUPS = 8;             // of workgroups in a barrier
constexpr int LP_BAR = 2 * LP_GROUPS * 64; // words of one: a line per group counter, then the copies of its flags
constexpr int LP_MOST_CUS = 256;           // tasks of a phase, at most
// How far each task is: words, in eight copies (a workgroup polls one of them), 16 tasks to a line of 256 bytes
constexpr int LP_COPY = 2 * LP_MOST_CUS / 16 * 64, LP_FLAGS = LP_GROUPS * LP_COPY;
__host__ __device__ __forceinline__ int lp_flag(int phase, int task) { return ((phase - 1) * LP_MOST_CUS + task) / 16 * 64 + task % 16; }
constexpr int LP_SYNC = LP_BAR + LP_FLAGS + 64; // the last 64: the word of a failed wait
constexpr int LP_FAILED = LP_BAR + LP_FLAGS;

struct LpArgs {
    LstmRunLayer l[LP_MAX_LAYERS];
    const float *dh_top;
    float *xh, *xt; // exchanged: h (forward; step t at t + 1, the initial state at 0) or dz (backward); T or dT
    unsigned *sync;
    i64 xh_step, xt_step; // floats from one step's copy to the next
    int T, B, h, r, G, gr, L;
    int BT;               // rows of a step in the arrays, B or more: a launch may take some of them
    int hp, rp;           // h and r up to whole groups of 32 contraction indices
    int n1, n2, nwg;      // tasks (one per workgroup) of the two phases of a slot
    int nt1;              // 8-column tiles of a T / dT task
};

// ------------------------------------------------------------------ tasks
// Workgroups go to the dies in turn.  Those of one die get neighbouring tasks: they read the same activations and, where a row of
// the factors is shared by column tiles, the same lines.  (n workgroups take part: a multiple of LP_GROUPS; some have no task)
__host__ __device__ __forceinline__ int lp_task(int wg, int n) { return (wg % LP_GROUPS) * (n / LP_GROUPS) + wg / LP_GROUPS; }

// product p of the 2 L - 1 of a slot: layer (p + 1) / 2, its hidden path (p = 0 or odd) or input path
__host__ __device__ __forceinline__ int lp_layer(int p) { return (p + 1) >> 1; }
__host__ __device__ __forceinline__ int lp_path(int p) { return p > 0 && !(p & 1); }
__host__ __device__ __forceinline__ float *lp_xt(const LpArgs &a, int l, int path, int t)
{
    return a.xt + ((i64)(2 * l + path) * a.T + t) * a.xt_step;
}
__host__ __device__ __forceinline__ float *lp_xh(const LpArgs &a, int l, int slot) { return a.xh + ((i64)l * (a.T + 1) + slot) * a.xh_step; }

// A workgroup's units u0 .. u0 + n - 1 of layer l (n workgroups of U units each take part; !has: none for this one)
struct LpUnits {
    bool has;
    int l, u0, n, task;
};
__host__ __device__ __forceinline__ LpUnits lp_units(const LpArgs &a, int wg, int parts, int U)
{
    LpUnits t;
    const int per_layer = (a.hp + U - 1) / U, task = lp_task(wg, parts);
    t.has = wg < parts && task < a.L * per_layer;
    t.l = t.has ? task / per_layer : 0;
    t.u0 = t.has ? (task - t.l * per_layer) * U : 0;
    t.n = U;
    t.task = task;
    return t;
}
// Its columns col .. col + n - 1 of T (or dT) of product p: of `cols` columns, in tiles of TW, block q of the product's `blocks`
struct LpColumns {
    bool has;
    int p, q, l, path, col, n, task;
};
__host__ __device__ __forceinline__ LpColumns lp_columns(const LpArgs &a, int wg, int parts, int cols, int TW, int blocks)
{
    LpColumns t;
    const int per_block = (cols / TW + a.nt1 - 1) / a.nt1, task = lp_task(wg, parts);
    t.has = wg < parts && task < (2 * a.L - 1) * blocks * per_block;
    const int b = t.has ? task / per_block : 0;
    t.p = b / blocks, t.q = b - t.p * blocks;
    t.l = lp_layer(t.p), t.path = lp_path(t.p);
    t.col = t.has ? (task - b * per_block) * TW * a.nt1 : 0;
    t.n = TW * a.nt1 < cols - t.col ? TW * a.nt1 : cols - t.col;
    t.task = task;
    return t;
}

// The tasks whose results a wavefront reads (at most 64, one per lane that polls): `blocks` runs of n tasks, `stride` apart, from
// base + first on, a run going on at base after base + wrap - 1.  Their results fill whole groups of 32 indices of an exchanged
// matrix, and so whole lines: none of those is read before every task that writes to it is done.
struct LpWatch {
    int base, first, n, wrap, blocks, stride;
    __host__ __device__ __forceinline__ int task(int lane) const
    {
        const int b = lane < n * blocks ? lane / n : 0, i = lane < n * blocks ? lane - b * n : 0;
        return base + b * stride + (first + i < wrap ? first + i : first + i - wrap);
    }
};
// those of units k0 .. k0 + len - 1 of layer l, in tasks of U (past hp: on from unit 0)
__host__ __device__ __forceinline__ LpWatch lp_watch_units(const LpArgs &a, int l, int k0, int len, int U)
{
    const int per_layer = (a.hp + U - 1) / U;
    LpWatch w = {l * per_layer, k0 / U, 0, per_layer, 1, 0};
    if (len <= 0) return w;
    const int last = k0 + len - 1;
    w.n = (last < a.hp ? last / U : per_layer + (last - a.hp) / U) - w.first + 1;
    if (w.n > per_layer) w.n = per_layer;
    return w;
}
// those of columns k0 .. k0 + len - 1 of T of product p (all gates' columns, rp each where a block is one gate; else every block)
__host__ __device__ __forceinline__ LpWatch lp_watch_columns(const LpArgs &a, int p, int k0, int len, int cols, int TW, int blocks, bool gates)
{
    const int per_block = (cols / TW + a.nt1 - 1) / a.nt1, tile = TW * a.nt1, last = k0 + len - 1;
    const int q0 = gates ? k0 / cols : 0, q1 = gates ? last / cols : 0;
    LpWatch w = {p * blocks * per_block, q0 * per_block + (k0 - q0 * cols) / tile, 0, 1 << 30, gates ? 1 : blocks, per_block};
    if (len > 0) w.n = q1 * per_block + (last - q1 * cols) / tile - w.first + 1;
    return w;
}

// Wavefront w's share of a task's contraction: n groups of 32 indices from group `first` on, and whom it waits for before it reads
// them (!waits: nobody, they are there or there are none).
struct LpShare {
    int first, n;
    bool waits;
    LpWatch on;
};
__host__ __device__ __forceinline__ int lp_left(int per, int left) { return per < left ? per : left; }
__host__ __device__ __forceinline__ LpShare lp_fwd_share1(const LpArgs &a, const LpColumns &c, int w, int U)
{
    LpShare s;
    const int total = a.hp / 32, per = (total + LP_WAVES - 1) / LP_WAVES;
    s.first = w * per, s.n = c.has ? lp_left(per, total - s.first) : 0;
    s.waits = s.n > 0;
    s.on = lp_watch_units(a, c.path ? c.l - 1 : c.l, 32 * s.first, 32 * s.n, U);
    return s;
}
__host__ __device__ __forceinline__ LpShare lp_fwd_share2(const LpArgs &a, const LpUnits &z, int w) // (wavefronts 0 - 3: Th, 4 - 7: Tx)
{
    LpShare s;
    const int total = a.rp / 32, per = a.G != 1 ? total : (total + 3) / 4, p = w >= 4 ? 2 * z.l : z.l ? 2 * z.l - 1 : 0;
    s.first = (w & 3) * per, s.n = !z.has ? 0 : a.G != 1 ? per : lp_left(per, total - s.first);
    s.waits = s.n > 0 && (z.l > 0 || w < 4); // (the first layer's Tx is there)
    s.on = lp_watch_columns(a, p, 32 * s.first, 32 * s.n, a.G * a.rp, 8, 1, false);
    return s;
}
__host__ __device__ __forceinline__ LpShare lp_bwd_share1(const LpArgs &a, const LpUnits &z, int w, int SL)
{
    LpShare s;
    const bool two = z.l + 1 < a.L;
    const int parts = two ? 4 : 8, total = a.G * a.rp / 32, per = (total + parts - 1) / parts, p = two && w >= 4 ? 2 * z.l + 2 : z.l ? 2 * z.l - 1 : 0;
    s.first = (w & (parts - 1)) * per, s.n = z.has ? lp_left(per, total - s.first) : 0;
    s.waits = s.n > 0;
    s.on = a.G != 1 ? lp_watch_columns(a, p, 32 * s.first, 32 * s.n, a.rp, 8, 4, true)
                    : lp_watch_columns(a, p, 32 * s.first, 32 * s.n, a.rp, 16, SL, false);
    return s;
}
__host__ __device__ __forceinline__ LpShare lp_bwd_share2(const LpArgs &a, const LpColumns &c, int w, int SL, int U) // (slice q of 4 hp, or gate q)
{
    LpShare s;
    const int total = (a.G != 1 ? a.hp : 4 * a.hp) / 32, slice = (total + SL - 1) / SL, per = (slice + LP_WAVES - 1) / LP_WAVES;
    const int s0 = a.G != 1 ? 0 : c.q * slice;
    s.first = s0 + w * per, s.n = c.has ? lp_left(per, lp_left(s0 + slice, total) - s.first) : 0;
    s.waits = s.n > 0;
    s.on = lp_watch_units(a, c.l, 32 * s.first % a.hp, 32 * s.n, U);
    return s;
}

// Walks the elements first, first + step, ... of a list of rows of n elements each; row and o are the current element's row
// and place in it.  All steps' rows together have more elements than 32 bits count (three layers of rank 384, batch 32: from
// 34953 steps on), the rows alone do not, and no division is needed after the first element.
struct LpWalk {
    int row, o, n, rows_per_step, left_per_step;
    __host__ __device__ __forceinline__ LpWalk(int n_, int first, int step)
    {
        n = n_;
        row = first / n, o = first - row * n;
        rows_per_step = step / n, left_per_step = step - rows_per_step * n;
    }
    __host__ __device__ __forceinline__ void next()
    {
        row += rows_per_step;
        o += left_per_step;
        if (o >= n) o -= n, ++row;
    }
};

// ------------------------------------------------------------------ a wait that gave up
// A workgroup that leaves the launch early writes NaN over what it has not written: its own outputs of the steps from the
// current one on, and no one else's.  (Every wait that succeeded had all its data, so what was written before is right.)
__host__ __device__ inline float lp_nan() { return __builtin_nanf(""); }

__host__ __device__ inline void lp_void_columns(const LpArgs &a, float *out, int col, int n, int t0, int t1, int tid)
{
    for (int t = t0; t < t1; ++t)
        for (int e = tid; e < a.B * n; e += LP_NT) {
            const int m = e / n, c = col + e - m * n, q = c / a.rp, cc = c - q * a.rp;
            if (q < a.G && cc < a.r) out[((i64)t * a.BT + m) * a.gr + q * a.r + cc] = lp_nan();
        }
}
// forward, in slot `slot`
__host__ __device__ inline void lp_void_fwd(const LpArgs &a, const LpColumns &c, const LpUnits &z, int slot, int tid)
{
    if (c.has) lp_void_columns(a, c.path ? a.l[c.l].Tx : a.l[c.l].Th, c.col, c.n, slot > c.l ? slot - c.l : 0, a.T, tid);
    if (!z.has) return;
    const LstmRunLayer &y = a.l[z.l];
    for (int t = slot > z.l ? slot - z.l : 0; t < a.T; ++t)
        for (int e = tid; e < a.B * z.n; e += LP_NT) {
            const int m = e / z.n, un = z.u0 + e - m * z.n;
            if (un >= a.h) continue;
            const i64 row = (i64)t * a.BT + m;
            y.h_all[row * a.h + un] = y.c_all[row * a.h + un] = lp_nan();
            for (int q = 0; q < 4; ++q) y.gates[(row * 4 + q) * a.h + un] = lp_nan();
        }
}
// backward, in slot `u`; with SL > 1 slices of dT it is their sums at the end that are written, RB row blocks wide
__host__ __device__ inline void lp_void_bwd(const LpArgs &a, const LpColumns &c, const LpUnits &z, int u, int SL, int RB, int wg, int tid)
{
    // steps that a layer has left: all below
    const auto left = [&](int l) {
        const int t1 = a.T - (u - (a.L - 1 - l));
        return t1 < a.T ? t1 : a.T;
    };
    if (c.has && SL == 1)
        lp_void_columns(a, c.path ? a.l[c.l].dTx : a.l[c.l].dTh, (a.G != 1 ? c.q * a.rp : 0) + c.col, c.n, 0, left(c.l), tid);
    if (wg < a.n1 && SL > 1) {
        const int per = a.rp * 4 * RB; // (this workgroup's share of the sums, in any order)
        for (LpWalk at(per, wg * LP_NT + tid, a.n1 * LP_NT); at.row < (2 * a.L - 1) * a.T; at.next()) {
            const int pr = at.row / a.T, t = at.row - pr * a.T, l = lp_layer(pr), k = at.o / (4 * RB), m = at.o - k * (4 * RB);
            if (k < a.r && m < a.B) (lp_path(pr) ? a.l[l].dTx : a.l[l].dTh)[((i64)t * a.BT + m) * a.gr + k] = lp_nan();
        }
    }
    if (!z.has || left(z.l) < 0) return;
    const LstmRunLayer &y = a.l[z.l];
    for (int t = -1; t < left(z.l); ++t)
        for (int e = tid; e < a.B * z.n; e += LP_NT) {
            const int m = e / z.n, un = z.u0 + e - m * z.n;
            if (un >= a.h) continue;
            if (t < 0) y.dh0[(i64)m * a.h + un] = y.dc0[(i64)m * a.h + un] = lp_nan();
            else
                for (int q = 0; q < 4; ++q) y.dz[(((i64)t * a.BT + m) * 4 + q) * a.h + un] = lp_nan();
        }
}

// ------------------------------------------------------------------ plan
static int lp_row_blocks(int B) { return B <= 4 ? 1 : B <= 8 ? 2 : B <= 12 ? 3 : B <= 20 ? 5 : 8; }

struct LpPlan {
    int RB, NT, SL, nt1, n1, n2, nwg, hp, rp; // NT 0: the registers of the chip do not hold the factors
    i64 xh_step, xt_step;
    size_t floats;
};
// One task per workgroup and phase, the smallest tiles that come out at no more tasks than compute units.  The bounds are the
// kernels': groups of 32 contraction indices per wavefront, tiles, and what fits beside the accumulators of RB row blocks.
static LpPlan lp_plan(const LstmGeom &g, bool bwd, int cus)
{
    LpPlan p = {};
    p.RB = lp_row_blocks(g.B);
    p.hp = (g.h + 31) & ~31;
    p.rp = (g.r + 31) & ~31;
    p.xh_step = (i64)(bwd ? 4 : 1) * p.hp * 4 * p.RB;
    p.xt_step = (i64)(bwd && g.G == 1 ? 3 : 1) * g.G * p.rp * 4 * p.RB;
    p.floats = (size_t)p.xh_step * g.L * (g.T + 1) + (size_t)p.xt_step * 2 * g.L * g.T + LP_SYNC;
    if (p.hp > 1536 || p.rp > 384 || (g.G != 1 && p.RB == 8)) return p;
    const int products = 2 * g.L - 1;
    int tasks = 0;
    p.SL = p.nt1 = 1;
    if (bwd && g.G == 1) {
        // dT = dz U contracts 4 h: tiles of 16 columns, up to three slices (the readers add them up; one slice of 8 columns per
        // workgroup read three times the activations: 9 instead of 5 us at 1500 units)
        const int groups = p.hp / 8, cols = p.rp / 16;
        for (p.SL = 3; p.SL > 1; --p.SL)
            if (products * cols * p.SL <= cus && groups >= LP_WAVES * p.SL) break;
        tasks = products * cols * p.SL;
        const int per_wave = ((groups + p.SL - 1) / p.SL + LP_WAVES - 1) / LP_WAVES;
        if (tasks > cus || per_wave > (p.SL == 3 ? 8 : 12)) return p;
    } else {
        const int blocks = products * (bwd ? g.G : 1), cols = (bwd ? 1 : g.G) * p.rp / 8, most = g.G == 1 ? 1 : 3;
        for (p.nt1 = 1;; ++p.nt1) {
            tasks = blocks * ((cols + p.nt1 - 1) / p.nt1);
            if (tasks <= cus) break;
            if (p.nt1 == most) return p;
        }
    }
    int units = 0, most = g.G != 1 ? 1 : bwd ? (p.RB == 8 ? 1 : 2) : p.RB == 8 ? 2 : p.RB == 5 ? 3 : 5, NT = 1;
    for (; NT <= most; ++NT) {
        const int U = bwd || g.G != 1 ? 16 * NT : 4 * NT;
        units = g.L * ((p.hp + U - 1) / U);
        if (units <= cus) break;
    }
    if (units > cus) return p;
    p.NT = NT == 4 ? 5 : NT;
    if (p.NT == 5) units = g.L * ((p.hp + 19) / 20);
    units = (units + LP_GROUPS - 1) / LP_GROUPS * LP_GROUPS; // (the barrier's groups are even)
    tasks = (tasks + LP_GROUPS - 1) / LP_GROUPS * LP_GROUPS;
    p.n1 = bwd ? units : tasks;
    p.n2 = bwd ? tasks : units;
    p.nwg = p.n1 > p.n2 ? p.n1 : p.n2;
    if (p.nwg > cus) p.NT = 0;
    return p;
}

// What the launches of a slot take beyond two launches of the recurrence with half the rows each, us a call.  A slot is 7.1 us of launches and their
// gaps, 3.7 more a layer and half for every million weights that it reads, less what two exchanges over the chip take, which grow with the row
// blocks, units and, with a pair per gate, the columns of T; a second cooperative launch and its start are 59.  Backward with one pair for all gates the
// launches of a slot are fewer, and slices of dT are summed at the end.  Fitted to 1218 calls of 21 to 32 rows.  us, slots / halves:
//   one pair, three layers of 704 units, batch 24, 34 steps forward 968 / 546, two of 1152, batch 30, 4 steps 179 / 188, three of 1378, batch 29, 4 steps
//   backward 319 / 459, of 1365, batch 23, 37 steps 1877 / 1371;
//   a pair per gate, three layers of 128 units, batch 27, 57 steps forward 1727 / 670, of 960, 55 steps 2465 / 1486, backward 2758 / 1899, two of 1392,
//   batch 22, 51 steps forward 2069 / 1400, one of 1216, batch 26 1274 / 1501, backward 1433 / 1338, two of 832, batch 32, 8 steps backward 317 / 346.
// The rule is 0.2 % behind the faster way (geometric mean), one call in 70 by more than a twentieth, 15 % at most.
static double lp_halves_gain(const LstmGeom &g, bool bwd)
{
    const int first = (g.B + 1) / 2, blocks = lp_row_blocks(first) + lp_row_blocks(g.B - first), slots = g.T + g.L - 1;
    const double weights = 1e-6 * g.L * (2.0 * g.gr * g.h + 8.0 * g.h * g.r);
    const double all = -59 + slots * (7.12 + 3.73 * g.L + 0.5 * weights - 0.185 * blocks - 3.52e-3 * g.h - (g.G == 1 ? 2.89 : 3.1e-3 * g.r * blocks));
    return bwd && g.G == 1 ? all - 25.4 - 7.4 * blocks + slots * (12.3 - 2.4 * blocks) : all;
}
// Rows of a launch: all, or half of them, one launch after the other, where only the halves' row blocks fit beside the factors and that is
// the faster way.
static int lp_rows_at_once(const LstmGeom &g, bool bwd, int cus)
{
    if (lp_plan(g, bwd, cus).NT > 0) return g.B;
    LstmGeom half = g;
    half.B = (g.B + 1) / 2;
    return g.B > 1 && lp_plan(half, bwd, cus).NT > 0 && lp_halves_gain(g, bwd) > 0 ? half.B : 0;
}

// Whether the largest device could take the call, and what it needs there: sizes do not depend on the device (a workspace may be
// asked for before one is chosen).  A single step uses the factors once: 125 us as launches, 160 here (1216 units, batch 28).
static size_t lp_floats(const LstmGeom &g, bool bwd)
{
    LstmGeom some = g;
    some.B = lp_rows_at_once(g, bwd, LP_MOST_CUS);
    return g.T + g.L < 3 || some.B == 0 ? 0 : lp_plan(some, bwd, LP_MOST_CUS).floats;
}
// (Halves with a pair per gate are no reason for a larger workspace than that of the launches of a slot: they are taken where their exchange buffers,
// which hold every step, fit into it, so for shorter sequences or larger layers, whose slices and copied factors are more.)
static size_t lp_wants(const LstmGeom &g, bool bwd) { return g.G != 1 && lp_rows_at_once(g, bwd, LP_MOST_CUS) != g.B ? 0 : lp_floats(g, bwd); }
// rows b0 .. b0 + g.B - 1 of arrays with BT of them
static LstmRunLayer lp_rows(const LstmRunLayer &l, const LstmGeom &g, int b0)
{
    LstmRunLayer y = l;
    const i64 h = (i64)b0 * g.h, gr = (i64)b0 * g.gr;
    for (const float **p : {&y.h0, &y.c0, &y.dhT, &y.dcT})
        if (*p) *p += h;
    for (float **p : {&y.h_all, &y.c_all, &y.dh0, &y.dc0})
        if (*p) *p += h;
    for (float **p : {&y.gates, &y.dz})
        if (*p) *p += 4 * h;
    for (float **p : {&y.Tx, &y.Th, &y.dTh, &y.dTx})
        if (*p) *p += gr;
    return y;
}

static void lp_fill(LpArgs &a, const LpPlan &p, const LstmGeom &g, const LstmRunLayer *l, const float *dh_top, float *ws, int b0 = 0, int BT = 0)
{
    a = {};
    a.BT = BT ? BT : g.B;
    for (int q = 0; q < g.L; ++q) a.l[q] = lp_rows(l[q], g, b0);
    a.dh_top = dh_top ? dh_top + (i64)b0 * g.h : nullptr;
    a.xh = ws;
    a.xt = a.xh + p.xh_step * g.L * (g.T + 1);
    a.sync = (unsigned *)(a.xt + p.xt_step * 2 * g.L * g.T);
    a.xh_step = p.xh_step;
    a.xt_step = p.xt_step;
    a.T = g.T, a.B = g.B, a.h = g.h, a.r = g.r, a.G = g.G, a.gr = g.gr, a.L = g.L;
    a.hp = p.hp, a.rp = p.rp;
    a.n1 = p.n1, a.n2 = p.n2, a.nwg = p.nwg, a.nt1 = p.nt1;
}

} // namespace pf
