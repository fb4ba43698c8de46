// Tiled matrix products for any shape (pf_tile.h): the choice of tile shape and split, and the sums over splits.
#include <math.h>

#include "pf_tile_host.h"

namespace pf {

// ------------------------------------------------------------------ host side
struct ShapeInfo {
    int bm, bn;
};
static const ShapeInfo SHAPES[TS_COUNT] = {{32, 32}, {64, 64}, {128, 64}, {128, 128}, {32, 64}, {32, 128}, {32, 32}};

TileProb tile_prob(int type, int M, int N, int K, const void *A, i64 lda, const void *B, i64 ldb, void *C, i64 ldc)
{
    TileProb p = {};
    p.type = type;
    p.M = M, p.N = N, p.K = K;
    p.nb = 1;
    p.A = A, p.lda = lda;
    p.B = B, p.ldb = ldb;
    p.o.C = C, p.o.ld = ldc;
    return p;
}

// Clocks of a compute unit, measured over products of 2000 to 16000 rows and contractions of 256 to 4096: `work` is what a
// chunk of the contraction costs a compute unit that several workgroups keep busy (the LDS traffic of the fragments for
// bf16, the matrix instructions for float), `tile` what a tile costs besides (finding it, the first loads, the store),
// `one` how long a chunk takes a workgroup that is alone.  Every split costs a partial sum to write and to read, and the
// first of them one more launch.
struct ChunkCost {
    double work, tile, one;
};
static ChunkCost chunk_cost(bool bf, TileShape sh)
{
    static const ChunkCost costs[2][4] = {{{469, 910, 400}, {1608, 1100, 1200}, {3440, 2140, 2600}, {6120, 20000, 5500}},
                                          {{282, 260, 380}, {600, 1000, 650}, {1000, 4800, 1100}, {1850, 8000, 1850}}};
    return costs[bf][sh];
}

TilePlan plan_tiles(int dtype, i64 M, i64 N, i64 K, int max_split)
{
    const TileNeed need = {M, N, K, max_split > 1};
    TileGroup g = plan_tile_group(dtype, &need, 1);
    return TilePlan{g.shape, g.ksplit[0] > max_split ? max_split : g.ksplit[0], g.cost};
}

TileGroup plan_tile_group(int dtype, const TileNeed *need, int n)
{
    const bool bf = dtype == PF_BF16;
    const int bk = bf ? 64 : 32;
    static const TileShape tries[4] = {TS_32, TS_64, TS_128x64, TS_128};
    TileGroup best = {TS_64, {1, 1, 1, 1, 1, 1}, 1e30};
    for (TileShape sh : tries) {
        const ChunkCost cc = chunk_cost(bf, sh);
        const i64 bm = SHAPES[sh].bm, bn = SHAPES[sh].bn;
        for (int most = 2; most <= (1 << 20); most *= 2) { // chunks a workgroup of a split product may have
            TileGroup g = {sh, {1, 1, 1, 1, 1, 1}, 0};
            double total = 0, longest = 0, part = 0, count = 0;
            bool any = false, last = true;
            for (int i = 0; i < n; ++i) {
                const i64 tiles = ((need[i].M + bm - 1) / bm) * ((need[i].N + bn - 1) / bn);
                const i64 chunks = (need[i].K + bk - 1) / bk;
                i64 ks = need[i].split ? (chunks + most - 1) / most : 1;
                if (ks > 32) ks = 32;
                while (ks > 1 && ks * need[i].M * need[i].N > (2 << 20)) --ks; // at most 8 MB of partial sums
                const i64 per = (chunks + ks - 1) / ks;
                ks = (chunks + per - 1) / per;
                if (ks > 1) {
                    any = true;
                    part += (double)ks * need[i].M * need[i].N * 8;
                }
                if (need[i].split && chunks > most) last = false;
                g.ksplit[i] = (int)ks;
                total += (double)tiles * ks * (per * cc.work + cc.tile);
                count += (double)tiles * ks;
                if (per * cc.one + cc.tile > longest) longest = per * cc.one + cc.tile;
            }
            const double each = count > 0 ? ceil(count / 256) * (total / count) : 0; // the fullest compute unit's share
            g.cost = (each > longest ? each : longest) + 3000 + (any ? 6000 + part / 2000 : 0);
            if (g.cost < best.cost) best = g;
            if (last) break;
        }
    }
    // bf16 gradients that contract over many rows: bringing the lines of both operands in takes 8 bytes a clock of a compute unit, twice
    // what `work` says, and 128 x 128 tiles need half as much, if they come out at most two to a compute unit, all at once.  A
    // backward call of one layer (dX, dU and dV in one launch), us, the plan above / 128 x 128: 8192 rows, 512 -> 128 -> 2048 49.1 /
    // 43.7, rank 256 69.8 / 64.1; 7500 rows, two layers of 640 -> 256 -> 384 that share their input 88.3 / 47.4; the launch of three 512
    // -> 128 -> 512 48.4 / 27.1.  Not so
    //   with fewer rows (4096, 512 -> 128 -> 2048 33.3 / 37.2),
    //   with more than two to a compute unit (16384, 512 -> 128 -> 2048 72.5 / 86.1) or fewer than one and a half,
    //   with more than 32 chunks to a workgroup (6100, 1024 -> 384 -> 1024 66 / 73) or padding of the rank (8192, 768 -> 192 -> 768 48.9 /
    //   53.7),
    //   where the plan above has nearly seven workgroups to a compute unit or more, which hide each other's waits (7500, 1000 -> 128 ->
    //   256 34.6 / 49.4), or splits more than five ways, so that its chunks are few (20000, 320 -> 128 -> 128 33.1 / 56.9),
    //   where it brings less than 400 KB into a compute unit (8192, 384 -> 128 -> 384 25.7 / 30.1),
    //   or where padding takes more than a seventeenth of the work (10183, 576 -> 128 -> 1344 47.5 / 56.8; 7740, 832 -> 128 -> 176 34 / 39).
    // Measured over 399 shapes of 6000 to 40000 rows, widths 64 to 4096, ranks 128 to 512, one to four layers, that pass all but the
    // last line: 0.88 of the plan above (geometric mean), but 31 more than 5 % slower, at most 1.24 times.  180 are taken, 0.86 of the
    // plan above, one of them more than 5 % slower (1.06).
    if (bf && n == 3 && need[1].tn && need[2].tn && need[1].K >= 6000 && need[1].N % 128 == 0 && need[2].N % 128 == 0 && best.ksplit[1] <= 5 &&
        best.ksplit[2] <= 5) {
        const auto tiles = [&](int i, TileShape sh) {
            return ((need[i].M + SHAPES[sh].bm - 1) / SHAPES[sh].bm) * ((need[i].N + SHAPES[sh].bn - 1) / SHAPES[sh].bn);
        };
        i64 now = 0, bytes = 0; // workgroups of the plan above, and what they bring into all compute units
        double work = 0, dealt = 0; // of all products; of their 128 x 128 tiles
        for (int i = 0; i < 3; ++i) {
            work += (double)need[i].M * need[i].N * need[i].K;
            dealt += 128.0 * 128.0 * tiles(i, TS_128) * need[i].K;
            now += tiles(i, best.shape) * best.ksplit[i];
            bytes += tiles(i, best.shape) * need[i].K * (SHAPES[best.shape].bm + SHAPES[best.shape].bn) * 2;
        }
        const i64 rest = 512 - tiles(0, TS_128), each = tiles(1, TS_128) + tiles(2, TS_128);
        i64 ks = rest / each;
        for (int i = 1; i < 3; ++i)
            while (ks > 1 && ks * need[i].M * need[i].N > (2 << 20)) --ks;
        if (ks >= 1 && rest >= each && tiles(0, TS_128) + ks * each >= 384 && need[1].K <= 64 * 32 * ks && now <= 1740 &&
            bytes >= 256 * 400 * 1024 && work >= 0.94 * dealt) {
            best.shape = TS_128;
            best.ksplit[0] = 1;
            best.ksplit[1] = best.ksplit[2] = (int)ks;
            return best;
        }
    }
    // 32 x 32 tiles that leave a compute unit with one workgroup: eight wavefronts share its chunks, twice as long, so that two
    // wavefronts of a SIMD cover each other's waits.  Float, 188 workgroups of 47 chunks (64 x 1500 times 1500 x 3000) 18.2 -> 15.2 us,
    // 256 of 16 chunks 9.7 -> 8.0, of 8 chunks 6.8 -> 6.4; with two workgroups there already (bf16, 470 of 10 chunks) 6.6 -> 7.2.
    if (best.shape == TS_32) {
        i64 count = 0, shortest = 1 << 30;
        for (int i = 0; i < n; ++i) {
            const i64 chunks = (need[i].K + bk - 1) / bk;
            count += ((need[i].M + 31) / 32) * ((need[i].N + 31) / 32) * best.ksplit[i];
            shortest = chunks / best.ksplit[i] < shortest ? chunks / best.ksplit[i] : shortest;
        }
        if (count <= 256 && shortest >= 8) best.shape = TS_32D;
    }
    return best;
}

// A chain's compute unit has a workgroup of the others beside it while there are any left; until then, at two to a compute unit, a chunk of
// it takes twice `work` instead of `one`.
double tile_chain_cost(int dtype, TileShape shape, const TileNeed *need, int n, int chains)
{
    const ChunkCost cc = chunk_cost(dtype == PF_BF16, shape);
    const i64 bm = SHAPES[shape].bm, bn = SHAPES[shape].bn, bk = dtype == PF_BF16 ? 64 : 32;
    double longest = 0, rest = 0;
    for (int i = 0; i < n; ++i) {
        const double tiles = (double)(((need[i].M + bm - 1) / bm) * ((need[i].N + bn - 1) / bn)), chunks = (double)((need[i].K + bk - 1) / bk);
        if (i >= chains) rest += tiles * (chunks * cc.work + cc.tile);
        else if (chunks * cc.one + cc.tile > longest) longest = chunks * cc.one + cc.tile;
    }
    return 3000 + longest + (1 - cc.one / (2 * cc.work)) * rest / 256;
}

// (a workgroup of the readers brings its slices in at 50 bytes a clock; bf16 at 25, for its own intermediate is half of one of them)
MidGroup plan_mid_group(int dtype, const TileNeed *need, int n, TileShape reader, i64 all, i64 most)
{
    MidGroup best = {plan_tile_group(dtype, need, n), false};
    if (reader != TS_32 && reader != TS_32D) return best;
    const ChunkCost cc = chunk_cost(dtype == PF_BF16, TS_32);
    const int bk = dtype == PF_BF16 ? 64 : 32;
    const double rate = dtype == PF_BF16 ? 25 : 50;
    for (int ks = 2; ks <= TILE_MAX_SLICES; ++ks) {
        i64 count = 0, longest = 0, shortest = 1 << 30;
        double total = 0;
        bool empty = false;
        for (int i = 0; i < n; ++i) {
            const i64 tiles = ((need[i].M + 31) / 32) * ((need[i].N + 31) / 32), chunks = (need[i].K + bk - 1) / bk, per = (chunks + ks - 1) / ks;
            empty = empty || (ks - 1) * per >= chunks;
            count += tiles * ks;
            total += (double)tiles * ks * (per * cc.work + cc.tile);
            longest = per > longest ? per : longest;
            shortest = per < shortest ? per : shortest;
        }
        if (empty) continue;
        const bool deep = count <= 256 && shortest >= 8;
        const double own = ceil(count / 256.0) * total / count, alone = longest * cc.one * (deep ? 0.85 : 1) + cc.tile;
        const double cost = (own > alone ? own : alone) + 3000 + ks * (all > 256 * most ? all / 256.0 : most) / rate;
        if (cost >= best.g.cost) continue;
        best.g.shape = deep ? TS_32D : TS_32;
        for (int i = 0; i < n; ++i) best.g.ksplit[i] = ks;
        best.g.cost = cost;
        best.sliced = true;
    }
    return best;
}

MidPlan plan_mid(int dtype, i64 M, i64 N, i64 K, int max_split, TileShape reader, i64 all, i64 most)
{
    const TileNeed need = {M, N, K, true};
    const MidGroup m = plan_mid_group(dtype, &need, 1, reader, all, most);
    if (!m.sliced) return MidPlan{plan_tiles(dtype, M, N, K, max_split), false};
    return MidPlan{TilePlan{m.g.shape, m.g.ksplit[0], m.g.cost}, true};
}

void tile_add(TileArgs &a, TileShape shape, int dtype, const TileProb &q, int ksplit)
{
    TileProb &p = a.p[a.n++];
    p = q;
    const int bk = (dtype == PF_BF16 ? 64 : 32) * (shape == TS_32D ? 2 : 1);
    p.tm = (p.M + SHAPES[shape].bm - 1) / SHAPES[shape].bm;
    p.tn = (p.N + SHAPES[shape].bn - 1) / SHAPES[shape].bn;
    p.ksplit = ksplit < 1 ? 1 : ksplit;
    if (p.type == TILE_WG || p.type == TILE_WGG || p.type == TILE_WGT) {
        p.kper = (p.pa.N + p.ksplit - 1) / p.ksplit;
        p.ksplit = (p.pa.N + p.kper - 1) / p.kper;
    } else if (p.type == TILE_PACK) {
        const i64 total = (i64)p.M * p.N * p.pb.ntap;
        p.tm = (int)((total + 4 * TILE_THREADS - 1) / (4 * TILE_THREADS));
        p.tn = p.ksplit = 1;
    } else {
        p.kper = ((p.K + p.ksplit - 1) / p.ksplit + bk - 1) / bk * bk;
        if (p.kper < bk) p.kper = bk; // (an empty contraction is one empty split)
        p.ksplit = p.K > 0 ? (p.K + p.kper - 1) / p.kper : 1;
    }
    p.block0 = a.blocks;
    a.blocks += (p.tm * p.tn * p.ksplit * p.nb + 7) / 8 * 8;
}

void tile_pair(TileArgs &a)
{
    a.p[a.n - 2].pair = 1;
    a.blocks = a.p[a.n - 1].block0;
}

template <typename CT>
int launch_linear_t(hipStream_t s, const char *name, TileShape shape, const TileArgs &a);
template <typename CT>
int launch_conv_t(hipStream_t s, const char *name, TileShape shape, TileShape wg, const TileArgs &a);

int launch_tiles_linear(hipStream_t s, const char *name, int dtype, TileShape shape, const TileArgs &a)
{
    if (a.blocks <= 0) return PF_OK;
    return dtype == PF_F32 ? launch_linear_t<float>(s, name, shape, a) : launch_linear_t<bf16_t>(s, name, shape, a);
}

int launch_tiles_conv(hipStream_t s, const char *name, int dtype, TileShape shape, TileShape wg, const TileArgs &a)
{
    if (a.blocks <= 0) return PF_OK;
    return dtype == PF_F32 ? launch_conv_t<float>(s, name, shape, wg, a) : launch_conv_t<bf16_t>(s, name, shape, wg, a);
}

// ------------------------------------------------------------------ sums over splits
// 64 groups of four neighbouring outputs per workgroup; the splits are dealt to four threads per group, eight in flight
// each, and the four sums are added in a fixed order.
template <bool VEC>
__device__ __forceinline__ f32x4_t split_share(const SplitSum &q, i64 i, int part)
{
    const int per = (q.splits + 3) / 4, end = min(q.splits, (part + 1) * per);
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    for (int s = part * per; s < end; s += 8) {
        f32x4_t t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float *r = q.src + i + (i64)min(s + u, q.splits - 1) * q.stride;
            if (VEC) {
                t[u] = *(const f32x4_t *)r;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) t[u][e] = r[i + e < q.count ? e : 0];
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s + u < end) v += t[u];
    }
    return v;
}

__global__ __launch_bounds__(256) void split_sums_kernel(SplitSumArgs a)
{
    __shared__ f32x4_t share[3][64];
    int k = 0;
#pragma unroll
    for (int i = 1; i < 4; ++i)
        if (i < a.n && (int)blockIdx.x >= a.blocks[i]) k = i;
    const SplitSum &q = a.s[k];
    const int part = threadIdx.x >> 6, o = threadIdx.x & 63;
    const i64 i = ((i64)(blockIdx.x - a.blocks[k]) * 64 + o) * 4;
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    if (i < q.count) // (the partial sums start 256-byte aligned)
        v = q.count % 4 == 0 && q.stride % 4 == 0 ? split_share<true>(q, i, part) : split_share<false>(q, i, part);
    if (part > 0) share[part - 1][o] = v;
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int u = 0; u < 3; ++u) v += share[u][o];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (i + e >= q.count) return;
        i64 at = i + e;
        if (q.np > 0) {
            const i64 per = q.count / q.tm, m = at / per, n = at - m * per, img = n / q.np, pos = n - img * q.np;
            if (pos >= q.hw) continue;
            at = (img * q.tm + m) * q.hw + pos;
        } else if (q.tn > 0) {
            const i64 m = at / q.tn;
            at = (at - m * q.tn) * q.tm + m;
        }
        float w = v[e];
        if (q.rscale) w *= q.rscale[at / q.rlen];
        if (q.bf16) ((uint16_t *)q.dst)[at] = float_to_bf16_bits(w);
        else q.dst[at] = q.accumulate ? q.dst[at] + w : w;
    }
}

void split_sum_add(SplitSumArgs &a, const SplitSum &s)
{
    if (!s.dst || s.count <= 0) return;
    a.s[a.n] = s;
    a.blocks[a.n + 1] = a.blocks[a.n] + (int)((s.count + 255) / 256);
    ++a.n;
}

int launch_split_sums(hipStream_t s, const SplitSumArgs &a)
{
    int st = PF_OK;
    if (a.n == 0) return st;
    PF_LAUNCH(st, "split_sums", split_sums_kernel, dim3(a.blocks[a.n]), dim3(256), s, a);
    return st;
}

} // namespace pf
