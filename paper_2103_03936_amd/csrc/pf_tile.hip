// Tiled matrix products for any shape (pf_tile.h): the kernels, the choice of tile shape and split, and the sums over
// splits.  One launch runs a list of problems: a workgroup finds its problem, its tile and its share of the contraction
// from its index.
#include "pf_tile_host.h"

namespace pf {

// Workgroups are dealt to the eight dies in turn: give every die a run of consecutive tiles, which share operands
// in its L2.
__device__ __forceinline__ int die_order(int b, int n)
{
    const int q = n >> 3, r = n & 7, x = b & 7;
    return x * q + min(x, r) + (b >> 3);
}

// One 16-byte piece of the output: V neighbouring columns n .. n + V - 1 of row m (n a multiple of V).
template <typename CT, int V>
__device__ __forceinline__ void put_piece(const TileProb &p, int ks, int zb, int m, int n, float *v)
{
    typedef typename TileEl<CT>::elem elem;
    const TileOut &o = p.o;
    if (m >= p.M || n >= p.N) return;
    if (o.f32) {
        float *c = (float *)o.C + ks * o.split_stride + zb * p.sc + (i64)m * o.ld + n;
        const int nv = min(V, p.N - n);
        if (nv == V && !o.accumulate) {
#pragma unroll
            for (int e = 0; e < V; e += 4) stg16(c + e, floats_piece<float>(v + e));
        } else {
            for (int e = 0; e < V; ++e)
                if (e < nv) c[e] = o.accumulate ? c[e] + v[e] : v[e];
        }
        return;
    }
    i64 at;
    int nv;
    int pos = 0;
    if (o.HC > 0) {
        const int cn = n / V, img = cn / o.HC;
        pos = (cn - img * o.HC) * V;
        nv = min(V, o.HW - pos);
        if (img >= o.N) return;
        if (o.s > 1) {
            at = ((i64)img * o.CH + m) * ((i64)o.H * o.W);
        } else {
            at = ((i64)img * o.CH + m) * o.HW + pos;
        }
    } else {
        at = zb * p.sc + (i64)m * o.ld + n;
        nv = min(V, p.N - n);
    }
    elem *c = (elem *)o.C;
    const elem *add = (const elem *)o.add, *mask = (const elem *)o.mask, *bias = (const elem *)o.bias;
    const float sc = o.scale ? o.scale[m] : 1.f, sh = o.shift ? o.shift[m] : 0.f;
    if (o.scale || o.shift) {
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = v[e] * sc + sh;
    }
    if (nv == V && !(o.s > 1)) {
        float f[8];
        if (bias) {
            piece_floats<CT>(ldg16(bias + n), f);
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] += f[e];
        }
        if (add) {
            piece_floats<CT>(ldg16(add + at), f);
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] += f[e];
        }
        if (o.relu) {
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = fmaxf(v[e], 0.f);
        }
        if (mask) {
            piece_floats<CT>(ldg16(mask + at), f);
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = f[e] > 0.f ? v[e] : 0.f;
        }
        stg16(c + at, floats_piece<CT>(v));
        return;
    }
    int y = 0, x = 0;
    if (o.s > 1) y = pos / o.gW, x = pos - y * o.gW;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        if (e < nv) {
            i64 i = at + e;
            bool in = true;
            if (o.s > 1) {
                const int yy = y * o.s + o.ph, xx = x * o.s + o.pw;
                in = yy < o.H && xx < o.W;
                i = at + (i64)yy * o.W + xx;
                if (++x == o.gW) x = 0, ++y;
            }
            if (in) {
                union {
                    uint32_t w[4];
                    elem e[V];
                } u;
                float t = v[e];
                if (bias) t += sizeof(elem) == 4 ? ((const float *)bias)[n + e] : bf16_bits_to_float((uint16_t)bias[n + e]);
                if (add) t += sizeof(elem) == 4 ? ((const float *)add)[i] : bf16_bits_to_float((uint16_t)add[i]);
                if (o.relu) t = fmaxf(t, 0.f);
                if (mask)
                    t = (sizeof(elem) == 4 ? ((const float *)mask)[i] : bf16_bits_to_float((uint16_t)mask[i])) > 0.f ? t
                                                                                                                   : 0.f;
                if (sizeof(elem) == 4) u.w[0] = __float_as_uint(t);
                else u.w[0] = float_to_bf16_bits(t);
                c[i] = u.e[0];
            }
        }
    }
}

template <typename CT, class CFG, class LA, class LB>
__device__ __forceinline__ void finish(const TileProb &p, int ks, int zb, int m0, int n0, LA &la, bool sums, unsigned char *smem,
                                       int tid)
{
    constexpr int V = TileEl<CT>::V;
    tile_pieces<CT, CFG>(smem, tid, [&](int m, int n, float *v) { put_piece<CT, V>(p, ks, zb, m0 + m, n0 + n, v); });
    if (sums) {
        __syncthreads();
        float *out = p.o.sums + ks * p.o.sums_stride + zb * p.ssums;
        const bool acc = p.o.accumulate != 0;
        la.put_sums((float *)smem, tid, [&](int m, float v) {
            if (m0 + m < p.M) out[m0 + m] = acc ? out[m0 + m] + v : v;
        });
    }
}

// The argument block where the launch put it.  (Indexed by problem and, for the taps, by lane, the by-value parameter
// would be copied to scratch memory by every thread.)
__device__ __forceinline__ const TileArgs &tile_args(const TileArgs &a)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const TileArgs *)(const __attribute__((address_space(4))) TileArgs *)__builtin_amdgcn_kernarg_segment_ptr();
#else
    return a;
#endif
}

struct TileAt {
    int prob, ks, zb, m0, n0;
};
template <class CFG>
__device__ __forceinline__ TileAt find_tile(const TileArgs &a)
{
    TileAt t;
    const int b = die_order(blockIdx.x, a.blocks);
    t.prob = 0;
#pragma unroll
    for (int i = 1; i < TILE_MAX_PROBS; ++i)
        if (i < a.n && b >= a.p[i].block0) t.prob = i;
    const TileProb &p = a.p[t.prob];
    const int l = b - p.block0, per = p.tm * p.tn;
    const int zk = l / per, q = l - zk * per, tm = q / p.tn;
    t.zb = zk / p.ksplit;
    t.ks = zk - t.zb * p.ksplit;
    t.m0 = tm * CFG::BM;
    t.n0 = (q - tm * p.tn) * CFG::BN;
    return t;
}

template <typename CT, class CFG>
__global__ __launch_bounds__(TILE_THREADS) void tile_linear_kernel(TileArgs by_value)
{
    const TileArgs &a = tile_args(by_value);
    constexpr int BM = CFG::BM, BN = CFG::BN, BK = TileEl<CT>::BK;
    typedef LoadKC<CT, BM> AK;
    typedef LoadMC<CT, BM, true> AM;
    typedef LoadKC<CT, BN> BKC;
    typedef LoadMC<CT, BN> BMC;
    constexpr int s1 = TileSize<CT, CFG, AK, BKC>::bytes, s2 = TileSize<CT, CFG, AK, BMC>::bytes,
                  s3 = TileSize<CT, CFG, AM, BMC>::bytes;
    constexpr int bytes = s1 > s2 ? (s1 > s3 ? s1 : s3) : (s2 > s3 ? s2 : s3);
    __shared__ __attribute__((aligned(16))) unsigned char smem[bytes];
    const int tid = threadIdx.x;
    const TileAt t = find_tile<CFG>(a);
    const TileProb &p = a.p[t.prob];
    const int kbeg = t.ks * p.kper, kend = min(p.K, kbeg + p.kper), nch = (kend - kbeg + BK - 1) / BK;
    typedef typename TileEl<CT>::elem elem;
    const elem *A = (const elem *)p.A + t.zb * p.sa, *B = (const elem *)p.B + t.zb * p.sb;
    if (p.type == TILE_NT) {
        AK la;
        BKC lb;
        la.init(A, p.lda, p.M, p.K, t.m0, kbeg, tid);
        lb.init(B, p.ldb, p.N, p.K, t.n0, kbeg, tid);
        tile_product<CT, CFG>(la, lb, nch, smem, tid);
        tile_pieces<CT, CFG>(smem, tid, [&](int m, int n, float *v) {
            put_piece<CT, TileEl<CT>::V>(p, t.ks, t.zb, t.m0 + m, t.n0 + n, v);
        });
    } else if (p.type == TILE_NN) {
        AK la;
        BMC lb;
        la.init(A, p.lda, p.M, p.K, t.m0, kbeg, tid);
        lb.init(B, p.ldb, p.N, p.K, t.n0, kbeg, tid);
        tile_product<CT, CFG>(la, lb, nch, smem, tid);
        tile_pieces<CT, CFG>(smem, tid, [&](int m, int n, float *v) {
            put_piece<CT, TileEl<CT>::V>(p, t.ks, t.zb, t.m0 + m, t.n0 + n, v);
        });
    } else {
        AM la;
        BMC lb;
        la.init(A, p.lda, p.M, p.K, t.m0, kbeg, tid);
        lb.init(B, p.ldb, p.N, p.K, t.n0, kbeg, tid);
        tile_product<CT, CFG>(la, lb, nch, smem, tid);
        finish<CT, CFG, AM, BMC>(p, t.ks, t.zb, t.m0, t.n0, la, p.o.sums && t.n0 == 0, smem, tid);
    }
}

// filters [q][c][kk] -> [c][q][selected taps], one element per thread
template <typename CT>
__device__ __forceinline__ void pack_filters(const TileProb &p, int block, int tid)
{
    typedef typename TileEl<CT>::elem elem;
    const int nt = p.pb.ntap, kk = p.kper;
    const i64 total = (i64)p.M * p.N * nt; // M = channels c, N = rank
    const elem *src = (const elem *)p.A;
    elem *dst = (elem *)p.o.C;
    for (int u = 0; u < 4; ++u) {
        const i64 i = ((i64)block * 4 + u) * TILE_THREADS + tid;
        if (i >= total) return;
        const int t = (int)(i % nt);
        const i64 cq = i / nt;
        const int q = (int)(cq % p.N);
        const i64 c = cq / p.N;
        dst[i] = src[((i64)q * p.M + c) * kk + p.pb.dy[t]]; // (dy holds the index of the tap here)
    }
}

template <typename CT, class CFG, bool GATHER>
__global__ __launch_bounds__(TILE_THREADS) void tile_conv_kernel(TileArgs by_value)
{
    const TileArgs &a = tile_args(by_value);
    constexpr int BM = CFG::BM, BN = CFG::BN, BK = TileEl<CT>::BK;
    typedef LoadKC<CT, BM> AK;
    typedef LoadMC<CT, BM, false, true> AS;
    typedef LoadPixMC<CT, BN, false> BP;
    typedef LoadPixMC<CT, BN, true> BPG;
    typedef LoadPixKC<CT, BM, false, true> AW;
    typedef LoadPixKC<CT, BN, false> BW;
    typedef LoadPixKC<CT, BN, true> BWG;
    constexpr int s1 = TileSize<CT, CFG, AK, BP>::bytes, s2 = TileSize<CT, CFG, AS, BP>::bytes,
                  s3 = TileSize<CT, CFG, AW, BW>::bytes;
    constexpr int bytes = s1 > s2 ? (s1 > s3 ? s1 : s3) : (s2 > s3 ? s2 : s3);
    __shared__ __attribute__((aligned(16))) unsigned char smem[bytes];
    extern __shared__ __attribute__((aligned(16))) unsigned char tile_tables[];
    const int tid = threadIdx.x;
    const TileAt t = find_tile<CFG>(a);
    const TileProb &p = a.p[t.prob];
    const auto put = [&](int m, int n, float *v) { put_piece<CT, TileEl<CT>::V>(p, t.ks, t.zb, t.m0 + m, t.n0 + n, v); };
    const int nch = (p.K + BK - 1) / BK; // (not TILE_WG)
    if (p.type == TILE_CONV || (GATHER && p.type == TILE_CONVG)) {
        AK la;
        la.init(p.A, p.lda, p.M, p.K, t.m0, 0, tid);
        if (GATHER && p.type == TILE_CONVG) {
            BPG lb;
            lb.init(p.pb, t.n0, 0, tid, tile_tables);
            tile_product<CT, CFG>(la, lb, nch, smem, tid);
        } else {
            BP lb;
            lb.init(p.pb, t.n0, 0, tid, tile_tables);
            tile_product<CT, CFG>(la, lb, nch, smem, tid);
        }
        tile_pieces<CT, CFG>(smem, tid, put);
    } else if (p.type == TILE_CONVT) {
        AS la;
        BP lb;
        la.init(p.A, p.lda, p.M, p.K, t.m0, 0, tid, p.ascale);
        lb.init(p.pb, t.n0, 0, tid, tile_tables);
        tile_product<CT, CFG>(la, lb, nch, smem, tid);
        tile_pieces<CT, CFG>(smem, tid, put);
    } else if (p.type == TILE_PACK) {
        const int l = die_order(blockIdx.x, a.blocks) - p.block0;
        pack_filters<CT>(p, l, tid);
    } else {
        const int img0 = t.ks * p.kper, img1 = min(p.pa.N, img0 + p.kper);
        const int pieces = (img1 - img0) * p.pa.HC, n = (pieces + BK / TileEl<CT>::V - 1) / (BK / TileEl<CT>::V);
        AW la;
        unsigned char *tb = tile_tables + (AW::table_bytes(p.pa) + 15) / 16 * 16;
        la.init(p.pa, t.m0, img0, img1, tid, tile_tables);
        if (GATHER && p.type == TILE_WGG) {
            BWG lb;
            lb.init(p.pb, t.n0, img0, img1, tid, tb);
            __syncthreads();
            tile_product<CT, CFG>(la, lb, n, smem, tid);
        } else {
            BW lb;
            lb.init(p.pb, t.n0, img0, img1, tid, tb);
            __syncthreads();
            tile_product<CT, CFG>(la, lb, n, smem, tid);
        }
        finish<CT, CFG, AW, BW>(p, t.ks, t.zb, t.m0, t.n0, la, p.o.sums && t.n0 == 0, smem, tid);
    }
}

// ------------------------------------------------------------------ host side
struct ShapeInfo {
    int bm, bn;
};
static const ShapeInfo SHAPES[TS_COUNT] = {{32, 32}, {64, 64}, {128, 64}, {128, 128}, {32, 128}};

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

// A chunk costs a compute unit `work` cycles (its matrix instructions, or the LDS traffic of its fragments) when several
// workgroups keep it busy, and at least `lat` (the next chunk's loads, the LDS round trip, the barrier) when one is
// alone; every split costs a partial sum to write and to read, and the first of them one more launch.
struct ChunkCost {
    double work, one;
};
static ChunkCost chunk_cost(bool bf, TileShape sh)
{
    const double bm = SHAPES[sh].bm, bn = SHAPES[sh].bn;
    const double mma = (bm / 32) * (bn / 32) * (bf ? 4 * 32 : 16 * 64) / 4.0;
    const double wm = bm == 32 ? 1 : 2, wn = bn == 32 ? 1 : 2;
    const double lds = bm * wn + bn * wm + bm + bn;
    const double lat = bf ? 350 : 300;
    const double work = mma > lds ? mma : lds;
    return ChunkCost{work, work > lat ? work : lat};
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
    TileGroup best = {TS_64, {1, 1, 1, 1}, 1e30};
    for (TileShape sh : tries) {
        const ChunkCost cc = chunk_cost(bf, sh);
        const i64 bm = SHAPES[sh].bm, bn = SHAPES[sh].bn;
        for (int most = 2; most <= (1 << 20); most *= 2) { // chunks a workgroup of a split product may have
            TileGroup g = {sh, {1, 1, 1, 1}, 0};
            double total = 0, longest = 0, part = 0;
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
                total += (double)tiles * ks * (per * cc.work + 500 + bm * bn / 32.0);
                if (per * cc.one > longest) longest = per * cc.one;
            }
            g.cost = (total / 256 > longest ? total / 256 : longest) + 3000 + (any ? 6000 + part / 2000 : 0);
            if (g.cost < best.cost) best = g;
            if (last) break;
        }
    }
    return best;
}

void tile_add(TileArgs &a, TileShape shape, int dtype, const TileProb &q, int ksplit)
{
    TileProb &p = a.p[a.n++];
    p = q;
    const int bk = dtype == PF_BF16 ? 64 : 32;
    p.tm = (p.M + SHAPES[shape].bm - 1) / SHAPES[shape].bm;
    p.tn = (p.N + SHAPES[shape].bn - 1) / SHAPES[shape].bn;
    p.ksplit = ksplit < 1 ? 1 : ksplit;
    if (p.type == TILE_WG || p.type == TILE_WGG) {
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
    a.blocks += p.tm * p.tn * p.ksplit * p.nb;
}

template <typename CT, class CFG>
static int launch_linear(hipStream_t s, const char *name, const TileArgs &a)
{
    int st = PF_OK;
    PF_LAUNCH(st, name, (tile_linear_kernel<CT, CFG>), dim3(a.blocks), dim3(TILE_THREADS), s, a);
    return st;
}
template <typename CT>
static int launch_linear_t(hipStream_t s, const char *name, TileShape shape, const TileArgs &a)
{
    switch (shape) {
    case TS_32: return launch_linear<CT, TileCfg<32, 32, 1, 1, 4>>(s, name, a);
    case TS_64: return launch_linear<CT, TileCfg<64, 64, 2, 2, 4>>(s, name, a);
    case TS_128x64: return launch_linear<CT, TileCfg<128, 64, 2, 2, 2>>(s, name, a);
    case TS_128: return launch_linear<CT, TileCfg<128, 128, 2, 2, 2>>(s, name, a);
    default: return PF_ERR_UNSUPPORTED;
    }
}

int launch_tiles_linear(hipStream_t s, const char *name, int dtype, TileShape shape, const TileArgs &a)
{
    if (a.blocks <= 0) return PF_OK;
    return dtype == PF_F32 ? launch_linear_t<float>(s, name, shape, a) : launch_linear_t<bf16_t>(s, name, shape, a);
}

template <typename CT, class CFG>
static int launch_conv(hipStream_t s, const char *name, const TileArgs &a)
{
    typedef LoadPixMC<CT, CFG::BN, false> BP;
    int st = PF_OK, tab = 0;
    bool gather = false;
    for (int i = 0; i < a.n; ++i) {
        const TileProb &p = a.p[i];
        int b = BP::TAB;
        if (p.type == TILE_WG) b = (LoadPixKC<CT, 64, false>::table_bytes(p.pa) + 15) / 16 * 16 + LoadPixKC<CT, 64, false>::table_bytes(p.pb);
        if (p.type == TILE_WGG) b = (LoadPixKC<CT, 64, false>::table_bytes(p.pa) + 15) / 16 * 16 + LoadPixKC<CT, 64, true>::table_bytes(p.pb);
        if (b > tab) tab = b;
        gather = gather || p.type == TILE_CONVG || p.type == TILE_WGG;
    }
    tab = (tab + 15) / 16 * 16;
    if (gather) {
        PF_LAUNCH_LDS(st, name, (tile_conv_kernel<CT, CFG, true>), dim3(a.blocks), dim3(TILE_THREADS), tab, s, a);
    } else {
        PF_LAUNCH_LDS(st, name, (tile_conv_kernel<CT, CFG, false>), dim3(a.blocks), dim3(TILE_THREADS), tab, s, a);
    }
    return st;
}
template <typename CT>
static int launch_conv_t(hipStream_t s, const char *name, TileShape shape, const TileArgs &a)
{
    switch (shape) {
    case TS_32x128: return launch_conv<CT, TileCfg<32, 128, 1, 4, 4>>(s, name, a);
    case TS_64: return launch_conv<CT, TileCfg<64, 64, 2, 2, 4>>(s, name, a);
    case TS_128x64: return launch_conv<CT, TileCfg<128, 64, 2, 2, 2>>(s, name, a);
    default: return PF_ERR_UNSUPPORTED;
    }
}

int launch_tiles_conv(hipStream_t s, const char *name, int dtype, TileShape shape, const TileArgs &a)
{
    if (a.blocks <= 0) return PF_OK;
    return dtype == PF_F32 ? launch_conv_t<float>(s, name, shape, a) : launch_conv_t<bf16_t>(s, name, shape, a);
}

// ------------------------------------------------------------------ sums over splits
// Four outputs per thread where the arrays allow 16-byte accesses, up to eight splits in flight, added in order.
template <bool VEC>
__device__ __forceinline__ void split_sum(const SplitSum &q, i64 i)
{
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    const float *p = q.src + i;
    for (int s = 0; s < q.splits; s += 8) {
        f32x4_t t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float *r = p + (i64)min(s + u, q.splits - 1) * q.stride;
            if (VEC) t[u] = *(const f32x4_t *)r;
            else t[u][0] = *r;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s + u < q.splits) {
#pragma unroll
                for (int e = 0; e < (VEC ? 4 : 1); ++e) v[e] += t[u][e];
            }
    }
#pragma unroll
    for (int e = 0; e < (VEC ? 4 : 1); ++e) {
        float w = v[e];
        if (q.rscale) w *= q.rscale[(i + e) / q.rlen];
        if (q.bf16) ((uint16_t *)q.dst)[i + e] = float_to_bf16_bits(w);
        else q.dst[i + e] = q.accumulate ? q.dst[i + e] + w : w;
    }
}

__global__ __launch_bounds__(256) void split_sums_kernel(SplitSumArgs a)
{
    int k = 0;
#pragma unroll
    for (int i = 1; i < 4; ++i)
        if (i < a.n && (int)blockIdx.x >= a.blocks[i]) k = i;
    const SplitSum &q = a.s[k];
    const i64 b = blockIdx.x - a.blocks[k];
    if (q.count % 4 == 0 && q.stride % 4 == 0) { // (the partial sums start 256-byte aligned)
        const i64 i = (b * 256 + threadIdx.x) * 4;
        if (i < q.count) split_sum<true>(q, i);
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const i64 i = (b * 4 + u) * 256 + threadIdx.x;
            if (i < q.count) split_sum<false>(q, i);
        }
    }
}

void split_sum_add(SplitSumArgs &a, const SplitSum &s)
{
    if (!s.dst || s.count <= 0) return;
    a.s[a.n] = s;
    a.blocks[a.n + 1] = a.blocks[a.n] + (int)((s.count + 1023) / 1024);
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
