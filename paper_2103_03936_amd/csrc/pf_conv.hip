// Factorized convolution (paper Section 2.2): thin k x k convolution into r channels
// followed by a 1x1 convolution, forward and backward, plus the dense comparator.
// Host-side validation, workspace planning and dispatch; most shapes run on the tiled
// products (pf_tile.h), what those do not take as implicit GEMMs (operands gathered by
// functors) on the guarded element-wise GEMM.
#include "pf_conv_chain.h"
#include "pf_conv_px.h"
#include "pf_conv_wgrad.h"
#include "pf_epilogue.h"
#include "pf_tile_host.h"

#include <math.h>

namespace pf {

struct ConvGeom {
    int N, C, H, W, Cout, r, k, s, p, Ho, Wo;
};

// B(kidx = (c,i,j), n = (img,y,x)) = Xpad[img, c, y s + i - p, x s + j - p]
template <typename T>
struct OpB_Im2col {
    const T *X;
    ConvGeom g;
    __device__ __forceinline__ float at(int kidx, int n) const
    {
        const int kk = g.k * g.k;
        const int c = kidx / kk, t = kidx % kk, i = t / g.k, j = t % g.k;
        const int hw = g.Ho * g.Wo;
        const int img = n / hw, pix = n % hw, y = pix / g.Wo, x = pix % g.Wo;
        const int yy = y * g.s + i - g.p, xx = x * g.s + j - g.p;
        if (yy < 0 || yy >= g.H || xx < 0 || xx >= g.W) return 0.f;
        return to_float(X[(((i64)img * g.C + c) * g.H + yy) * g.W + xx]);
    }
    __device__ __forceinline__ float operator()(int k, int n, int) const { return at(k, n); }
};
// B(k = (img,y,x), n = (c,i,j)): the same view with the roles swapped (weight gradient)
template <typename T>
struct OpB_Im2colT {
    OpB_Im2col<T> v;
    __device__ __forceinline__ float operator()(int k, int n, int) const { return v.at(n, k); }
};

// Tensor P[img, ch, pix] (NCHW with HW flattened) seen as a matrix over (channel, pixel).
template <typename T>
struct OpB_NCHW { // B(k = ch, n = (img,pix))
    const T *p;
    int CH, HW;
    __device__ __forceinline__ float operator()(int k, int n, int) const
    {
        const int img = n / HW, pix = n % HW;
        return to_float(p[((i64)img * CH + k) * HW + pix]);
    }
};
template <typename T>
struct OpB_NCHW_T { // B(k = (img,pix), n = ch)
    const T *p;
    int CH, HW;
    __device__ __forceinline__ float operator()(int k, int n, int) const
    {
        const int img = k / HW, pix = k % HW;
        return to_float(p[((i64)img * CH + n) * HW + pix]);
    }
};
template <typename T>
struct OpA_NCHW { // A(m = ch, k = (img,pix))
    const T *p;
    int CH, HW;
    __device__ __forceinline__ float operator()(int m, int k, int) const
    {
        const int img = k / HW, pix = k % HW;
        return to_float(p[((i64)img * CH + m) * HW + pix]);
    }
};

// A(m = c, kidx = (q,i,j)) = Uk[q, c, i, j]
template <typename T>
struct OpA_FilterT {
    const T *Uk;
    int C, kk;
    __device__ __forceinline__ float operator()(int m, int kidx, int) const
    {
        const int q = kidx / kk, t = kidx % kk;
        return to_float(Uk[((i64)q * C + m) * kk + t]);
    }
};

// B(kidx = (q,i,j), n = (img,yy,xx)) = dT[img, q, y, x] where y s + i - p = yy, x s + j - p = xx
template <typename T>
struct OpB_Col2im {
    const T *dT;
    ConvGeom g;
    int CH; // channels of dT
    __device__ __forceinline__ float operator()(int kidx, int n, int) const
    {
        const int kk = g.k * g.k;
        const int q = kidx / kk, t = kidx % kk, i = t / g.k, j = t % g.k;
        const int hw = g.H * g.W;
        const int img = n / hw, pix = n % hw, yy = pix / g.W, xx = pix % g.W;
        const int ys = yy + g.p - i, xs = xx + g.p - j;
        if (ys < 0 || xs < 0 || ys % g.s || xs % g.s) return 0.f;
        const int y = ys / g.s, x = xs / g.s;
        if (y >= g.Ho || x >= g.Wo) return 0.f;
        return to_float(dT[(((i64)img * CH + q) * g.Ho + y) * g.Wo + x]);
    }
};

// C(m = ch, n = (img,pix)) -> P[img, ch, pix], optionally to a second buffer
template <typename T1, typename T2>
struct EpiNCHW {
    T1 *c1;
    T2 *c2;
    int CH, HW;
    __device__ __forceinline__ void operator()(int m, int n, float acc, int, int) const
    {
        const int img = n / HW, pix = n % HW;
        const i64 off = ((i64)img * CH + m) * HW + pix;
        if (c1) c1[off] = from_float<T1>(acc);
        if (c2) c2[off] = from_float<T2>(acc);
    }
};

// ------------------------------------------------------------ validation
static int check_conv_desc(const pf_conv_desc *d, ConvGeom *g)
{
    if (!d) return PF_ERR_NULL;
    if (d->dtype != PF_F32 && d->dtype != PF_BF16) return PF_ERR_UNSUPPORTED;
    if (d->layout != PF_NCHW || d->wgrad_dtype != PF_F32) return PF_ERR_UNSUPPORTED;
    if (d->N < 0 || d->Cin <= 0 || d->H <= 0 || d->W <= 0 || d->Cout <= 0 || d->r <= 0) return PF_ERR_SHAPE;
    if (d->k <= 0 || d->stride <= 0 || d->pad < 0 || d->k > 15) return PF_ERR_SHAPE;
    const i64 Ho = (d->H + 2 * (i64)d->pad - d->k) / d->stride + 1, Wo = (d->W + 2 * (i64)d->pad - d->k) / d->stride + 1;
    if (d->H + 2 * (i64)d->pad < d->k || d->W + 2 * (i64)d->pad < d->k || Ho <= 0 || Wo <= 0) return PF_ERR_SHAPE;
    const i64 lim = 0x7fffffffLL;
    if (d->N * d->H * d->W > lim || d->N * Ho * Wo > lim || d->Cin * d->k * d->k > lim || d->r * d->k * d->k > lim ||
        d->Cout > lim || d->r > lim)
        return PF_ERR_SHAPE;
    if (d->N * d->Cin * d->H * d->W > (lim << 4) || d->N * d->Cout * Ho * Wo > (lim << 4)) return PF_ERR_SHAPE;
    if (g) *g = ConvGeom{(int)d->N, (int)d->Cin, (int)d->H, (int)d->W, (int)d->Cout, (int)d->r,
                         d->k,      d->stride,   d->pad,    (int)Ho,   (int)Wo};
    return PF_OK;
}

// What the kernels apply as they store their output (all optional): forward scale / shift / residual / ReLU,
// backward the gradient arriving over a skip connection and the mask of a ReLU input.
struct ConvEpilogue {
    const float *scale, *shift;
    const void *add, *mask;
    int relu;
    float *dshift; // backward: sums of dZ per channel
};

struct ConvPlan {
    int ks_dVp, ks_dUk;
    size_t n_T, n_part, fwd_bytes, bwd_bytes;
    bool chain;              // the fused small-image kernel applies (bf16 only)
    bool wgrad;              // the small-image filter-gradient kernel applies (bf16 only)
    int wg_groups, wg_ipg;   // image groups and images per group of that kernel, k x k stage
    int wg_groups2, wg_ipg2; // the same for the 1x1 stage
    size_t n_w1, n_w2;       // packed weight elements, forward direction
    size_t n_w1b, n_w2b;     // packed weight elements, backward direction
    bool tiles;              // the tiled products of pf_tile.h take the shape
    bool gather;             // ... and read the k x k stage's input with stride
    TileShape sh_T, sh_Y, sh_dT, sh_g, sh_w; // ... the tile shapes of their launches
    int ks_T, ks_dT;         // ... splits of the products that give T and dT
    int ks_tU, ks_tV;        // ... image splits of the two filter gradients
    i64 t_U, t_V;            // ... and their tiles
    size_t n_part_T;         // ... their partial sums (floats)
    size_t n_pack, n_part_t; // ... re-ordered filters (elements), partial sums (floats)
    int px_fwd, px_fwd_threads; // pixels and threads per workgroup of the pixel-major kernels where they take the direction, 0: not
    bool plain_chain, plain_chain_kept; // ... but the chain kernel takes the calls without an epilogue; those that keep filters for px_bwd
    int px_bwd, px_bwd_threads;
    int px_groups[2], px_per[2]; // ... and the pixel groups of their filter gradients, tiles per group
    size_t px_pack, px_dT, px_part; // ... elements of the re-ordered thin filters and of dT, floats of the partial sums
    size_t saved_bytes;      // the backward direction's packed weights when the forward call saves them
};

// Which filter taps reach the input pixels (s y + a) of one phase of a strided convolution's input gradient, and the
// row of dT each of them reads relative to y: y s + a + p = i + s (row), i.e. row = y + (a + p - i) / s.
static int phase_taps(const ConvGeom &g, int a, int *tap, int *off)
{
    int n = 0;
    for (int i = 0; i < g.k; ++i)
        if ((a + g.p - i) % g.s == 0) {
            tap[n] = i;
            off[n++] = (a + g.p - i) / g.s;
        }
    return n;
}

// The convolution on the tiled products (pf_tile.h): every extent holds a 16-byte piece, the filter fits the tap
// table, and the grids of forward and backward have the row length of the planes they read (always for unit stride
// with same padding; for stride s when no input pixel lies beyond s * output extent).
static void plan_conv_tiles(const ConvGeom &g, int dtype, ConvPlan &p)
{
    const int V = dtype == PF_BF16 ? 8 : 4, kk = g.k * g.k, HW = g.Ho * g.Wo;
    const i64 big = 1LL << 30;
    p.tiles = false;
    if (g.N < 1 || kk > TILE_MAX_TAPS || g.C < 1 || (i64)g.C * kk < V || g.r < V || g.Cout < 1) return;
    const i64 planes = (i64)g.N * HW;
    if (planes * g.r < V || planes * g.Cout < V || (i64)g.N * g.C * g.H * g.W < V) return;
    // (32-bit byte offsets, a row of channels past the end included)
    const i64 lim = (1LL << 31) / (16 / V) - (1 << 20), over = 400LL * (HW > g.H * g.W ? HW : g.H * g.W);
    if (planes * g.r + over > lim || planes * g.Cout + over > lim || (i64)g.N * g.C * g.H * g.W + over > lim) return;
    const int HC = (HW + V - 1) / V, HCin = (g.H * g.W + V - 1) / V;
    if ((i64)g.N * HC * V > big || (i64)g.N * HCin * V > big) return;
    const bool same = g.s == 1 && g.Ho == g.H && g.Wo == g.W;
    // gather: the k x k stage reads X by element offsets; backward needs one grid of Ho x Wo pixels per phase
    if (!same && !(g.s > 1 && (g.H + g.s - 1) / g.s <= g.Ho && (g.W + g.s - 1) / g.s <= g.Wo && g.s <= 2)) return;
    p.gather = !same;
    const int tab = 2 * (4096 + (kk * HC + 15) / 16 * 16 + (p.gather ? 4 * V * HC : 0));
    if (tab > 28 * 1024) return;
    p.tiles = true;
    const i64 npx = (i64)g.N * HC * V;
    p.sh_Y = g.Cout <= 32 ? TS_32x64 : g.Cout >= 128 && (g.Cout + 127) / 128 * ((npx + 63) / 64) >= 512 ? TS_128x64 : TS_64;
    // T and dT: too few tiles for the chip split their contraction (at least four chunks each)
    const auto split_k = [&](i64 K, i64 bm, i64 &tiles) {
        tiles = (g.r + bm - 1) / bm * ((npx + 63) / 64);
        const i64 chunks = (K + 8 * V - 1) / (8 * V);
        i64 ks = tiles >= 200 ? 1 : 384 / tiles;
        if (ks > chunks / 4) ks = chunks / 4;
        if (ks > 16) ks = 16;
        return (int)(ks < 1 ? 1 : ks);
    };
    // Tiles that leave half the chip idle, splits and all: half as high, for a chunk of theirs takes half the time and they are twice as many.
    // Both directions, us, 64 x 64 / 32 x 64, at most 128 of them: float 6 x 224 x 5 x 5, rank 39 60.0 / 54.4, 26 x 256 x 8 x 8, rank 64, stride 2
    // 64.8 / 60.3, bf16 22 x 384 x 5 x 5, rank 80 56 / 53.5; with a full chip they are the slower ones (float 6 x 396 x 16 x 16, rank 99, T in
    // 384 workgroups 110 / 118); bf16 T and dT from 64 on (36 x 343 x 12 x 12, rank 61, 81 tiles 45 / 46.4).
    const auto mid = [&](i64 K, bool taps, TileShape &shape, int &ks) {
        i64 tiles = 0;
        ks = split_k(K, 64, tiles);
        shape = g.r <= 32 || tiles * ks <= (dtype == PF_BF16 ? 64 : 128) ? TS_32x64 : TS_64;
        if (shape == TS_32x64) ks = split_k(K, 32, tiles);
        // Short chains without a split, where it would cost more than it saves: a launch for the sums (4.3 us and their bytes) against chunks of
        // 0.5 us in float, 0.3 in bf16, while a compute unit has one or two tiles.  Both directions, us, split / not: float 128 x 128 x 16 x 16 ->
        // 256, rank 64, stride 2 105.7 / 102.0, 26 x 256 x 8 x 8 59.3 / 56.8, 75 x 512 x 18 x 7, rank 151, 1 x 1 138 / 131; bf16 12 x 464 x 4 x 4 51.8 /
        // 49.8; but float 2 x 192 x 13 x 13 -> 448, 14 chunks 56.0 / 58.5.
        const bool bf = dtype == PF_BF16;
        const double chunks = (double)((K + 8 * V - 1) / (8 * V)), low = (double)((g.r + 31) / 32 * ((npx + 63) / 64)) / 256;
        const double alone = chunks * (bf ? 0.3 : 0.5) * (low > 1 ? low : 1);
        if (!taps && ks > 1 && low <= 2 && alone < 3.3 + ks * g.r * npx * 2.7e-6 + alone / ks) shape = TS_32x64, ks = 1;
    };
    mid((i64)g.C * kk, kk > 1 || p.gather, p.sh_T, p.ks_T);
    mid(g.Cout, false, p.sh_dT, p.ks_dT);
    if (p.sh_Y == TS_64 && (g.Cout + 63) / 64 * ((npx + 63) / 64) <= 128) p.sh_Y = TS_32x64;
    const size_t part_T = (size_t)(p.ks_T > p.ks_dT ? p.ks_T : p.ks_dT) * g.r * npx;
    p.n_part_T = p.ks_T > 1 || p.ks_dT > 1 ? part_T : 0;
    // dX in float, beside the gradients: 9 x 272 x 5 x 5 71 / 65, 4 x 448 x 13 x 13 92 / 83; 52 x 64 x 9 x 9, 134 tiles 50 / 57; bf16 3 x 320 x 12 x
    // 12 48 / 51; the phases of stride 2 within 3 % either way.
    p.sh_g = dtype == PF_F32 && g.s == 1 && (g.C + 63) / 64 * ((npx + 63) / 64) <= 96 ? TS_32x64 : TS_64;
    p.sh_w = g.r <= 32 ? TS_32x128 : TS_64;
    // both filter gradients in one launch: about two workgroups per compute unit, each at least four chunks long.  With at most 32
    // filters the gradients of both stages have the rank as their rows (dVp is formed transposed).
    const bool low = p.sh_w == TS_32x128;
    const i64 tU = low ? ((i64)g.C * kk + 127) / 128 : ((g.r + 63) / 64) * (((i64)g.C * kk + 63) / 64);
    const i64 tV = low ? (g.Cout + 127) / 128 : ((g.Cout + 63) / 64) * ((g.r + 63) / 64);
    const i64 want = 512;
    const auto split = [&](i64 tiles, i64 floats) {
        i64 ks = (want + tiles - 1) / tiles;
        const i64 chunks = (i64)g.N * HC * V / (dtype == PF_BF16 ? 64 : 32);
        if (ks > chunks / 4) ks = chunks / 4;
        if (ks > g.N) ks = g.N;
        if (ks > 64) ks = 64;
        while (ks > 1 && ks * floats > (4 << 20)) --ks;
        if (ks < 1) ks = 1;
        const i64 per = (g.N + ks - 1) / ks;
        return (int)((g.N + per - 1) / per);
    };
    p.t_U = tU, p.t_V = tV;
    p.ks_tU = split(tU, (i64)g.r * g.C * kk);
    p.ks_tV = split(tV, (i64)g.Cout * (g.r + 1));
    p.n_pack = kk > 1 || g.s > 1 ? (size_t)g.r * g.C * kk : 0;
    p.n_part_t = (size_t)p.ks_tU * g.r * g.C * kk + (size_t)p.ks_tV * ((size_t)g.Cout * g.r + g.Cout) + 320;
}

// The pixel-major kernels (pf_conv_px.h): which takes a direction, and whether one does.  Costs in microseconds, fitted to times of 190
// shapes in bf16, 140 in float and 100 with stride over 1 to 256 images of 4 x 4 to 32 x 32 pixels, 32 to 2048 channels, ranks 1 to 128
// (3 to 15 % rms).
// A workgroup of P pixels costs a fixed part, one for the filters that it reads (per 64 channels and 32 ranks), one per chunk of
// input channels and per 64 output channels, one where planes are not whole 16-byte pieces, and memory traffic as far as the chip is full;
// small tiles read the filters more often, large ones leave compute units idle.
struct PxCost {
    int P, threads, CH; // pixels, threads, channels of a chunk
    double round, filters, chunk, out, ragged, traffic, launch;
    double wg, wg_part, wg_both; // backward: the filter gradients' share
};
static const PxCost PX_FWD[] = {{128, 512, 128, 3.12, 0.17, 0.00, 0.72, 0.43, 0.32, 3.54}, {64, 512, 128, 3.15, 0.11, 0.23, 0.43, 0.37, 0.12, 2.81},
                                {32, 512, 256, 4.03, 0.09, 0.00, 0.09, 0.22, 0.08, 2.73},  {128, 256, 64, 0.00, 0.28, 0.00, 1.70, 0.66, 0.94, 4.27},
                                {64, 256, 64, 0.33, 0.16, 0.00, 1.01, 0.62, 0.58, 4.15},   {32, 256, 128, 1.27, 0.14, 0.00, 0.37, 0.37, 0.37, 3.93}};
static const PxCost PX_FWD_F32[] = {{128, 512, 64, 0.12, 1.11, 0.79, 1.10, 0.30, 1.44, 6.59}, {64, 512, 64, 1.26, 0.60, 0.98, 0.73, 0.29, 0.72, 3.93},
                                    {32, 512, 128, 3.22, 0.39, 0.69, 0.25, 0.17, 0.33, 2.66}};
static const PxCost PX_FWD_STRIDED[] = {{32, 512, 128, 2.97, 0.08, 0.77, 0.11, 0.20, 0.17, 3.29}, {64, 512, 128, 5.99, 0.13, 1.37, 0.17, 0.00, 1.19, 0.00}};
static const PxCost PX_FWD_STRIDED_F32[] = {{32, 512, 64, 0.36, 0.36, 0.87, 0.04, 0.07, 1.15, 6.65}, {64, 512, 64, 6.22, 0.43, 0.93, 0.79, 0.41, 1.12, 0.00}};
static const PxCost PX_BWD[] = {{128, 512, 128, 1.58, 0.19, 0.35, 0.70, 0.64, 0.13, 15.50, 0.74, 0.00, 2.52},
                                {64, 512, 128, 1.48, 0.13, 0.30, 0.29, 0.56, 0.00, 15.46, 0.54, 0.32, 4.55},
                                {32, 512, 256, 4.46, 0.11, 0.21, 0.00, 0.41, 0.06, 13.32, 0.21, 0.00, 5.34},
                                {128, 256, 64, 2.13, 0.20, 0.24, 1.50, 0.91, 0.27, 13.62, 0.77, 7.71, 1.86},
                                {64, 256, 64, 0.00, 0.12, 0.25, 0.81, 0.87, 0.00, 15.60, 0.81, 11.55, 2.47},
                                {32, 256, 128, 0.00, 0.09, 0.03, 0.23, 0.60, 0.00, 16.59, 1.14, 13.10, 2.17}};
static const PxCost PX_BWD_F32[] = {{128, 512, 64, 0.72, 2.06, 0.14, 0.13, 0.51, 2.81, 18.49, 0.81, 0.00, 0.00},
                                    {64, 512, 64, 2.64, 1.08, 1.03, 0.00, 0.49, 1.55, 15.49, 0.44, 12.60, 0.00},
                                    {32, 512, 128, 2.69, 0.00, 3.07, 0.38, 0.56, 1.04, 15.13, 0.00, 37.05, 0.00}};
// Whether they take a direction: the estimate, corrected, against that of the tiled products, both of the geometric mean of a call without
// epilogue and one with, fitted to 2050 shapes forward and 1130 backward, half of them of 60 to 4000 pixels, planes of 3 x 3 to 80 x 80 (6
// to 10 % rms, hence the margins).  Over these shapes a call is 1.52 (bf16) and 1.30 times (float) as fast forward as on the tiled products
// alone, 1.20 and 1.5 backward; of a hundred shapes two are more than 5 % slower.  These kernels are the slower ones where a few
// workgroups pass through many channels, which the tiled products deal out (us, tiled / here: 1 image of 992 x 4 x 4 -> 128, rank 57, 3 x 3
// 20 / 30, 7 of 816 x 3 x 3 -> 168 backward 22 / 38), and in float where a large plane's traffic counts (215 of 64 x 40 x 40, stride 2 92 / 113).
struct PxCorrection {
    double estimate, outputs, ragged_outputs, rounds; // forward: per round, of it and a piece of output channels (as that, in ragged planes); per round after the first
};
static const PxCorrection PX_FWD_COR[2][2] = {{{0.907, 0.894, 0.5, 0.765}, {0.956, 0.853, 0, 1.717}}, // stride 1: bf16, float
                                              {{0.933, 0.699, 0.817, 0}, {0.968, 0.567, 1.168, 2.18}}}; // more
struct PxBwdCorrection {
    double estimate, ragged, odd, in, out, chain, chain_ranks; // per round in ragged planes, with ranks that are not whole pieces; per 10^7
                                                              // elements of dX, of dZ; per round and 64 channels of dZ, and 32 ranks of them
};
static const PxBwdCorrection PX_BWD_COR[2] = {{0.861, 1.131, 1.04, 4.777, 3.669, 0.214, 0.089}, {0.833, 0.602, 0.411, 7.081, 9.211, 0, 0}};
// The tiled products: the launches, one more where the first stage's contraction is split; its chain of chunks (times the rounds that its
// workgroups need), 10^7 terms of 32 ranks, 10^6 partial sums; the second stage's chain, 10^7 elements out and in; ragged planes, and their
// elements and terms.  Backward the first stage is dT; then dX and both gradients side by side: rounds of chunks, the longest chain,
// 10^6 partial sums and factor elements.
struct TiledFwdCost {
    double launches, split, chain, thin, part, wide, out, in, ragged, ragged_elements;
};
static const TiledFwdCost TILED_FWD[2][2] = {{{8.711, 4.405, 0.504, 0.316, 2.025, 1.544, 14.777, 1.258, 3.646, 0.365}, {8.991, 4.409, 0.614, 4.427, 1.936, 3.136, 22.369, 0.358, 2.782, 0.412}},
                                             {{9.495, 4.275, 1.468, 1.13, 2.693, 2.383, 6.862, 2.389, 2.878, 5.239}, {8.73, 3.831, 0.951, 4.24, 1.457, 4.34, 14.368, 3.389, 2.024, 3.259}}};
// The chain kernel, planes of 8 x 8, of 7 x 7 and others, over 313 shapes of 1 to 256 images (plain calls 4 to 7 % rms, with epilogue 11 to 13):
// an image, 32 ranks of 64 terms and of 64 output channels, a full chip's 4096 elements in or out, 64 input channels.  (7 x 7 with epilogue: 0.327
// per output channel fits best, but makes 512 -> 2048 of rank 128, 45 us, 53.)
struct ChainCost {
    double image, thin, wide, move, in;
};
static const ChainCost CHAIN_PLAIN[3] = {{8.54, 0.0526, 0.1001, 0.1915, 0.0531}, {8.011, 0.0609, 0.1075, 0.2105, 0.0297}, {9.6, 0.0655, 0.116, 0.2988, 0.1316}};
static const ChainCost CHAIN_EP[3] = {{9.422, 0.0511, 0.3086, 0.1989, 0.0858}, {9.345, 0.0596, 0.26, 0.128, 0.0302}, {11.113, 0.0658, 0.3066, 0.3898, 0.0964}};
struct TiledBwdCost {
    double launches, split, chain, rounds, longest, part, factors, in, out, ragged, ragged_elements;
};
static const TiledBwdCost TILED_BWD[2] = {{14.609, 3.899, 0.493, 0.348, 0.854, 2.17, 0, 24.072, 3.553, 5.189, 2.854},
                                          {14.145, 3.915, 0.894, 1.727, 1.092, 0, 36.439, 18.785, 1.8, 4.532, 12.376}};

template <typename T>
static void plan_conv_px(const ConvGeom &g, ConvPlan &p)
{
    constexpr bool f32 = sizeof(T) == 4;
    constexpr int V = PxEl<T>::V, S = PxEl<T>::S;
    if (!p.tiles || !px_fits<T>(g.N, g.C, g.H, g.W, g.Cout, g.r, g.k, g.s, g.p, g.Ho, g.Wo)) return;
    const PxPlane<S> pl = px_plane<S>(g.N, g.H, g.W, g.k), po = px_plane<S>(g.N, g.Ho, g.Wo, 1);
    const i64 npx = (i64)g.N * g.Ho * g.Wo;
    const int kk = g.k * g.k, RB = px_rank_blocks(g.r), s1 = px_slab<T>(g.k, g.r), s2 = px_slab<T>(1, g.r);
    const double ragged = g.Ho * g.Wo % V ? 1 : 0, filters = (g.C * kk + g.Cout) * RB / 64.0, mf = 1e-6 * g.r * ((double)g.C * kk + g.Cout);
    const double wg = (npx + 127) / 128 / 256.0 *
                      ((g.C + s1 - 1) / s1 * px_wgrad_cost<T>(g.k, g.r) + (g.Cout + s2 - 1) / s2 * px_wgrad_cost<T>(1, g.r)) * (1 + 0.2 * ragged);
    // in: channels of the direction's input, out: of its output
    const auto best = [&](const auto &list, int in, int out, int &P, int &threads) {
        double least = 1e30;
        for (const PxCost &c : list) {
            const i64 tiles = (npx + c.P - 1) / c.P, room = c.threads == 256 ? 512 : 256, rounds = (tiles + room - 1) / room;
            if ((g.r > 64 && c.threads == 256) || (g.s > 1 && kk == 9 && c.P == 64) || !px_tile_fits(pl, po, g.s, c.P)) continue;
            const double full = tiles < room ? (double)tiles / room : 1;
            const double t = c.launch + c.wg * wg + 4 * c.wg_part * mf + c.wg_both * sqrt(4 * wg * mf) +
                             rounds * (c.round + c.filters * filters + c.chunk * ((in + c.CH - 1) / c.CH) + c.out * out / 64 +
                                       c.ragged * ragged * (in + 2 * out) / 64 + c.traffic * full * (in + out) / 64);
            if (t < least) least = t, P = c.P, threads = c.threads;
        }
        return least;
    };
    const double m = npx * 1e-7, padded = (double)((g.Ho * g.Wo + V - 1) / V * V) * g.N, ragged_m = ragged * m * (g.C * kk + g.Cout);
    // rounds that workgroups of 64 columns and `rows` of `of` rows need, two to a compute unit
    const auto turns = [&](int of, int rows, int ks) {
        const double r = (double)((of + rows - 1) / rows) * ceil(padded / 64) * ks / 512;
        return r < 1 ? 1 : r;
    };
    const int rows1 = g.r <= 32 ? 32 : 64, K = 8 * V; // of the first stage; a chunk of a contraction
    const auto chunks = [&](int n) { return (n + K - 1) / K; };
    const auto tiled_fwd = [&](const TiledFwdCost &c) {
        return c.launches + c.split * (p.ks_T > 1) + c.chain * turns(g.r, rows1, p.ks_T) * chunks(g.C * kk) / p.ks_T + c.thin * m * RB * g.C * kk +
               (p.ks_T > 1 ? c.part * 1e-6 * p.ks_T * g.r * padded : 0) + c.wide * turns(g.Cout, 64, 1) * chunks(g.r) + c.out * m * g.Cout +
               c.in * 1e-7 * g.N * g.H * g.W * g.C + c.ragged * ragged + c.ragged_elements * ragged_m;
    };
    const auto tiled_bwd = [&](const TiledBwdCost &c) {
        const double runs = padded / (f32 ? 32 : 64), rows = chunks(g.r * kk), U = runs / p.ks_tU, W = runs / p.ks_tV;
        return c.launches + c.split * (p.ks_dT > 1) + c.chain * turns(g.r, rows1, p.ks_dT) * chunks(g.Cout) / p.ks_dT +
               c.rounds * (ceil(g.C / 64.0) * ceil(padded / 64) * rows + (p.t_U + p.t_V) * runs) / 512 + c.longest * (rows > U ? (rows > W ? rows : W) : U > W ? U : W) +
               c.part * 1e-6 * ((double)p.ks_tU * g.r * g.C * kk + (double)p.ks_tV * g.Cout * g.r) + c.factors * mf + c.in * m * g.C + c.out * m * g.Cout +
               c.ragged * ragged + c.ragged_elements * ragged_m;
    };
    const auto rounds = [&](int P, int threads) { return (double)(((npx + P - 1) / P + (threads == 256 ? 511 : 255)) / (threads == 256 ? 512 : 256)); };
    // the chain kernel's shapes: one workgroup per image streams both factors
    const auto chain = [&](const ChainCost (&list)[3]) {
        const ChainCost &c = list[g.H != g.W || (g.H != 7 && g.H != 8) ? 2 : g.H == 7];
        return (g.N + 255) / 256 * (c.image + RB / 64.0 * (c.thin * g.C * kk + c.wide * g.Cout) + c.in * g.C / 64) +
               (g.N < 256 ? g.N / 256.0 : 1) * c.move * g.H * g.W / 4096 * (g.C + g.Cout);
    };
    int P = 0, threads = 0;
    double t;
    if constexpr (f32) t = g.s > 1 ? best(PX_FWD_STRIDED_F32, g.C, g.Cout, P, threads) : best(PX_FWD_F32, g.C, g.Cout, P, threads);
    else t = g.s > 1 ? best(PX_FWD_STRIDED, g.C, g.Cout, P, threads) : best(PX_FWD, g.C, g.Cout, P, threads);
    if (P) {
        const int at_once = px_outputs(RB, P, threads);
        const double n = rounds(P, threads), pieces = n * ((g.Cout + at_once - 1) / at_once);
        bool takes;
        if (p.chain) {
            takes = 0.92 * t + 0.852 * pieces < 0.95 * chain(CHAIN_EP);
            // Calls without an epilogue stay with the chain kernel where it is the faster one, us, chain / here: 128 images of 256 x 8 x 8, rank
            // 64, 3 x 3 14.3 / 14.2, and 37.8 / 40.5 with the backward direction, replayed from a graph (its filters are kept beside: hence the wide
            // margin); 94 of 512 -> 1024 21.3 / 24.9; one tap, rank 128, 134 of 256 -> 1024 18.0 / 20.8, but 28 of 512 -> 256 12.5 / 9.5
            // ... and where filters are to be kept for the pixel-major backward direction, if it pays the launch that re-orders them as well: 33
            // images of 512 x 5 x 9 -> 2048, rank 128, one tap 27.6 / 37.1
            const double here = 0.824 * t + 0.318 * pieces, there = chain(CHAIN_PLAIN);
            p.plain_chain = here >= 0.86 * there;
            p.plain_chain_kept = here >= there + 4;
        } else {
            const PxCorrection &c = PX_FWD_COR[g.s > 1][f32];
            t = c.estimate * t + (c.outputs + c.ragged_outputs * ragged) * pieces + c.rounds * (n - 1);
            takes = t < (f32 ? 0.9 : 0.95) * tiled_fwd(TILED_FWD[g.s > 1][f32]);
        }
        if (takes) p.px_fwd = P, p.px_fwd_threads = threads;
    }
    // backward: unit stride
    if (g.s > 1 || !px_bwd_takes<T>(g.k, g.r) || (p.chain && p.wgrad) || !px_wgrad_fits(pl)) return;
    P = 0;
    if constexpr (f32) t = best(PX_BWD_F32, g.Cout, g.C, P, threads);
    else t = best(PX_BWD, g.Cout, g.C, P, threads);
    const PxBwdCorrection &c = PX_BWD_COR[f32];
    if (!P) return;
    t = c.estimate * t + m * (c.in * g.C + c.out * g.Cout) +
        rounds(P, threads) * (c.ragged * ragged + c.odd * (g.r % 8 ? 1 : 0) + (c.chain + c.chain_ranks * RB) * g.Cout / 64);
    if (!p.chain && t >= 0.95 * tiled_bwd(TILED_BWD[f32])) return;
    p.px_bwd = P, p.px_bwd_threads = threads;
    px_wgrad_plan<T>((int)npx, g.r, g.C, g.k, g.Cout, p.px_groups, p.px_per);
    p.px_pack = px_pack_elems(g.C, g.r, g.k);
    p.px_dT = (size_t)npx * px_ranks<T>(g.r);
    p.px_part = (size_t)p.px_groups[0] * g.r * g.C * kk + (size_t)p.px_groups[1] * g.Cout * (g.r + 1) + 256;
}

static ConvPlan make_conv_plan(const ConvGeom &g, int dtype)
{
    ConvPlan p;
    p.chain = dtype == PF_BF16 && chain_supported(g.C, g.Cout, g.r, g.H, g.W, g.k, g.s, g.p);
    // One workgroup per image, 64 pixel columns whatever the image has: of 3x3 layers the tiled products are faster where most
    // of the columns would be empty (4 x 4 images, 512 channels, forward and backward together, tiled against chain: rank 128
    // 51 against 76 us at batch 4, 86 against 97 at 128, equal at 256; rank 64 45 against 50 and 66 against 69) and where a few
    // images would have to stream megabytes of filters through a few compute units (7 x 7 images, rank 128: 57 against 66 us
    // at batch 4, 67 against 70 at 16, 83 against 74 at 32).  Of 1x1 layers they never are (4 x 4 images: 37 against 36 us at
    // batch 4, 59 against 49 at 256; 7 x 7, 2048 -> 512: 49 against 48 and 182 against 77).
    plan_conv_tiles(g, dtype, p);
    if (p.tiles && g.k == 3 && (g.H * g.W < 32 || (g.r > 64 && g.N < 32))) p.chain = false;
    p.n_w1 = chain_w1_elems(g.C, g.r, g.k);
    p.n_w2 = chain_w2_elems(g.Cout, g.r, 1);
    p.n_w1b = chain_w1_elems(g.Cout, g.r, 1);
    p.n_w2b = chain_w2_elems(g.C, g.r, g.k);
    p.wgrad = p.chain && wgrad_supported(g.r, g.C, g.H, g.W, g.k, g.s, g.p) &&
              wgrad_supported(g.r, g.Cout, g.H, g.W, 1, 1, 0);
    p.px_fwd = p.px_bwd = 0;
    p.plain_chain = p.plain_chain_kept = false;
    if (dtype == PF_BF16) plan_conv_px<uint16_t>(g, p);
    else plan_conv_px<float>(g, p);
    // (saved by a forward call for the kernels that take the backward direction)
    p.saved_bytes = p.px_bwd ? (p.px_fwd ? align_up(p.px_pack * (dtype == PF_BF16 ? 2 : 4)) : 0) : p.chain ? align_up(p.n_w1b * 2) + align_up(p.n_w2b * 2) : 0;
    p.wg_groups = p.wg_ipg = p.wg_groups2 = p.wg_ipg2 = 1;
    if (p.wgrad && g.N > 0) {
        // Image groups of the two problems of the launch.  A problem has `units` independent output blocks;
        // with g groups it runs units * g workgroups of ceil(N / g) images each and writes g partial sums.  Both
        // problems should fit the chip in one round (one workgroup per compute unit) and finish together, and
        // every extra group costs a partial sum to write and to add up.  Costs in thousands of cycles, from
        // traces of the kernel: an image of a 3x3 block 0.7 (rank 64) or 1.4, of a 1x1 block 1.0 (rank 64) or 2.0;
        // a megabyte of partial sums 1.0.  The search is tiny: every g1, and for it the fewest groups g2 that
        // do not make problem 2 the longer one.
        const int units1 = (g.C / wgrad_nchunk(g.r, g.k, 1)) * (g.k == 3 ? 2 : 1);
        const int units2 = g.Cout / wgrad_nchunk(g.r, 1, 2);
        const double c1 = g.k == 3 ? (g.r == 128 ? 1.4 : 0.7) : g.r == 128 ? 2.0 : 1.0, c2 = g.r == 128 ? 2.0 : 1.0;
        const double mb1 = 1.0e-6 * 4.0 * g.r * g.C * g.k * g.k, mb2 = 1.0e-6 * 4.0 * g.r * g.Cout;
        const int budget = 256;
        double best = 1e30;
        for (int g1 = 1; g1 <= g.N && (g1 == 1 || units1 * g1 + units2 <= budget); ++g1) {
            const int ipg1 = (g.N + g1 - 1) / g1;
            int g2max = (budget - units1 * g1) / units2;
            g2max = g2max < 1 ? 1 : g2max > g.N ? g.N : g2max;
            int ipg2 = (int)(ipg1 * c1 / c2); // images a workgroup of problem 2 may take
            ipg2 = ipg2 < 1 ? 1 : ipg2;
            int g2 = (g.N + ipg2 - 1) / ipg2;
            g2 = g2 > g2max ? g2max : g2;
            ipg2 = (g.N + g2 - 1) / g2;
            const double t1 = ipg1 * c1, t2 = ipg2 * c2;
            const double t = (t1 > t2 ? t1 : t2) + g1 * mb1 + g2 * mb2;
            if (t < best) {
                best = t;
                p.wg_ipg = ipg1;
                p.wg_ipg2 = ipg2;
            }
        }
        p.wg_groups = (g.N + p.wg_ipg - 1) / p.wg_ipg;
        p.wg_groups2 = (g.N + p.wg_ipg2 - 1) / p.wg_ipg2;
    }
    const i64 npix = (i64)g.N * g.Ho * g.Wo;
    p.ks_dVp = choose_ksplit(g.Cout, g.r, npix);
    p.ks_dUk = choose_ksplit(g.r, (i64)g.C * g.k * g.k, npix);
    p.n_T = (size_t)(npix * g.r);
    size_t a = (size_t)p.ks_dVp * g.Cout * g.r, b = (size_t)p.ks_dUk * g.r * g.C * g.k * g.k;
    p.n_part = a > b ? a : b;
    if (p.wgrad) { // both partial sets live side by side
        const size_t both = (size_t)p.wg_groups2 * g.Cout * g.r + (size_t)p.wg_groups * g.r * g.C * g.k * g.k;
        if (both > p.n_part) p.n_part = both;
    }
    p.fwd_bytes = align_up(p.n_T * sizeof(float));
    p.bwd_bytes = 2 * align_up(p.n_T * sizeof(float)) + align_up(p.n_part * sizeof(float));
    if (p.chain) { // the fused path needs packed weights instead of float copies of T (take the larger)
        const size_t f = align_up(p.n_w1 * 2) + align_up(p.n_w2 * 2);
        const size_t b = align_up(p.n_w1b * 2) + align_up(p.n_w2b * 2) + 2 * align_up(p.n_T * 2) +
                         align_up(p.n_part * sizeof(float));
        if (f > p.fwd_bytes) p.fwd_bytes = f;
        if (b > p.bwd_bytes) p.bwd_bytes = b;
    }
    if (p.tiles) {
        const size_t el = dtype == PF_BF16 ? 2 : 4;
        const size_t f = align_up(p.n_T * el) + align_up(p.n_part_T * 4);
        const size_t b = 2 * align_up(p.n_T * el) + 4 * align_up(p.n_pack * el) +
                         align_up((p.n_part_t > p.n_part_T ? p.n_part_t : p.n_part_T) * 4);
        if (f > p.fwd_bytes) p.fwd_bytes = f;
        if (b > p.bwd_bytes) p.bwd_bytes = b;
    }
    if (p.px_bwd) {
        const size_t el = dtype == PF_BF16 ? 2 : 4;
        const size_t b = align_up(p.px_dT * el) + align_up(p.px_pack * el) + align_up(p.px_part * 4);
        if (b > p.bwd_bytes) p.bwd_bytes = b;
    }
    return p;
}

static const ConvPlan &plan_conv(const ConvGeom &g, int dtype)
{
    static thread_local PlanCache<PlanKey<10>, ConvPlan> cache;
    return cache.get(PlanKey<10>{{g.N, g.C, g.H, g.W, g.Cout, g.r, g.k, g.s, g.p, dtype}}, [&] { return make_conv_plan(g, dtype); });
}

// ------------------------------------------------------------- any-shape
template <typename T>
static int conv_T_generic(const ConvGeom &g, const T *X, const T *Uk, float *Tws, T *T_save, hipStream_t s)
{
    const int npix = g.N * g.Ho * g.Wo, K = g.C * g.k * g.k;
    return launch_gemm_generic<T, true, false>("conv_T=Uk*X", s, GemmShape{g.r, npix, K, 1, 1},
                                               OpA_RowMajor<T>{Uk, K, 0}, OpB_Im2col<T>{X, g},
                                               EpiNCHW<float, T>{Tws, T_save, g.r, g.Ho * g.Wo});
}

template <typename T>
static int conv_fwd_generic(const ConvGeom &g, const T *X, const T *Uk, const T *Vp, T *Y, T *T_save, Workspace &ws,
                            hipStream_t s)
{
    const int npix = g.N * g.Ho * g.Wo;
    float *Tws = ws.take<float>((size_t)npix * g.r);
    int st = conv_T_generic<T>(g, X, Uk, Tws, T_save, s);
    if (st != PF_OK) return st;
    return launch_gemm_generic<T, true, false>("conv_Y=Vp*T", s, GemmShape{g.Cout, npix, g.r, 1, 1},
                                               OpA_RowMajor<T>{Vp, g.r, 0}, OpB_NCHW<float>{Tws, g.r, g.Ho * g.Wo},
                                               EpiNCHW<T, T>{Y, nullptr, g.Cout, g.Ho * g.Wo});
}

// Filter gradients from the saved / recomputed T and from dT (both [N][r][pixels], any element type).
template <typename T, typename TT, typename TD>
static int conv_wgrads(const ConvGeom &g, const ConvPlan &p, const T *X, const T *dY, const TT *Tt, const TD *dT,
                       float *dUk, float *dVp, int accumulate, float *part, hipStream_t s)
{
    const int npix = g.N * g.Ho * g.Wo, HW = g.Ho * g.Wo, kk = g.k * g.k;
    int st = PF_OK;
    if (dVp) { // dVp[o,q] = sum_pixel dY[o,pixel] T[q,pixel]
        st = launch_gemm_generic<T, true, true>("conv_dVp=dY*Tt", s, GemmShape{g.Cout, g.r, npix, 1, p.ks_dVp},
                                                OpA_NCHW<T>{dY, g.Cout, HW}, OpB_NCHW_T<TT>{Tt, g.r, HW},
                                                EpiPartial{part, g.r, (i64)g.Cout * g.r});
        if (st == PF_OK) st = launch_splitk_reduce(s, part, dVp, (i64)g.Cout * g.r, p.ks_dVp, accumulate);
        if (st != PF_OK) return st;
    }
    if (dUk) { // dUk[q,(c,i,j)] = sum_pixel dT[q,pixel] Xcol[(c,i,j),pixel]
        st = launch_gemm_generic<T, true, true>("conv_dUk=dT*Xcolt", s, GemmShape{g.r, g.C * kk, npix, 1, p.ks_dUk},
                                                OpA_NCHW<TD>{dT, g.r, HW}, OpB_Im2colT<T>{OpB_Im2col<T>{X, g}},
                                                EpiPartial{part, (i64)g.C * kk, (i64)g.r * g.C * kk});
        if (st == PF_OK) st = launch_splitk_reduce(s, part, dUk, (i64)g.r * g.C * kk, p.ks_dUk, accumulate);
    }
    return st;
}

template <typename T>
static int conv_bwd_generic(const ConvGeom &g, const ConvPlan &p, const T *X, const T *Uk, const T *Vp, const T *dY,
                            const T *T_saved, T *dX, float *dUk, float *dVp, int accumulate, Workspace &ws,
                            hipStream_t s)
{
    const int npix = g.N * g.Ho * g.Wo, HW = g.Ho * g.Wo, kk = g.k * g.k;
    float *Tws = ws.take<float>(p.n_T);
    float *dTws = ws.take<float>(p.n_T);
    float *part = ws.take<float>(p.n_part);
    int st = PF_OK;
    if (dVp && !T_saved) {
        st = conv_T_generic<T>(g, X, Uk, Tws, nullptr, s);
        if (st != PF_OK) return st;
    }
    if (dX || dUk) { // dT[q, pixel] = sum_o Vp[o,q] dY[o, pixel]
        st = launch_gemm_generic<T, false, false>("conv_dT=Vpt*dY", s, GemmShape{g.r, npix, g.Cout, 1, 1},
                                                  OpA_ColMajor<T>{Vp, g.r, 0}, OpB_NCHW<T>{dY, g.Cout, HW},
                                                  EpiNCHW<float, float>{dTws, nullptr, g.r, HW});
        if (st != PF_OK) return st;
    }
    if (dX) { // dX[c, in-pixel] = sum_{q,i,j} Uk[q,c,i,j] dT[q, out-pixel(in-pixel,i,j)]
        st = launch_gemm_generic<T, true, false>("conv_dX=Ukt*dT", s, GemmShape{g.C, g.N * g.H * g.W, g.r * kk, 1, 1},
                                                 OpA_FilterT<T>{Uk, g.C, kk}, OpB_Col2im<float>{dTws, g, g.r},
                                                 EpiNCHW<T, T>{dX, nullptr, g.C, g.H * g.W});
        if (st != PF_OK) return st;
    }
    if (T_saved) return conv_wgrads<T, T, float>(g, p, X, dY, T_saved, dTws, dUk, dVp, accumulate, part, s);
    return conv_wgrads<T, float, float>(g, p, X, dY, Tws, dTws, dUk, dVp, accumulate, part, s);
}

// ------------------------------------------------------------- any shape of at least a 16-byte piece
// T [n][pixel] etc. as the right operand of a product: every channel through one tap, or through all k x k.
static PixView pix_view(const ConvGeom &g, int dtype, const void *p, int CH, int H, int W, int gH, int gW)
{
    const int V = dtype == PF_BF16 ? 8 : 4;
    PixView v = {};
    v.p = p;
    v.total = (i64)g.N * CH * H * W;
    v.N = g.N, v.CH = CH, v.H = H, v.W = W, v.gH = gH, v.gW = gW;
    v.s = 1;
    v.HC = (gH * gW + V - 1) / V;
    v.ntap = 1;
    return v;
}
static PixView conv_input_view(const ConvGeom &g, int dtype, const void *X)
{
    PixView v = pix_view(g, dtype, X, g.C, g.H, g.W, g.Ho, g.Wo);
    v.s = g.s;
    v.ntap = g.k * g.k;
    for (int t = 0; t < v.ntap; ++t) {
        v.dy[t] = (signed char)(t / g.k - g.p);
        v.dx[t] = (signed char)(t % g.k - g.p);
    }
    return v;
}
static void out_planes(TileOut &o, const PixView &v, int CH)
{
    o.N = v.N, o.CH = CH, o.HC = v.HC, o.HW = v.gH * v.gW, o.gW = v.gW;
    o.s = 1;
}

// The rank-r intermediate from one product (and what else is in the launch), through partial sums when it is split.
template <typename T>
static int conv_mid_tiles(hipStream_t s, const char *name, const ConvGeom &g, TileShape shape, TileArgs &a, TileProb q, const PixView &v,
                          int ks, T *out, float *part)
{
    const int dt = sizeof(T) == 2 ? PF_BF16 : PF_F32, V = 16 / (int)sizeof(T);
    if (ks > 1) {
        q.o.C = part;
        q.o.f32 = 1;
        q.o.ld = q.N;
        q.o.split_stride = (i64)g.r * q.N;
    } else {
        q.o.C = out;
        out_planes(q.o, v, g.r);
    }
    tile_add(a, shape, dt, q, ks);
    const int got = a.p[a.n - 1].ksplit;
    int st = launch_tiles_conv(s, name, dt, shape, TS_64, a);
    if (st != PF_OK || ks <= 1) return st;
    SplitSumArgs ss = {};
    split_sum_add(ss, SplitSum{part, (float *)out, (i64)g.r * q.N, (i64)g.r * q.N, got, 0, nullptr, 0, sizeof(T) == 2, g.r, 0,
                               v.HC * V, v.gH * v.gW});
    return launch_split_sums(s, ss);
}

template <typename T>
static int conv_T_tiles(const ConvGeom &g, const ConvPlan &p, const T *X, const T *Uk, T *out, float *part, hipStream_t s)
{
    const int dt = sizeof(T) == 2 ? PF_BF16 : PF_F32, K = g.C * g.k * g.k;
    const PixView v = conv_input_view(g, dt, X);
    TileArgs a = {};
    TileProb q = tile_prob(p.gather ? TILE_CONVG : TILE_CONV, g.r, g.N * v.HC * (16 / (int)sizeof(T)), K, Uk, K, nullptr, 0,
                           nullptr, 0);
    q.pb = v;
    return conv_mid_tiles<T>(s, "conv_T=Uk*X", g, p.sh_T, a, q, v, p.ks_T, out, part);
}

// Two launches: T = Uk * X (an implicit product over (channel, tap), the order in which the filters lie in memory), then
// Y = act(scale (Vp T) + shift + residual) with the epilogue on the tile.
template <typename T>
static int conv_fwd_tiles(const ConvGeom &g, const ConvPlan &p, const T *X, const T *Uk, const T *Vp, T *Y, T *T_save,
                          Workspace &ws, hipStream_t s, const ConvEpilogue &ep)
{
    const int dt = sizeof(T) == 2 ? PF_BF16 : PF_F32;
    T *Tws = ws.take<T>(p.n_T), *Tt = T_save ? T_save : Tws;
    int st = conv_T_tiles<T>(g, p, X, Uk, Tt, ws.take<float>(p.n_part_T), s);
    if (st != PF_OK) return st;
    TileArgs a = {};
    const PixView v = pix_view(g, dt, Tt, g.r, g.Ho, g.Wo, g.Ho, g.Wo);
    TileProb q = tile_prob(TILE_CONV, g.Cout, g.N * v.HC * (16 / (int)sizeof(T)), g.r, Vp, g.r, nullptr, 0, Y, 0);
    q.pb = v;
    out_planes(q.o, v, g.Cout);
    q.o.scale = ep.scale;
    q.o.shift = ep.shift;
    q.o.add = ep.add;
    q.o.relu = ep.relu;
    tile_add(a, p.sh_Y, dt, q, 1);
    return launch_tiles_conv(s, "conv_Y=Vp*T", dt, p.sh_Y, TS_64, a);
}

// Three launches: dT = (scale Vp)^T dZ, with the filters re-ordered for the next launch in extra workgroups; then dX, dUk,
// dVp and the shift gradient side by side; then the sums over the image groups of the filter gradients.  With stride s,
// dX is s^2 products, one per phase of the input pixels, each over the taps that reach it.
template <typename T>
static int conv_bwd_tiles(const ConvGeom &g, const ConvPlan &p, const T *X, const T *Uk, const T *Vp, const T *dY,
                          const T *T_saved, T *dX, float *dUk, float *dVp, int accumulate, Workspace &ws, hipStream_t s,
                          const ConvEpilogue &ep)
{
    const int dt = sizeof(T) == 2 ? PF_BF16 : PF_F32, V = 16 / (int)sizeof(T), kk = g.k * g.k;
    T *Tws = ws.take<T>(p.n_T), *dT = ws.take<T>(p.n_T), *pack[4];
    for (int i = 0; i < 4; ++i) pack[i] = ws.take<T>(p.n_pack);
    float *part = ws.take<float>(p.n_part_t > p.n_part_T ? p.n_part_t : p.n_part_T);
    int st = PF_OK;
    if (dVp && !T_saved) {
        st = conv_T_tiles<T>(g, p, X, Uk, Tws, part, s);
        if (st != PF_OK) return st;
    }
    const PixView vdY = pix_view(g, dt, dY, g.Cout, g.Ho, g.Wo, g.Ho, g.Wo);
    const PixView vdT = pix_view(g, dt, dT, g.r, g.Ho, g.Wo, g.Ho, g.Wo);
    const PixView vT = pix_view(g, dt, T_saved ? T_saved : Tws, g.r, g.Ho, g.Wo, g.Ho, g.Wo);
    const int npx = g.N * vdT.HC * V, phases = g.s * g.s;
    TileArgs a = {}, b = {};
    if (dX) {
        // The two phases of a row in one workgroup.  Where half a piece lies in a row of the grid and both phases are all of it, every piece
        // leaves whole; elsewhere those do that hold no end of a row, as long as a row holds half a piece.  Half as many workgroups, each
        // twice as long: with enough of them.  Both directions, us, phase by phase / so: bf16 161 x 128 x 18 x 18, 444 tiles a phase 127 / 102, 45 x 64 x
        // 26 x 26, 124 tiles 62 / 48, 56 x 58 x 27 x 10, 63 tiles 66 / 61, 24 x 256 x 7 x 7, 24 tiles 44 / 49; rows of three cells, 225 x 384 x 5 x 5,
        // 127 / 132; float 75 x 256 x 30 x 6, 228 tiles 93 / 82, 192 x 64 x 19 x 19 155 / 152, 24 x 192 x 15 x 15, 72 tiles 72 / 78.
        const bool whole = g.H == 2 * g.Ho && g.W == 2 * g.Wo && g.Wo % (V / 2) == 0;
        // Filters of one tap (three phases are zero, and what is added): bf16 192 x 64 x 15 x 25 78 / 55, 53 x 304 x 28 x 28 179 / 148, float 23 x 199 x 28
        // x 28 90 / 68, 1 x 196 x 4 x 4, 4 tiles 38.7 / 40.3.
        const i64 each = (i64)((g.C + 63) / 64) * ((npx + 63) / 64);
        const bool many = g.Wo >= V / 2 && each >= (V == 8 ? 50 : 100);
        const bool rows = g.s == 2 && ((whole && (kk > 1 || V == 8 || each >= 20)) || many), packed = kk > 1 || rows;
        for (int f = 0; f < phases; ++f) {
            int ti[TILE_MAX_TAPS], oi[TILE_MAX_TAPS], tj[TILE_MAX_TAPS], oj[TILE_MAX_TAPS];
            const int ni = phase_taps(g, f / g.s, ti, oi), nj = phase_taps(g, f % g.s, tj, oj), nt = ni * nj;
            const T *W = Uk;
            PixView v = vdT;
            TileProb pk = tile_prob(TILE_PACK, g.C, g.r, 0, Uk, 0, nullptr, 0, pack[f], 0);
            for (int t = 0; t < nt; ++t) {
                v.dy[t] = (signed char)oi[t / nj];
                v.dx[t] = (signed char)oj[t % nj];
                pk.pb.dy[t] = (signed char)(ti[t / nj] * g.k + tj[t % nj]);
            }
            v.ntap = nt > 0 ? nt : 1;
            if (packed && nt > 0) {
                pk.pb.ntap = nt;
                pk.kper = kk;
                tile_add(a, p.sh_dT, dt, pk, 1);
                W = pack[f];
            }
            TileProb q = packed ? tile_prob(TILE_CONV, g.C, npx, g.r * nt, W, g.r * nt, nullptr, 0, dX, 0)
                                : tile_prob(TILE_CONVT, g.C, npx, nt > 0 ? g.r : 0, Uk, g.C, nullptr, 0, dX, 0);
            q.pb = v;
            out_planes(q.o, vdT, g.C);
            q.o.add = ep.add;
            q.o.mask = ep.mask;
            if (g.s > 1) {
                q.o.s = g.s;
                q.o.ph = f / g.s;
                q.o.pw = f % g.s;
                q.o.H = g.H;
                q.o.W = g.W;
            }
            tile_add(b, p.sh_g, dt, q, 1);
            if (rows && f % 2) tile_pair(b);
        }
    }
    if (dX || dUk) {
        TileProb q = tile_prob(TILE_CONVT, g.r, npx, g.Cout, Vp, g.r, nullptr, 0, nullptr, 0);
        q.pb = vdY;
        q.ascale = ep.scale;
        st = conv_mid_tiles<T>(s, "conv_dT=Vpt*dY", g, p.sh_dT, a, q, vdT, p.ks_dT, dT, part);
        if (st != PF_OK) return st;
    }
    SplitSumArgs ss = {};
    // [m][n] over the pixels (`transposed`: the result is wanted as [n][m]); sums: those of pa's rows, transposed: of pb's
    const auto grad = [&](const PixView &pa, const PixView &pb, int type, int m, int n, float *dst, int ks, float *sums,
                          const float *rscale, bool transposed) {
        TileProb q = tile_prob(type, m, n, 0, nullptr, 0, nullptr, 0, part, n);
        q.pa = pa;
        q.pb = pb;
        q.o.f32 = 1;
        q.o.split_stride = (i64)m * n;
        const int nsum = transposed ? n : m;
        float *ps = part + (i64)ks * m * n;
        ps += (64 - ((uintptr_t)ps / 4) % 64) % 64;
        part = ps;
        if (sums) {
            q.o.sums = ps;
            q.o.sums_stride = nsum;
            part += (i64)ks * nsum;
        }
        part += (64 - ((uintptr_t)part / 4) % 64) % 64;
        tile_add(b, p.sh_w, dt, q, ks);
        const int got = b.p[b.n - 1].ksplit;
        split_sum_add(ss, SplitSum{(const float *)q.o.C, dst, (i64)m * n, (i64)m * n, got, accumulate, rscale,
                                   transposed ? m : n, 0, m, transposed ? n : 0});
        if (sums) split_sum_add(ss, SplitSum{ps, sums, nsum, nsum, got, accumulate, nullptr, 0, 0});
    };
    if (dUk)
        grad(vdT, conv_input_view(g, dt, X), p.gather ? TILE_WGG : TILE_WG, g.r, g.C * kk, dUk, p.ks_tU, nullptr, nullptr, false);
    if ((dVp || ep.dshift) && p.sh_w == TS_32x128)
        grad(vT, vdY, TILE_WGT, g.r, g.Cout, dVp, p.ks_tV, ep.dshift, ep.scale, true);
    else if (dVp || ep.dshift)
        grad(vdY, vT, TILE_WG, g.Cout, g.r, dVp, p.ks_tV, ep.dshift, ep.scale, false);
    st = launch_tiles_conv(s, "conv_dX,dUk,dVp", dt, p.sh_g, p.sh_w, b);
    if (st != PF_OK) return st;
    return launch_split_sums(s, ss);
}

// ----------------------------------------------------- fused small-image path (bf16)
// What a forward call keeps for a backward call that is given the same scale: both factors the way the backward direction reads them
// (its first stage runs on scale * Vp).
static PackW1 chain_saved_w1(const ConvGeom &g, const void *Vp, void *W_save, const float *scale)
{
    PackW1 q = make_pack_w1(W_save ? (const uint16_t *)Vp : nullptr, (uint4 *)W_save, g.Cout, g.r, 1, 1, g.r, 0, g.H, g.W);
    q.cscale = scale;
    return q;
}
static PackW2 chain_saved_w2(const ConvGeom &g, const ConvPlan &p, const void *Uk, void *W_save)
{
    const int T = g.k * g.k;
    return make_pack_w2(W_save ? (const uint16_t *)Uk : nullptr, W_save ? (uint4 *)((char *)W_save + align_up(p.n_w1b * 2)) : nullptr, g.C,
                        g.r, g.k, T - 1, T, (i64)g.C * T, -1);
}

static int conv_fwd_chain(const ConvGeom &g, const ConvPlan &p, const bf16_t *X, const bf16_t *Uk, const bf16_t *Vp,
                          bf16_t *Y, bf16_t *T_save, void *W_save, Workspace &ws, hipStream_t s, const ConvEpilogue &ep)
{
    const int T = g.k * g.k;
    uint16_t *w1 = ws.take<uint16_t>(p.n_w1);
    uint16_t *w2 = ws.take<uint16_t>(p.n_w2);
    // Both factors are re-ordered into MFMA fragment order by one small launch (read in place, one lane per row,
    // the 1x1 filters Vp[Cout][r] reach the compute unit at a quarter of the rate).  The same launch can re-order
    // both factors the way the backward pass wants them (W_save), which saves that pass a launch of its own.
    int st = launch_pack_chain(s, make_pack_w1((const uint16_t *)Uk, (uint4 *)w1, g.C, g.r, g.k, (i64)g.C * T, T, 1, g.H, g.W),
                               chain_saved_w2(g, p, Uk, W_save), chain_saved_w1(g, Vp, W_save, ep.scale),
                               make_pack_w2((const uint16_t *)Vp, (uint4 *)w2, g.Cout, g.r, 1, 0, g.r, 1, 0));
    if (st != PF_OK) return st;
    ChainArgs a{(const uint16_t *)X, (const uint4 *)w1, (const uint4 *)w2, nullptr, (uint16_t *)Y,
                (uint16_t *)T_save,  g.C,               g.Cout,            g.H,     g.W,
                0,                   nullptr,           ep.scale,          ep.shift, (const uint16_t *)ep.add,
                (const uint16_t *)ep.mask, ep.relu};
    return launch_conv_chain(s, "conv_fwd_fused", a, g.N, g.k, 1, g.r);
}

static int conv_bwd_chain(const ConvGeom &g, const ConvPlan &p, const bf16_t *X, const bf16_t *Uk, const bf16_t *Vp,
                          const bf16_t *dY, const bf16_t *T_saved, const void *W_saved, bf16_t *dX, float *dUk,
                          float *dVp, int accumulate, Workspace &ws, hipStream_t s, const ConvEpilogue &ep)
{
    const int T = g.k * g.k;
    const uint16_t *w1 = ws.take<uint16_t>(p.n_w1b);
    const uint16_t *w2 = ws.take<uint16_t>(p.n_w2b);
    if (W_saved) { // the forward call packed them already
        w1 = (const uint16_t *)W_saved;
        w2 = (const uint16_t *)((const char *)W_saved + align_up(p.n_w1b * 2));
    }
    bf16_t *dT16 = ws.take<bf16_t>(p.n_T);
    bf16_t *T16 = ws.take<bf16_t>(p.n_T);
    float *part = ws.take<float>(p.n_part);
    int st = PF_OK;
    if (dVp && !T_saved) { // T was not saved: recompute it (thin convolution only)
        st = launch_gemm_generic<bf16_t, true, false>(
            "conv_T=Uk*X", s, GemmShape{g.r, g.N * g.Ho * g.Wo, g.C * T, 1, 1}, OpA_RowMajor<bf16_t>{Uk, (i64)g.C * T, 0},
            OpB_Im2col<bf16_t>{X, g}, EpiNCHW<bf16_t, bf16_t>{T16, nullptr, g.r, g.Ho * g.Wo});
        if (st != PF_OK) return st;
    }
    // stage 1: dT = Vp^T dY (1x1); stage 2: dX = flipped-Uk * dT (k x k)
    if (!W_saved) {
        PackW1 q = make_pack_w1((const uint16_t *)Vp, (uint4 *)w1, g.Cout, g.r, 1, 1, g.r, 0, g.H, g.W);
        q.cscale = ep.scale; // dT = Vp^T (scale dZ) = (scale Vp)^T dZ
        st = launch_pack_chain(s, q, make_pack_w2((const uint16_t *)Uk, (uint4 *)w2, g.C, g.r, g.k, T - 1, T, (i64)g.C * T, -1));
    }
    if (st != PF_OK) return st;
    ChainArgs a{(const uint16_t *)dY, (const uint4 *)w1, (const uint4 *)w2, nullptr, (uint16_t *)dX,
                (uint16_t *)dT16,     g.Cout,            g.C,               g.H,     g.W,
                0,                    nullptr,           nullptr,           nullptr, (const uint16_t *)ep.add,
                (const uint16_t *)ep.mask, 0};
    st = launch_conv_chain(s, "conv_bwd_data_fused", a, g.N, 1, g.k, g.r);
    if (st != PF_OK) return st;
    const bf16_t *Tt = T_saved ? T_saved : T16;
    if (!p.wgrad) return conv_wgrads<bf16_t, bf16_t, bf16_t>(g, p, X, dY, Tt, dT16, dUk, dVp, accumulate, part, s);
    float *part_dUk = part, *part_dVp = part + (size_t)p.wg_groups * g.r * g.C * T;
    WgradArgs wa1{(const uint16_t *)dT16, (const uint16_t *)X, dUk ? part_dUk : nullptr, g.r, g.C, g.H, g.W, g.N,
                  p.wg_ipg,               p.wg_groups, 0};
    WgradArgs wa2{(const uint16_t *)Tt, (const uint16_t *)dY, dVp ? part_dVp : nullptr, g.r, g.Cout, g.H, g.W, g.N,
                  p.wg_ipg2,            p.wg_groups2, 0};
    st = launch_conv_wgrad_pair(s, wa1, g.k, wa2);
    if (st != PF_OK) return st;
    WgradReduceArgs r0{part_dUk, dUk, p.wg_groups, T, g.r, g.C, (i64)g.C * T, T, 1, accumulate, nullptr};
    WgradReduceArgs r1{part_dVp, dVp, p.wg_groups2, 1, g.r, g.Cout, 1, g.r, 0, accumulate, ep.scale}; // dVp = scale (dZ T^T)
    const ColsumTilesArgs cs{nullptr, ep.dshift, 0, g.Cout, accumulate, dY, g.N, g.Ho * g.Wo};
    return launch_wgrad_reduce(s, r0, r1, ep.dshift ? &cs : nullptr);
}

// ----------------------------------------------------- pixel-major kernels
// Three launches: dT and dX, the partial sums of both filter gradients (and of the shift gradient), their sums.  Without the re-ordered
// filters of the forward call one more before them.
template <typename T>
static int conv_bwd_px(const ConvGeom &g, const ConvPlan &p, const T *X, const T *Uk, const T *Vp, const T *dY, const T *T_saved,
                       const T *W_saved, T *dX, float *dUk, float *dVp, int accumulate, Workspace &ws,
                       hipStream_t s, const ConvEpilogue &ep)
{
    T *dT = ws.take<T>(p.px_dT), *pack = ws.take<T>(p.px_pack);
    float *part = ws.take<float>(p.px_part);
    const PxPlaneOf<T> pl = px_plane<PxEl<T>::S>(g.N, g.H, g.W, g.k);
    int st = PF_OK;
    if (!W_saved) st = launch_px_pack(s, PxPack<T>{Uk, pack, g.C, g.r, g.k * g.k});
    if (st != PF_OK) return st;
    const PxBwdArgs<T> b{pl, g.C, g.Cout, g.r, dY, Vp, W_saved ? W_saved : pack, dX, dT, ep.scale, {nullptr, nullptr, (const T *)ep.add, (const T *)ep.mask, 0}};
    st = launch_px_bwd(s, b, g.k, p.px_bwd, p.px_bwd_threads);
    if (st != PF_OK) return st;
    const int kk = g.k * g.k, s1 = px_slab<T>(g.k, g.r), s2 = px_slab<T>(1, g.r);
    const i64 nU = (i64)g.r * g.C * kk, nV = (i64)g.r * g.Cout;
    float *partV = part + p.px_groups[0] * nU, *sums = partV + (p.px_groups[1] * nV + 63) / 64 * 64;
    const PxWgradArgs<T> w{px_plane<PxEl<T>::S>(g.N, g.H, g.W, 1), pl, g.r, 2,
                           {{dT, X, px_ranks<T>(g.r), g.C, kk, (g.C + s1 - 1) / s1, p.px_groups[0], p.px_per[0], part, nullptr},
                            {T_saved, dY, g.r, g.Cout, 1, (g.Cout + s2 - 1) / s2, p.px_groups[1], p.px_per[1], partV, ep.dshift ? sums : nullptr}}};
    st = launch_px_wgrad(s, w);
    if (st != PF_OK) return st;
    SplitSumArgs ss = {};
    split_sum_add(ss, SplitSum{part, dUk, nU, nU, p.px_groups[0], accumulate, nullptr, 0, 0});
    split_sum_add(ss, SplitSum{partV, dVp, nV, nV, p.px_groups[1], accumulate, ep.scale, g.r, 0, g.r, g.Cout});
    if (ep.dshift) split_sum_add(ss, SplitSum{sums, ep.dshift, g.Cout, g.Cout, p.px_groups[1], accumulate, nullptr, 0, 0});
    return launch_split_sums(s, ss);
}

// ------------------------------------------------------------------ dense
struct DenseConvPlan {
    int ks;
    size_t n_part, bytes;
};
static DenseConvPlan plan_dense_conv(const ConvGeom &g)
{
    DenseConvPlan p;
    const i64 npix = (i64)g.N * g.Ho * g.Wo;
    p.ks = choose_ksplit(g.Cout, (i64)g.C * g.k * g.k, npix);
    p.n_part = (size_t)p.ks * g.Cout * g.C * g.k * g.k;
    p.bytes = align_up(p.n_part * sizeof(float));
    return p;
}

template <typename T>
static int dense_conv_fwd_t(const ConvGeom &g, const T *X, const T *Wd, T *Y, hipStream_t s)
{
    const int npix = g.N * g.Ho * g.Wo, K = g.C * g.k * g.k;
    return launch_gemm_generic<T, true, false>("dense_conv_Y=W*X", s, GemmShape{g.Cout, npix, K, 1, 1},
                                               OpA_RowMajor<T>{Wd, K, 0}, OpB_Im2col<T>{X, g},
                                               EpiNCHW<T, T>{Y, nullptr, g.Cout, g.Ho * g.Wo});
}

template <typename T>
static int dense_conv_bwd_t(const ConvGeom &g, const T *X, const T *Wd, const T *dY, T *dX, float *dW, int accumulate,
                            Workspace &ws, hipStream_t s)
{
    const DenseConvPlan p = plan_dense_conv(g);
    const int npix = g.N * g.Ho * g.Wo, HW = g.Ho * g.Wo, kk = g.k * g.k;
    float *part = ws.take<float>(p.n_part);
    int st = PF_OK;
    if (g.N == 0) return accumulate ? st : launch_zero_f32(s, dW, (i64)g.Cout * g.C * kk);
    if (dX) {
        // the transposed convolution of the dense layer: the same gather with Cout in place of r
        st = launch_gemm_generic<T, true, false>("dense_conv_dX=Wt*dY", s,
                                                 GemmShape{g.C, g.N * g.H * g.W, g.Cout * kk, 1, 1},
                                                 OpA_FilterT<T>{Wd, g.C, kk}, OpB_Col2im<T>{dY, g, g.Cout},
                                                 EpiNCHW<T, T>{dX, nullptr, g.C, g.H * g.W});
        if (st != PF_OK) return st;
    }
    if (dW) {
        st = launch_gemm_generic<T, true, true>("dense_conv_dW=dY*Xcolt", s, GemmShape{g.Cout, g.C * kk, npix, 1, p.ks},
                                                OpA_NCHW<T>{dY, g.Cout, HW}, OpB_Im2colT<T>{OpB_Im2col<T>{X, g}},
                                                EpiPartial{part, (i64)g.C * kk, (i64)g.Cout * g.C * kk});
        if (st == PF_OK) st = launch_splitk_reduce(s, part, dW, (i64)g.Cout * g.C * kk, p.ks, accumulate);
    }
    return st;
}

} // namespace pf

using namespace pf;

extern "C" {

size_t pf_lowrank_conv_fwd_workspace_bytes(const pf_conv_desc *d)
{
    ConvGeom g;
    if (check_conv_desc(d, &g) != PF_OK) return 0;
    return plan_conv(g, d->dtype).fwd_bytes;
}

size_t pf_lowrank_conv_bwd_workspace_bytes(const pf_conv_desc *d)
{
    ConvGeom g;
    if (check_conv_desc(d, &g) != PF_OK) return 0;
    return plan_conv(g, d->dtype).bwd_bytes;
}

size_t pf_lowrank_conv_saved_weights_bytes(const pf_conv_desc *d)
{
    ConvGeom g;
    if (check_conv_desc(d, &g) != PF_OK) return 0;
    return plan_conv(g, d->dtype).saved_bytes; // (what the forward call writes, in either type)
}

int pf_lowrank_conv_fwd(const pf_conv_desc *d, const void *X, const void *Uk, const void *Vp, void *Y, void *T_save,
                        void *W_save, void *workspace, size_t workspace_bytes, void *stream)
{
    bool fused = false;
    return pf::conv_fwd_entry_ep(d, X, Uk, Vp, nullptr, nullptr, nullptr, PF_ACT_NONE, Y, T_save, W_save, workspace,
                                 workspace_bytes, stream, &fused);
}

int pf_lowrank_conv_bwd(const pf_conv_desc *d, const void *X, const void *Uk, const void *Vp, const void *dY,
                        const void *T_saved, const void *W_saved, void *dX, void *dUk, void *dVp, int accumulate,
                        void *workspace, size_t workspace_bytes, void *stream)
{
    bool fused = false;
    return pf::conv_bwd_entry_ep(d, X, Uk, Vp, nullptr, dY, T_saved, W_saved, nullptr, 0, dX, dUk, dVp, accumulate,
                                 workspace, workspace_bytes, stream, &fused);
}

size_t pf_dense_conv_workspace_bytes(const pf_conv_desc *d)
{
    ConvGeom g;
    if (check_conv_desc(d, &g) != PF_OK) return 0;
    return plan_dense_conv(g).bytes;
}

int pf_dense_conv_fwd(const pf_conv_desc *d, const void *X, const void *Wd, void *Y, void *workspace,
                      size_t workspace_bytes, void *stream)
{
    (void)workspace;
    (void)workspace_bytes;
    ConvGeom g;
    int st = check_conv_desc(d, &g);
    if (st != PF_OK) return st;
    if (!Wd) return PF_ERR_NULL;
    if (g.N == 0) return PF_OK;
    if (!X || !Y) return PF_ERR_NULL;
    hipStream_t s = (hipStream_t)stream;
    if (d->dtype == PF_F32) return dense_conv_fwd_t<float>(g, (const float *)X, (const float *)Wd, (float *)Y, s);
    return dense_conv_fwd_t<bf16_t>(g, (const bf16_t *)X, (const bf16_t *)Wd, (bf16_t *)Y, s);
}

int pf_dense_conv_bwd(const pf_conv_desc *d, const void *X, const void *Wd, const void *dY, void *dX, void *dWd,
                      int accumulate, void *workspace, size_t workspace_bytes, void *stream)
{
    ConvGeom g;
    int st = check_conv_desc(d, &g);
    if (st != PF_OK) return st;
    if (!Wd) return PF_ERR_NULL;
    if (g.N > 0 && (!X || !dY)) return PF_ERR_NULL;
    const size_t need = plan_dense_conv(g).bytes;
    if (!workspace || workspace_bytes < need) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    Workspace ws(workspace, workspace_bytes);
    hipStream_t s = (hipStream_t)stream;
    if (d->dtype == PF_F32)
        return dense_conv_bwd_t<float>(g, (const float *)X, (const float *)Wd, (const float *)dY, (float *)dX,
                                       (float *)dWd, accumulate, ws, s);
    return dense_conv_bwd_t<bf16_t>(g, (const bf16_t *)X, (const bf16_t *)Wd, (const bf16_t *)dY, (bf16_t *)dX,
                                    (float *)dWd, accumulate, ws, s);
}

} // extern "C"

// The pixel-major kernels form all gradients from a T that was kept.
static bool bwd_on_px(const pf::ConvPlan &p, const void *T_saved, const void *dX, const void *dUk, const void *dVp)
{
    return p.px_bwd && dX && dUk && dVp && T_saved;
}

// What the backward call with these arguments does by itself: fold a batch-norm scale into the filters and the sum of
// their gradients, and form the shift gradient (pixel-major kernels, chain kernels with their filter gradients, tiled products).
// Otherwise the caller scales beforehand and sums afterwards.
void pf::conv_bwd_takes(const pf_conv_desc *d, const void *T_saved, const void *dX, const void *dUk, const void *dVp, bool *scale, bool *dshift)
{
    *scale = *dshift = false;
    ConvGeom g;
    if (check_conv_desc(d, &g) != PF_OK || g.N == 0) return;
    const ConvPlan &p = plan_conv(g, d->dtype);
    const bool chain = d->dtype == PF_BF16 && p.chain && dX;
    *scale = *dshift = bwd_on_px(p, T_saved, dX, dUk, dVp) || (chain ? p.wgrad : p.tiles);
}

// ------------------------------------------------ entry points with an epilogue
// (the element-wise part is applied by the caller when *fused stays false)
int pf::conv_fwd_entry_ep(const pf_conv_desc *d, const void *X, const void *Uk, const void *Vp, const float *scale,
                          const float *shift, const void *residual, int act, void *Y, void *T_save, void *W_save,
                          void *workspace, size_t workspace_bytes, void *stream, bool *fused)
{
    ConvGeom g;
    int st = check_conv_desc(d, &g);
    if (st != PF_OK) return st;
    if (!Uk || !Vp) return PF_ERR_NULL;
    if (g.N > 0 && (!X || !Y)) return PF_ERR_NULL;
    if (any_misaligned({X, Uk, Vp, Y, T_save, W_save}, 16)) return PF_ERR_UNSUPPORTED;
    const ConvPlan p = plan_conv(g, d->dtype);
    if (p.fwd_bytes > 0 && (!workspace || workspace_bytes < p.fwd_bytes)) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    if (g.N == 0) return PF_OK;
    Workspace ws(workspace, workspace_bytes);
    hipStream_t s = (hipStream_t)stream;
    const ConvEpilogue all = {scale, shift, residual, nullptr, act == PF_ACT_RELU ? 1 : 0, nullptr};
    if (!p.saved_bytes) W_save = nullptr;
    const bool plain = !scale && !shift && !residual && !all.relu;
    const bool px_kept = p.px_bwd && W_save;
    if (p.px_fwd && !(plain && (px_kept ? p.plain_chain_kept : p.plain_chain))) {
        *fused = true;
        PackW1 w1 = {};
        PackW2 w2 = {};
        if (W_save && p.saved_bytes && !p.px_bwd) w1 = chain_saved_w1(g, Vp, W_save, scale), w2 = chain_saved_w2(g, p, Uk, W_save);
        const auto go = [&](auto el) {
            typedef decltype(el) T;
            const PxPack<T> pack = {(const T *)Uk, p.px_bwd ? (T *)W_save : nullptr, g.C, g.r, g.k * g.k};
            const PxFwdArgs<T> x{px_plane<PxEl<T>::S>(g.N, g.H, g.W, g.k), px_plane<PxEl<T>::S>(g.N, g.Ho, g.Wo, 1), g.s, g.C, g.Cout, g.r, (const T *)X, (const T *)Uk, (const T *)Vp, (T *)Y,
                                 (T *)T_save, {scale, shift, (const T *)residual, nullptr, all.relu}, pack, w1, w2};
            return launch_px_fwd(s, x, g.k, p.px_fwd, p.px_fwd_threads);
        };
        return d->dtype == PF_F32 ? go(float()) : go(uint16_t());
    }
    if (p.tiles && !(d->dtype == PF_BF16 && p.chain)) {
        *fused = true;
        if (d->dtype == PF_F32)
            return conv_fwd_tiles<float>(g, p, (const float *)X, (const float *)Uk, (const float *)Vp, (float *)Y,
                                         (float *)T_save, ws, s, all);
        return conv_fwd_tiles<bf16_t>(g, p, (const bf16_t *)X, (const bf16_t *)Uk, (const bf16_t *)Vp, (bf16_t *)Y,
                                      (bf16_t *)T_save, ws, s, all);
    }
    if (d->dtype == PF_F32)
        return conv_fwd_generic<float>(g, (const float *)X, (const float *)Uk, (const float *)Vp, (float *)Y,
                                       (float *)T_save, ws, s);
    if (p.chain)
    {
        // the kernel applies the epilogue as it stores (its float4 loads of scale and shift need 16-byte alignment)
        ConvEpilogue ep = {};
        if (!any_misaligned({scale, shift}, 16)) {
            ep = all;
            *fused = true;
        }
        st = conv_fwd_chain(g, p, (const bf16_t *)X, (const bf16_t *)Uk, (const bf16_t *)Vp, (bf16_t *)Y, (bf16_t *)T_save,
                            px_kept ? nullptr : W_save, ws, s, ep);
        if (px_kept && st == PF_OK) st = launch_px_pack(s, PxPack<uint16_t>{(const uint16_t *)Uk, (uint16_t *)W_save, g.C, g.r, g.k * g.k});
        return st;
    }
    return conv_fwd_generic<bf16_t>(g, (const bf16_t *)X, (const bf16_t *)Uk, (const bf16_t *)Vp, (bf16_t *)Y,
                                    (bf16_t *)T_save, ws, s);
}

int pf::conv_bwd_entry_ep(const pf_conv_desc *d, const void *X, const void *Uk, const void *Vp, const float *scale,
                          const void *dY, const void *T_saved, const void *W_saved, const void *dX_add, int x_is_relu,
                          void *dX, void *dUk, void *dVp, int accumulate, void *workspace, size_t workspace_bytes,
                          void *stream, bool *fused, float *dshift)
{
    ConvGeom g;
    int st = check_conv_desc(d, &g);
    if (st != PF_OK) return st;
    if (!Uk || !Vp) return PF_ERR_NULL;
    if (g.N > 0 && (!X || !dY)) return PF_ERR_NULL;
    if (any_misaligned({X, Uk, Vp, dY, T_saved, W_saved, dX}, 16) || any_misaligned({dUk, dVp}, 4)) return PF_ERR_UNSUPPORTED;
    const ConvPlan p = plan_conv(g, d->dtype);
    if (p.bwd_bytes > 0 && (!workspace || workspace_bytes < p.bwd_bytes)) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    Workspace ws(workspace, workspace_bytes);
    hipStream_t s = (hipStream_t)stream;
    if (g.N == 0) {
        if (!accumulate) {
            st = launch_zero_f32(s, (float *)dUk, (i64)g.r * g.C * g.k * g.k);
            if (st == PF_OK) st = launch_zero_f32(s, (float *)dVp, (i64)g.Cout * g.r);
        }
        return st;
    }
    if (!p.saved_bytes) W_saved = nullptr;
    if (bwd_on_px(p, T_saved, dX, dUk, dVp)) {
        *fused = true;
        const auto go = [&](auto el) {
            typedef decltype(el) T;
            return conv_bwd_px(g, p, (const T *)X, (const T *)Uk, (const T *)Vp, (const T *)dY, (const T *)T_saved, (const T *)W_saved, (T *)dX,
                               (float *)dUk, (float *)dVp, accumulate, ws, s,
                               ConvEpilogue{scale, nullptr, dX_add, x_is_relu ? X : nullptr, 0, dshift});
        };
        return d->dtype == PF_F32 ? go(float()) : go(uint16_t());
    }
    if (p.px_bwd) W_saved = nullptr; // (in the order of the kernels above)
    if (p.tiles && !(d->dtype == PF_BF16 && p.chain && dX)) {
        *fused = true;
        const ConvEpilogue ep = {scale, nullptr, dX_add, x_is_relu ? X : nullptr, 0, dshift};
        if (d->dtype == PF_F32)
            return conv_bwd_tiles<float>(g, p, (const float *)X, (const float *)Uk, (const float *)Vp, (const float *)dY,
                                         (const float *)T_saved, (float *)dX, (float *)dUk, (float *)dVp, accumulate, ws, s,
                                         ep);
        return conv_bwd_tiles<bf16_t>(g, p, (const bf16_t *)X, (const bf16_t *)Uk, (const bf16_t *)Vp, (const bf16_t *)dY,
                                      (const bf16_t *)T_saved, (bf16_t *)dX, (float *)dUk, (float *)dVp, accumulate, ws, s,
                                      ep);
    }
    if (d->dtype == PF_F32)
        return conv_bwd_generic<float>(g, p, (const float *)X, (const float *)Uk, (const float *)Vp, (const float *)dY,
                                       (const float *)T_saved, (float *)dX, (float *)dUk, (float *)dVp, accumulate, ws,
                                       s);
    if (p.chain && dX)
    {
        *fused = true; // the kernel adds the skip gradient and masks as it stores dX
        return conv_bwd_chain(g, p, (const bf16_t *)X, (const bf16_t *)Uk, (const bf16_t *)Vp, (const bf16_t *)dY,
                              (const bf16_t *)T_saved, W_saved, (bf16_t *)dX, (float *)dUk,
                              (float *)dVp, accumulate, ws, s, ConvEpilogue{scale, nullptr, dX_add, x_is_relu ? X : nullptr, 0, dshift});
    }
    return conv_bwd_generic<bf16_t>(g, p, (const bf16_t *)X, (const bf16_t *)Uk, (const bf16_t *)Vp,
                                    (const bf16_t *)dY, (const bf16_t *)T_saved, (bf16_t *)dX, (float *)dUk,
                                    (float *)dVp, accumulate, ws, s);
}
