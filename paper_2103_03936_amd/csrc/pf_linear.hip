// Factorized fully connected layer (paper Section 2.1): Y = (X V) U^T + bias and its
// gradients, plus the dense comparator.  Host-side validation, workspace planning and
// dispatch; any shape runs on the tiled products (pf_tile.h), dimensions below one of their
// pieces on the guarded element-wise GEMM.
#include "pf_conv_chain.h"
#include "pf_linear_chain.h"
#include "pf_linear_grad.h"
#include "pf_linear_two.h"
#include "pf_skinny.h"
#include "pf_linear_small.h"
#include "pf_tile_plans.h"

#include <math.h>
#include "pf_conv_wgrad.h"
#include <mutex>
#include "pf_gemm.h"
#include "pf_epilogue.h"

namespace pf {

// dst[s][col] = sum over the s-th row chunk of src[row * ld + col]
template <typename T>
__global__ __launch_bounds__(256) void colsum_partial_kernel(const T *src, float *partial, int rows, int cols, i64 ld,
                                                              int rows_per_chunk)
{
    __shared__ float red[4][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    const int q = threadIdx.x >> 6;
    const int rbeg = blockIdx.y * rows_per_chunk;
    const int rend = min(rows, rbeg + rows_per_chunk);
    float acc = 0.f;
    if (c < cols)
        for (int r = rbeg + q; r < rend; r += 4) acc += to_float(src[(i64)r * ld + c]);
    red[q][threadIdx.x & 63] = acc;
    __syncthreads();
    if (q == 0 && c < cols)
        partial[(i64)blockIdx.y * cols + c] = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] +
                                              red[3][threadIdx.x];
}

// bf16, cols a multiple of 8: a thread owns 8 neighbouring columns (one 16-byte load per row) and every 32nd
// row of the chunk; the 32 row-lanes of a column group are added through LDS in a fixed order.
__global__ __launch_bounds__(256) void colsum_partial_bf16x8_kernel(const uint16_t *src, float *partial, int rows, int cols,
                                                                     i64 ld, int rows_per_chunk)
{
    __shared__ float red[32][64 + 1];
    const int cg = threadIdx.x & 7, rl = threadIdx.x >> 3; // column group within the block's 64 columns, row lane
    const int c0 = blockIdx.x * 64 + 8 * cg;
    const int rbeg = blockIdx.y * rows_per_chunk, rend = min(rows, rbeg + rows_per_chunk);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (c0 < cols) {
#pragma unroll 4
        for (int r = rbeg + rl; r < rend; r += 32) {
            const uint4 v = *(const uint4 *)(src + (i64)r * ld + c0);
            const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[2 * e] += __uint_as_float(d[e] << 16);
                acc[2 * e + 1] += __uint_as_float(d[e] & 0xffff0000u);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[rl][8 * cg + e] = acc[e];
    __syncthreads();
    if (threadIdx.x < 64 && blockIdx.x * 64 + threadIdx.x < cols) {
        float sum = 0.f;
#pragma unroll
        for (int q = 0; q < 32; ++q) sum += red[q][threadIdx.x];
        partial[(i64)blockIdx.y * cols + blockIdx.x * 64 + threadIdx.x] = sum;
    }
}

int colsum_chunks(i64 rows)
{
    i64 c = (rows + 511) / 512;
    return (int)(c > 64 ? 64 : c < 1 ? 1 : c);
}

// out[cols] (+)= column sums of src[rows x cols]; partial holds colsum_chunks(rows) * cols floats.
template <typename T>
int launch_colsum(hipStream_t stream, const T *src, float *partial, float *out, i64 rows, i64 cols, i64 ld,
                  int accumulate)
{
    int status = PF_OK;
    const int chunks = colsum_chunks(rows);
    const int per = (int)((rows + chunks - 1) / chunks);
    dim3 grid((unsigned)((cols + 63) / 64), chunks);
    if (sizeof(T) == 2 && cols % 8 == 0 && ld % 8 == 0) {
        PF_LAUNCH(status, "colsum_partial", colsum_partial_bf16x8_kernel, grid, dim3(256), stream,
                  (const uint16_t *)src, partial, (int)rows, (int)cols, ld, per);
    } else {
        PF_LAUNCH(status, "colsum_partial", (colsum_partial_kernel<T>), grid, dim3(256), stream, src, partial,
                  (int)rows, (int)cols, ld, per);
    }
    if (status != PF_OK) return status;
    return launch_splitk_reduce(stream, partial, out, cols, chunks, accumulate);
}

template int launch_colsum<float>(hipStream_t, const float *, float *, float *, i64, i64, i64, int);
template int launch_colsum<bf16_t>(hipStream_t, const bf16_t *, float *, float *, i64, i64, i64, int);

// ------------------------------------------------------------ validation
static int check_linear_desc(const pf_linear_desc *d)
{
    if (!d) return PF_ERR_NULL;
    if (d->dtype != PF_F32 && d->dtype != PF_BF16) return PF_ERR_UNSUPPORTED;
    if (d->wgrad_dtype != PF_F32) return PF_ERR_UNSUPPORTED; // parameter gradients are float sums
    if (d->M < 0 || d->in <= 0 || d->out <= 0 || d->r <= 0) return PF_ERR_SHAPE;
    const i64 lim = 0x7fffffffLL;
    if (d->M > lim || d->in > lim || d->out > lim || d->r > lim) return PF_ERR_SHAPE;
    if (d->M * d->in > (lim << 4) || d->M * d->out > (lim << 4)) return PF_ERR_SHAPE;
    return PF_OK;
}

// What the 32-row chain kernel applies as its output leaves (all optional; *used reports that it did).
struct LinEpilogue {
    const void *add, *mask;
    int relu;
    bool *used;
};

int linear_fwd_entry(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *bias, void *Y,
                     void *T_save, void *workspace, size_t workspace_bytes, void *stream, int align,
                     const LinEpilogue *ep = nullptr);
int linear_bwd_entry(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *dY,
                     const void *T_saved, void *dX, void *dU, void *dV, void *dbias, int accumulate, void *workspace,
                     size_t workspace_bytes, void *stream, int align, const LinEpilogue *ep = nullptr);

// ---------------------------------------------------------- workspace plan
// The tiled products' part of a plan, for G layers of this shape that share their input (side by side in every launch).
LinearTiles make_linear_tiles(const pf_linear_desc *d, int G)
{
    LinearTiles p = {};
    const i64 piece = d->dtype == PF_BF16 ? 8 : 4;
    p.ok = d->M > 0 && d->in >= piece && d->out >= piece && d->r >= piece && (G == 1 || d->r % piece == 0);
    if (!p.ok) return p;
    const i64 M = d->M, in = d->in, out = d->out, r = d->r;
    p.Y = plan_tiles(d->dtype, M, G * out, r, 1);
    const TileNeed need[3] = {{M, in, G * r, false}, {G * out, r, M, true, true}, {in, G * r, M, true, true}};
    p.grads = plan_tile_group(d->dtype, need, 3);
    const i64 rows = (M + 31) / 32 * 32, ins = (in + 31) / 32, outs = (G * out + 31) / 32; // (floats of T that the tiles of Y, dX and dV read)
    const MidPlan T = plan_mid(d->dtype, M, G * r, in, 16, p.Y.shape, 4 * outs * rows * r, 128 * r);
    const MidPlan dT = plan_mid(d->dtype, M, G * r, out, 16, p.grads.shape, 8 * ins * rows * G * r, 128 * (M > G * r ? M : G * r));
    p.T = T.t, p.T_sliced = T.sliced;
    p.dT = dT.t, p.dT_sliced = dT.sliced;
    const int ks = p.T.ksplit > p.dT.ksplit ? p.T.ksplit : p.dT.ksplit;
    p.n_mid = (size_t)(G * M * r);
    p.n_part_T = ks > 1 ? (size_t)(ks * G * M * r) : 0;
    p.n_part_g = (size_t)(G * (p.grads.ksplit[1] * (out * r + out) + p.grads.ksplit[2] * in * r)) + 192;
    const size_t el = d->dtype == PF_BF16 ? 2 : 4;
    p.fwd_bytes = align_up(p.n_mid * el) + align_up(p.n_part_T * 4);
    p.bwd_bytes = 2 * align_up(p.n_mid * el) + align_up((p.n_part_T > p.n_part_g ? p.n_part_T : p.n_part_g) * 4);
    if (p.dT_sliced) { // (not where these partial sums would make a call outgrow the library's own scratch)
        const size_t bwd = p.bwd_bytes + align_up(p.n_part_T * 4);
        if (bwd > PF_STATIC_SCRATCH_BYTES) p.dT_sliced = false;
        else p.bwd_bytes = bwd;
    }
    return p;
}

struct LinearPlan {
    int ks_dU, ks_dV;
    size_t fwd_bytes, bwd_bytes;
    size_t n_T, n_dT, n_part;
    bool fused;         // bf16 and shapes the fused chain / factor-gradient kernels take
    bool chain_fwd, chain_bwd; // ... and sizes where they are the faster ones
    bool chain2;        // ... and the rank the 32-row chain kernel is built for: no weight re-ordering pass
    size_t n_colsum;    // per-tile column sums of dY (bias gradient), floats
    int wg_groups, wg_ipg; // row-tile groups of the factor-gradient kernel and tiles per group
    int wg_cols;           // columns per workgroup of that kernel
    int two_fwd, two_split; // rows per workgroup and shares of the outputs where both stages forward are one launch of pf_linear_two.h, 0: not
    bool plain_chain;       // ... but the chain kernel takes the calls without residual input and ReLU
    int two_bwd, two_bwd_split; // the same for dT and dX; the factor gradients are then those of pf_linear_grad.h
    LinGradPlan lg;
    size_t n_lg; // their partial sums, floats
    bool skinny_fwd, skinny_bwd; // fp32, few rows and large factors: the weight-streaming kernels of the LSTM cell
    size_t n_part_sk;      // their slice sums, floats
    LinearTiles t;         // the tiled products of pf_tile.h
    bool small_fwd, small_bwd; // fp32 with at most 128 rows and dimensions in whole tiles: two launches per direction
    size_t n_small;        // slices of the rank-r intermediate(s) between them, floats
};

// Chain kernel or tiled products?  A workgroup of the chain kernel takes 32 rows through the whole layer, one stage after the
// other, so 8192 rows are one round of the chip whose length is the layer's width, however few rows there are; the
// tiled products spread few rows over the chip but move the intermediates through memory.  Measured with calls on one stream
// (us, chain / tiled), rank 128:
//   forward:  512 -> 512    8 / 10 at 64 rows,   8 / 12 at 4000,  9 / 14 at 8192,  16 / 20 at 16384
//             512 -> 2048  13 / 10              15 / 17           18 / 27           32 / 43
//            1024 -> 1024  13 / 11              14 / 14           17 / 22           31 / 32
//            2048 -> 512   16 / 12              19 / 17           20 / 22           38 / 31
//            4096 -> 512   26 / 13              32 / 25           33 / 32           62 / 44
//   backward: 512 -> 512   16 /  9              26 / 23           28 / 30           42 / 38
//             512 -> 2048  32 / 12              44 / 34           53 / 46           91 / 73
//            1024 -> 512   18 / 10              28 / 27           33 / 37           51 / 56
//            2048 -> 512   22 / 10              34 / 39           42 / 55           69 / 94
//            2048 -> 2048  38 / 12              54 / 56           67 / 82          116 / 106
//   three 512 -> 512 layers that share their input: forward 8 / 10 at 64 rows, 26 / 27 at 8192, 50 / 45 at 16384; backward
//   53 / 16, 88 / 51, 135 / 87
// and rank 64 (whose factors are re-ordered first): 1024 -> 256 forward 12 / 10, 13 / 13, 14 / 13, 16 / 17, at 32768 rows 29 / 25;
// backward 23 / 9, 33 / 24, 35 / 27, 42 / 39, 62 / 74.
// Few rows: while 32 rows x 128 outputs are at most one workgroup per compute unit, the kernel that deals them so is the fastest (us,
// this / what the rules below chose; at twice as many workgroups it takes twice as long):
//   512 -> 512   6.0 / 6.9 at 32 rows, 6.8 / 7.5 at 2048 (256 workgroups), 12.3 / 7.9 at 4096
//   256 -> 1024  5.0 / 8.7,            5.5 / 9.3 at 1024,                   9.9 / 9.6 at 2048
//   512 -> 2048  6.1 / 9.3,            6.8 / 10.6 at 512,                   12.4 / 11.1 at 1024
//  1024 -> 512   8.1 / 10.6,           9.2 / 11.3 at 2048,                  17.2 / 11.7 at 4096
//  1024 -> 4096  8.3 / 10.1,           8.9 / 11.5 at 256,                   16.8 / 11.8 at 512
static bool rows_fwd_pays(i64 M, i64 in, i64 out, i64 r, int G = 1)
{
    return linear_rows_supported(in, out, r) && (M + 31) / 32 * (out / 128) * G <= 256;
}
static bool chain_fwd_pays(i64 M, i64 in, i64 out, i64 r)
{
    if (rows_fwd_pays(M, in, out, r)) return true; // (linear_fwd_fused takes that kernel)
    if (r != 128) return M >= 10000 && M <= 16384;
    if (M > 8192) return in <= 512;
    return in + out <= 1536 || (M >= 4096 && in <= 2048);
}
static bool chain_bwd_pays(i64 M, i64 in, i64 out, i64 r)
{
    if (r != 128) return in > out && M >= 24000;
    if (in > out) return in >= 768 && M >= 4096;
    return in == out && M >= 5000 && M <= 10000;
}
// (several layers that share their input; backward, their dX is one tiled product over all ranks)
static bool chain_shared_fwd_pays(i64 M, i64 in) { return M <= 8192 && (in <= 512 || (in <= 1024 && M <= 4096)); }

// Both stages in one launch (pf_linear_two.h): rows per workgroup, or 0 for the other kernels.  Their times: the tiled products' two
// launches, or three where T is split, and the corrected ones of the two-stage kernel (plan_linear_two) against them, the geometric mean of
// a plain call and one with residual and ReLU, fitted to 785 shapes (7 and 10 % rms: ranks above 64, four blocks wide, cost it more than the
// plan says, most of all where they are not whole pieces and are fitted in registers: 7 x 576 -> 67 -> 2824 10.6 / 12.9 us, 1313 x 1104
// -> 83 -> 2016 16.0 / 19.3); at rank 128 and widths in multiples of 256 those of the chain kernel, fitted to 130 shapes.  Over the 785
// shapes 1.42 times as fast where it is taken, three of a thousand calls more than 5 % slower; over 60 of the others 1.14 (8192 x 512 -> 128 -> 512
// three times 25.4 -> 19.0 us, 8192 x 2048 -> 512 with residual 24.6 -> 18.9, 512 -> 2048 18.6 by both); few rows and inputs up to 1024 wide stay
// with the row kernel (423 x 512 -> 512: 6.6 against 7.3).
// Ranks from 136 to 256: tiled products fitted by themselves to 330 shapes of 64 to 19000 rows (7 % rms).  Taken for 128 of them, 1.31 times as
// fast, none more than a tenth slower (8192 x 640 -> 160 -> 2560 37.4 / 20.8 us, tiled / two-stage; 13797 x 448 -> 176 -> 3584 68.7 / 36.9; with few rows the tiles spread better: 1000 x 768 -> 192 -> 3072 12.4 / 14.9).
static int two_fwd_rows(i64 M, i64 in, i64 out, i64 r, int G, int &split)
{
    if (!linear_two_supported(M, in, out, r) || rows_fwd_pays(M, in, out, r, G)) return 0;
    int rows = 0;
    const double t = plan_linear_two(M, in, out, r, G, rows, split), m = 1e-6 * M;
    const double chain = 8.07 + m * (0.625 * G * out + 0.205 * (in + G * out)) + 2.44e-3 * in;
    if (linear_chain2_supported(in, out, r)) return t < chain ? rows : 0;
    const double odd = r % 8 ? 1 : 0, wide = r > 64 ? 1 : 0, tiles = (double)G * ((M + 63) / 64) * ((r + 63) / 64);
    if (r > 128) {
        const double rt = (double)((r + 63) / 64);
        const double tiled = 8.76 + m * G * (out * (0.485 + 0.235 * rt) + 0.227 * in * rt + 0.502 * r) + (0.746e-3 + (tiles > 100 ? 0.986e-3 : 0)) * in +
                             (in >= 512 && tiles < 200 ? 0.23 : 0) + 4.43e-3 * r + 1.89e-4 * G * out;
        return t < 0.92 * tiled ? rows : 0;
    }
    const double tiled = 8.37 + m * (0.359 * in + G * out * (0.808 + 0.22 * ((r + 63) / 64)) + 0.172 * odd * (in + G * out)) + 0.69 * odd + 0.52 * wide +
                         (1.07e-3 + (tiles > 100 ? 0.49e-3 : 0)) * in + (in >= 512 && tiles < 200 ? 0.67 : 0);
    // chunks of the first stage, pieces of outputs, rounds of workgroups
    const double chunk = wide && rows == 128 ? 64 : 128, steps = ceil(in / chunk), per = ceil(ceil(out / 128.0) / split);
    const double rounds = ceil((double)((M + rows - 1) / rows) * split * G / 256);
    const double two = 0.94 * t + 0.885 * wide + rounds * (0.164 * odd * per + wide * (0.059 * steps + 0.058 * per) + wide * odd * (0.188 * steps + 0.387 * per));
    return two < 0.95 * tiled ? rows : 0;
}

// The times above are of calls with a residual input.  Without one and without a ReLU the chain kernel is the faster one for inputs up to 512
// wide while it has one workgroup per compute unit (us, chain / two-stage, inputs from memory: 8192 x 512 -> 512 9.3 / 10.8, 8192 x 512 ->
// 256 7.4 / 8.6, 6000 x 256 -> 256 6.6 / 7.7, but 4096 x 256 -> 1024 10.4 / 8.8, 9000 x 512 -> 512 15.3 / 11.9).  Its times over 22 shapes, 2 % rms;
// the two-stage kernel's are 0.7 above the plan's there.  Of other widths it is the slower one at
// every number of rows from 1100 to 8192 (256 or 512 -> 768 1.02 to 1.50 times as long, 1280 1.11 to 1.66, 1536 1.13 to 1.51).
// G layers that share their input are G times the rows to it: three of 512 -> 512 at 1400 rows 8.3 / 10.0, of 256 -> 256 6.8 / 7.6, but at 2730
// rows (258 workgroups) 14.7 / 11.9.
static bool plain_chain_pays(i64 M, i64 in, i64 out, i64 r, int G = 1)
{
    int rows, split;
    return (M + 31) / 32 * G <= 256 && in <= 512 && (out == 256 || out == 512 || out == 1024) &&
           5.04 + 4.15e-3 * out - 2.4e-4 * in + 2.37e-7 * G * M * (in + out) < plan_linear_two(M, in, out, r, G, rows, split) + 0.7;
}

// Backward, dT and dX in one launch of it and the factor gradients in another (pf_linear_grad.h): rows per workgroup, or 0 for the other
// kernels, by times fitted to 170 shapes (600 to 17000 rows, 128 to 4096 wide, ranks 8 to 128; 9 and 8 % rms); of rank 128 and widths in
// multiples of 256 they are all that counts.  Elsewhere a closer fit has to agree, to 700 shapes from 200 rows on and calls without and with
// a skip gradient and a mask (9 and 5 % rms).  Of these the rule takes 180, 1.29 times as fast (geometric mean; a few small ranks up to a
// tenth slower with both, 6851 x 512 -> 40 -> 176 19.6 / 22.0).  512 -> 128 -> 2048, us, before / now: 44.5 / 40.3 at 8192
// rows; 2048 -> 512 with mask 53.9 / 42.1, at 16384 rows 102 / 66; 1536 -> 96 -> 384 52.0 / 31.8.  Few rows stay with the tiled products,
// which form dX and the gradients side by side (1000 rows, 512 -> 512: 13.5 / 19.2).
// Ranks from 136 to 256, fitted by themselves to 330 shapes (8 and 7 % rms): taken for 84, 1.34 times as fast, none more than a tenth slower
// (8192 rows, 640 -> 160 -> 2560 79.7 / 52.3, 3072 -> 192 -> 768 88.1 / 56.4; 3001 x 640 -> 160 -> 2560 39.4 / 42.6 stays).
static int two_bwd_rows(i64 M, i64 in, i64 out, i64 r, int &split)
{
    if (!linear_two_supported(M, out, in, r) || !plan_linear_grad(M, in, out, r).splits) return 0;
    int rows = 0;
    const LinGradPlan lg = plan_linear_grad(M, in, out, r);
    const double m = 1e-6 * M, w = (double)(in + out), tiles = ceil(M / 64.0) * ceil(r / 64.0), t = plan_linear_two(M, out, in, r, 1, rows, split);
    if (r > 128) {
        const double before = 9.38 + m * (2.27 * in + 0.984 * out + 3.3 * r + 0.415 * w * ceil(r / 64.0)) + 1.24e-3 * out;
        const double now = 10.4 + 0.898 * t + (0.619 + 0.00297 * r) * lg.per + 1.246e-6 * lg.splits * w * r + m * 0.12 * in + 5.5e-4 * w;
        return now < 0.92 * before ? rows : 0;
    }
    const double coarse_before = 11.56 + m * (1.488 * in + 0.699 * out + 6.26 * r + 0.00717 * w * r) + 2.1e-4 * w;
    const double coarse_now = 12.74 + m * (0.367 * w + 7.75 * r + 0.00246 * w * r) + 8.9e-4 * w + 2.24e-5 * w * r;
    if (coarse_now >= 0.97 * coarse_before) return 0;
    if (linear_chain2_supported(in, out, r)) return rows;
    const double before = 5.34 + m * (1.44 * in + 0.197 * out + 3.92 * r + 0.00137 * w * r + 0.743 * w * ceil(r / 64.0)) + (tiles < 200 ? 4.67 : 0) +
                          1.025e-3 * (tiles > 512 ? tiles / 512 : 1) * out + 3.62e-4 * M;
    const double now = 11.29 + 0.391 * t + (0.22 + 0.00389 * r) * lg.per + 1.835e-6 * lg.splits * w * r + m * (0.699 * in + 0.388 * out) + (r > 64 ? 2.73 : 0) + 5.0e-4 * w;
    return now < 0.95 * before ? rows : 0;
}

// The streaming kernels read a factor at 8 rows at a time and take four or five launches a direction, the tiled products two (their readers
// add the slices of T and dT) and pad to 32 rows; odd ranks cost these unaligned pieces, and a dX of few tiles is long on the gradients' larger
// ones.  Both in microseconds, fitted to 1107 calls of 1 to 32 rows, layers of 0.4 to 11 million weights (2.7 % rms here, 4.7 and 4.1 % the tiles;
// the means of factors in the caches and out of them).  us, here / tiled, in the caches and out of them:
//   forward 1 row, 1472 -> 591 -> 1664 14.1 / 16.5 and 17.4 / 19.3, 9 rows, 2224 -> 970 -> 2816 19.0 / 22.3 and 21.9 / 23.5, 8 rows, 2816 -> 704 -> 3696
//   19.1 / 17.7 and 21.4 / 19.3, 1 row, 2048 -> 512 -> 2048 14.5 / 13.6 and 17.5 / 16.7;
//   backward 14 rows, 2848 -> 712 -> 4000 28.2 / 33.7 and 32.0 / 36.2, 1 row, 4000 -> 500 -> 4000 21.4 / 28.2 and 26.6 / 31.0, 6 rows, 2432 -> 608 -> 3136
//   22.8 / 21.6 and 25.9 / 23.9, 16 rows, 2048 -> 512 -> 2048 22.4 / 17.5 and 25.1 / 19.9.
// The rule is 0.2 % behind the faster one (geometric mean), none more than 12 %; none more than a tenth behind the streaming kernels.  Below
// 0.8 million weights the tiles: 448 -> 112 -> 768 29.3 / 22.5 for both directions.
void linear_skinny_pays(const pf_linear_desc *d, const LinearTiles &t, bool &fwd, bool &bwd)
{
    const double m = 1e-6 * d->r * (d->in + d->out), M = (double)d->M, odd = d->r % 4 ? 1 : 0; // m: millions of weights
    fwd = bwd = false;
    if (d->dtype != PF_F32 || d->M <= 0 || d->M > SK_MAX_ROWS || !t.ok || m < 0.8) return;
    fwd = 14.25 + 0.96 * m + M * (0.129 + 0.016 * m) < 2.87 + (t.T.cost + t.Y.cost) / 1796 + 0.97 * odd;
    const double tiles = 0.56 + t.grads.cost / (t.grads.shape == TS_64 ? 1871 : 3042) + t.dT.cost / 1018 + odd * (0.32 + 0.0025 * d->r);
    bwd = 15.46 + 2.2 * m + M * (0.187 + 0.0218 * m) < 0.98 * tiles;
}

static LinearPlan make_linear_plan(const pf_linear_desc *d)
{
    LinearPlan p;
    p.ks_dU = choose_ksplit(d->out, d->r, d->M);
    p.ks_dV = choose_ksplit(d->in, d->r, d->M);
    p.n_T = (size_t)(d->M * d->r);
    p.n_dT = p.n_T;
    size_t part_dU = (size_t)p.ks_dU * d->out * d->r, part_dV = (size_t)p.ks_dV * d->in * d->r;
    size_t part_db = (size_t)colsum_chunks(d->M) * d->out;
    p.n_part = part_dU > part_dV ? part_dU : part_dV;
    if (part_db > p.n_part) p.n_part = part_db;
    p.fwd_bytes = align_up(p.n_T * sizeof(float));
    p.bwd_bytes = align_up(p.n_T * sizeof(float)) + align_up(p.n_dT * sizeof(float)) + align_up(p.n_part * sizeof(float));
    p.fused = d->dtype == PF_BF16 && linear_chain_supported(d->in, d->out, d->r);
    p.chain_fwd = p.fused && chain_fwd_pays(d->M, d->in, d->out, d->r);
    p.chain_bwd = p.fused && d->M > 0 && chain_bwd_pays(d->M, d->in, d->out, d->r);
    p.two_fwd = d->dtype == PF_BF16 ? two_fwd_rows(d->M, d->in, d->out, d->r, 1, p.two_split) : 0;
    p.plain_chain = p.chain_fwd && plain_chain_pays(d->M, d->in, d->out, d->r);
    p.two_bwd = d->dtype == PF_BF16 ? two_bwd_rows(d->M, d->in, d->out, d->r, p.two_bwd_split) : 0;
    p.n_lg = 0;
    if (p.two_bwd) {
        p.lg = plan_linear_grad(d->M, d->in, d->out, d->r);
        p.n_lg = (size_t)p.lg.splits * (d->r * (d->in + d->out) + d->out) + 128;
    }
    p.t = make_linear_tiles(d, 1);
    if (p.t.fwd_bytes > p.fwd_bytes) p.fwd_bytes = p.t.fwd_bytes;
    if (p.t.bwd_bytes > p.bwd_bytes) p.bwd_bytes = p.t.bwd_bytes;
    linear_skinny_pays(d, p.t, p.skinny_fwd, p.skinny_bwd);
    p.n_part_sk = 0;
    if (p.skinny_fwd || p.skinny_bwd) {
        SkinnyArgs a;
        const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
        const size_t n1 = skinny_one(M, nullptr, in, nullptr, r, in, r, nullptr, a);   // T = X V
        const size_t n2 = skinny_one(M, nullptr, r, nullptr, r, r, out, nullptr, a);   // Y = T U^T
        const size_t n3 = skinny_one(M, nullptr, out, nullptr, r, out, r, nullptr, a); // dT = dY U
        const size_t n4 = skinny_one(M, nullptr, r, nullptr, r, r, in, nullptr, a);    // dX = dT V^T
        const size_t f = n1 > n2 ? n1 : n2, b = n3 > n4 ? n3 : n4;
        p.n_part_sk = f > b ? f : b;
        const size_t fwd = align_up(p.n_T * sizeof(float)) + align_up(p.n_part_sk * sizeof(float));
        const size_t bwd = 2 * align_up(p.n_T * sizeof(float)) + align_up(p.n_part_sk * sizeof(float));
        if (fwd > p.fwd_bytes) p.fwd_bytes = fwd;
        if (bwd > p.bwd_bytes) p.bwd_bytes = bwd;
    }
    const bool small = d->dtype == PF_F32 && linear_small_supported(d->M, d->in, d->out, d->r);
    // (wide layers are faster on the tiled products: 4096 -> 128 -> 4096 forward 17.3 / 15.5 us at 128 rows, 12.7 / 13.7 at one; forward and
    // backward together 39.9 / 33.1 at 64 rows, 256 -> 64 -> 4096 28.4 / 25.7 at 128; 2048 -> 128 -> 512 21.4 / 23.9 at 64)
    p.small_fwd = small && (d->M <= 64 || d->in + d->out <= 6144);
    p.small_bwd = small && d->in + d->out <= 4096;
    p.n_small = small ? (size_t)(LS_MAX_SLICES * d->M * d->r) : 0; // slices per intermediate
    if (small) {
        const size_t one = align_up(p.n_small * sizeof(float));
        if (one > p.fwd_bytes) p.fwd_bytes = one;
        if (2 * one > p.bwd_bytes) p.bwd_bytes = 2 * one;
    }
    p.chain2 = p.fused && linear_chain2_supported(d->in, d->out, d->r);
    p.n_colsum = p.chain2 ? (size_t)(2 * ((d->M + LC_ROWS - 1) / LC_ROWS)) * d->out : 0;
    p.wg_groups = p.wg_ipg = 1;
    p.wg_cols = 256;
    if (p.fused) {
        const i64 tiles = (d->M + 63) / 64;
        i64 chunks = d->in / 256 + d->out / 256;
        // workgroups over half the chip, each keeping two 64-row tiles in flight: every group costs a partial sum to
        // write and to add (measured on the Transformer shapes: 0.322 ms per block against 0.328 with 256 and 0.352
        // with 64 here)
        i64 want = 128 / chunks;
        want = want < 1 ? 1 : want > 32 ? 32 : want; // (the cap bounds the partial sums the groups write)
        if (want > tiles) want = tiles > 0 ? tiles : 1;
        p.wg_cols = 256;
        if (chunks * want < 200) { // too few workgroups for the chip: narrower column tiles
            p.wg_cols = 128;
            chunks *= 2;
        }
        p.wg_ipg = (int)((tiles + want - 1) / want);
        if (p.wg_ipg < 1) p.wg_ipg = 1;
        p.wg_groups = (int)((tiles + p.wg_ipg - 1) / p.wg_ipg);
        if (p.wg_groups < 1) p.wg_groups = 1;
        const size_t wmax = (size_t)(d->in > d->out ? d->in : d->out) * d->r;
        const size_t fwd = align_up(wmax * 2);
        const size_t grads = (size_t)p.wg_groups * d->r * (d->in + d->out);
        const size_t part = grads > p.n_part ? grads : p.n_part;
        const size_t bwd = align_up(wmax * 2) + 2 * align_up(p.n_T * 2) + align_up(part * sizeof(float)) +
                           align_up(p.n_colsum * sizeof(float));
        if (fwd > p.fwd_bytes) p.fwd_bytes = fwd;
        if (bwd > p.bwd_bytes) p.bwd_bytes = bwd;
    }
    if (p.two_bwd) { // (not where its partial sums alone would make a call outgrow the library's own scratch)
        const size_t part = p.n_lg > p.t.n_part_T ? p.n_lg : p.t.n_part_T, bwd = 2 * align_up(p.n_T * 2) + align_up(part * 4);
        if (bwd > p.bwd_bytes && bwd > PF_STATIC_SCRATCH_BYTES) p.two_bwd = 0;
        else if (bwd > p.bwd_bytes) p.bwd_bytes = bwd;
    }
    return p;
}

static const LinearPlan &plan_linear(const pf_linear_desc *d)
{
    static thread_local PlanCache<PlanKey<6>, LinearPlan> cache;
    return cache.get(PlanKey<6>{{d->M, d->in, d->out, d->r, d->dtype, d->has_bias}}, [&] { return make_linear_plan(d); });
}

// ------------------------------------------------------------- any-shape
template <typename T>
static int linear_fwd_generic(const pf_linear_desc *d, const T *X, const T *V, const T *U, const T *bias, T *Y,
                              T *T_save, Workspace &ws, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    float *Tws = ws.take<float>((size_t)M * r);
    int st = launch_gemm_generic<T, true, false>(
        "linear_T=X*V", s, GemmShape{M, r, in, 1, 1}, OpA_RowMajor<T>{X, in, 0}, OpB_KN<T>{V, r, 0, 0},
        EpiRowMajor<float, T>{Tws, T_save, r, nullptr, 0});
    if (st != PF_OK) return st;
    return launch_gemm_generic<T, true, true>(
        "linear_Y=T*Ut", s, GemmShape{M, out, r, 1, 1}, OpA_RowMajor<float>{Tws, r, 0}, OpB_NK<T>{U, r, 0},
        EpiRowMajor<T, T>{Y, nullptr, out, d->has_bias ? bias : nullptr, 0});
}

template <typename T>
static int linear_bwd_generic(const pf_linear_desc *d, const T *X, const T *V, const T *U, const T *dY,
                              const T *T_saved, T *dX, float *dU, float *dV, float *dbias, int accumulate,
                              Workspace &ws, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    const LinearPlan p = plan_linear(d);
    float *Tws = ws.take<float>(p.n_T);
    float *dTws = ws.take<float>(p.n_dT);
    float *part = ws.take<float>(p.n_part);
    int st = PF_OK;
    if (M == 0) {
        if (!accumulate) {
            st = launch_zero_f32(s, dU, (i64)out * r);
            if (st == PF_OK) st = launch_zero_f32(s, dV, (i64)in * r);
            if (st == PF_OK && d->has_bias) st = launch_zero_f32(s, dbias, out);
        }
        return st;
    }
    if (dU && !T_saved) {
        st = launch_gemm_generic<T, true, false>(
            "linear_T=X*V", s, GemmShape{M, r, in, 1, 1}, OpA_RowMajor<T>{X, in, 0}, OpB_KN<T>{V, r, 0, 0},
            EpiRowMajor<float, float>{Tws, nullptr, r, nullptr, 0});
        if (st != PF_OK) return st;
    }
    if (dX || dV) {
        st = launch_gemm_generic<T, true, false>(
            "linear_dT=dY*U", s, GemmShape{M, r, out, 1, 1}, OpA_RowMajor<T>{dY, out, 0}, OpB_KN<T>{U, r, 0, 0},
            EpiRowMajor<float, float>{dTws, nullptr, r, nullptr, 0});
        if (st != PF_OK) return st;
    }
    if (dX) {
        st = launch_gemm_generic<T, true, true>(
            "linear_dX=dT*Vt", s, GemmShape{M, in, r, 1, 1}, OpA_RowMajor<float>{dTws, r, 0}, OpB_NK<T>{V, r, 0},
            EpiRowMajor<T, T>{dX, nullptr, in, nullptr, 0});
        if (st != PF_OK) return st;
    }
    if (dU) {
        const GemmShape g{out, r, M, 1, p.ks_dU};
        const EpiPartial epi{part, r, (i64)out * r};
        if (T_saved)
            st = launch_gemm_generic<T, false, false>("linear_dU=dYt*T", s, g, OpA_ColMajor<T>{dY, out, 0},
                                                      OpB_KN<T>{T_saved, r, 0, 0}, epi);
        else
            st = launch_gemm_generic<T, false, false>("linear_dU=dYt*T", s, g, OpA_ColMajor<T>{dY, out, 0},
                                                      OpB_KN<float>{Tws, r, 0, 0}, epi);
        if (st == PF_OK) st = launch_splitk_reduce(s, part, dU, (i64)out * r, p.ks_dU, accumulate);
        if (st != PF_OK) return st;
    }
    if (dV) {
        st = launch_gemm_generic<T, false, false>("linear_dV=Xt*dT", s, GemmShape{in, r, M, 1, p.ks_dV},
                                                  OpA_ColMajor<T>{X, in, 0}, OpB_KN<float>{dTws, r, 0, 0},
                                                  EpiPartial{part, r, (i64)in * r});
        if (st == PF_OK) st = launch_splitk_reduce(s, part, dV, (i64)in * r, p.ks_dV, accumulate);
        if (st != PF_OK) return st;
    }
    if (d->has_bias && dbias) st = launch_colsum<T>(s, dY, part, dbias, M, out, out, accumulate);
    return st;
}

// ---------------------------------------------------- any shape of at least a 16-byte piece
// T = A B_g (A [M][K], B_g [K][r]) for G layers, in the call's element type: T_g at out + g * sout with leading dimension
// ldo; through partial sums when the products have too few tiles for the chip (slices: how many, and they stay where they are,
// [split][G][M][r] at part).  A steps by sa from layer to layer.
template <typename T>
static int tiles_mid(hipStream_t s, const char *name, const TilePlan &t, int G, int M, int r, int K, const T *A, i64 sa,
                     const T *B, T *out, i64 ldo, i64 sout, float *part, int *slices = nullptr)
{
    const int dt = sizeof(T) == 2 ? PF_BF16 : PF_F32;
    TileArgs a = {};
    TileProb p = tile_prob(TILE_NN, M, r, K, A, K, B, r, out, ldo);
    p.nb = G;
    p.sa = sa;
    p.sb = (i64)K * r;
    p.sc = sout;
    const bool split = t.ksplit > 1;
    if (split) {
        p.o.C = part;
        p.o.f32 = 1;
        p.o.split_stride = (i64)G * M * r;
    }
    tile_add(a, t.shape, dt, p, t.ksplit);
    int st = launch_tiles_linear(s, name, dt, t.shape, a);
    if (slices) *slices = a.p[0].ksplit;
    if (st != PF_OK || !split || (slices && *slices > 1)) return st;
    SplitSumArgs ss = {};
    const i64 n = (i64)G * M * r;
    split_sum_add(ss, SplitSum{part, (float *)out, n, n, a.p[0].ksplit, 0, nullptr, 0, sizeof(T) == 2});
    return launch_split_sums(s, ss);
}

// Two launches: T_g = X V_g, then Y_g = act(T_g U_g^T + bias_g + residual) with the epilogue on the tile.
template <typename T>
static int linear_fwd_tiles(const pf_linear_desc *d, const LinearTiles &p, int G, const T *X, const T *V, const T *U,
                            const T *bias, T *Y, T *T_save, Workspace &ws, hipStream_t s, const LinEpilogue &ep)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    T *Tws = ws.take<T>(p.n_mid);
    float *part = ws.take<float>(p.n_part_T);
    T *Tt = T_save ? T_save : Tws;
    int slices = 1;
    int st = tiles_mid<T>(s, "linear_T=X*V", p.T, G, M, r, in, X, 0, V, Tt, r, (i64)M * r, part, p.T_sliced ? &slices : nullptr);
    if (st != PF_OK) return st;
    TileArgs a = {};
    TileProb q = tile_prob(TILE_NT, M, out, r, Tt, r, U, r, Y, out);
    if (slices > 1) q.A = part, q.aslices = slices, q.sstride = (i64)G * M * r, q.acopy = T_save;
    q.nb = G;
    q.sa = (i64)M * r;
    q.sb = (i64)out * r;
    q.sc = (i64)M * out;
    q.sbias = out;
    q.o.bias = d->has_bias ? bias : nullptr;
    q.o.add = ep.add;
    q.o.relu = ep.relu;
    if (ep.used) *ep.used = true;
    tile_add(a, p.Y.shape, d->dtype, q, 1);
    return launch_tiles_linear(s, "linear_Y=T*Ut", d->dtype, p.Y.shape, a);
}

// Two or three launches: dT_g = dY_g U_g (T_g = X V_g again when it was not kept), then dX = sum_g dT_g V_g^T, dU_g, dV_g
// and the bias gradients side by side, then the sums over their splits where the rows were split.  The dT_g of several
// layers lie side by side in one [M][G r] matrix, so that dX is one product with a contraction of G r.
template <typename T>
static int linear_bwd_tiles(const pf_linear_desc *d, const LinearTiles &p, int G, const T *X, const T *V, const T *U,
                            const T *dY, const T *T_saved, T *dX, float *dU, float *dV, float *dbias, int accumulate,
                            Workspace &ws, hipStream_t s, const LinEpilogue &ep)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    T *Tws = ws.take<T>(p.n_mid), *dT = ws.take<T>(p.n_mid);
    float *mid = p.dT_sliced ? ws.take<float>(p.n_part_T) : nullptr; // (partial sums of dT that the gradients' launch reads)
    float *part = ws.take<float>(p.n_part_T > p.n_part_g ? p.n_part_T : p.n_part_g);
    int st = PF_OK, slices = 1;
    if (dU && !T_saved) {
        st = tiles_mid<T>(s, "linear_T=X*V", p.T, G, M, r, in, X, 0, V, Tws, r, (i64)M * r, part);
        if (st != PF_OK) return st;
    }
    // (split, the partial sums of the layers are [G][M][r] like their sum)
    const bool side = G > 1 && p.dT.ksplit == 1;
    const i64 ldd = side ? (i64)G * r : r, sd = side ? r : (i64)M * r;
    if (dX || dV) {
        st = tiles_mid<T>(s, "linear_dT=dY*U", p.dT, G, M, r, out, dY, (i64)M * out, U, dT, ldd, sd, mid ? mid : part, mid ? &slices : nullptr);
        if (st != PF_OK) return st;
    }
    const TileShape sh = p.grads.shape;
    const bool want_db = d->has_bias && dbias;
    TileArgs a = {};
    SplitSumArgs ss = {};
    if (dX) {
        TileProb q = tile_prob(TILE_NT, M, in, G * r, dT, side ? ldd : r, V, r, dX, in);
        if (slices > 1) q.A = mid, q.aslices = slices, q.sstride = (i64)G * M * r;
        if (G > 1) {
            q.bseg = r;
            q.bjump = (i64)in * r;
        }
        if (G > 1 && !side) {
            q.aseg = r;
            q.ajump = (i64)M * r;
        }
        q.o.add = ep.add;
        q.o.mask = ep.mask;
        if (ep.used) *ep.used = true;
        tile_add(a, sh, d->dtype, q, 1);
    }
    const auto grad = [&](const T *A, i64 sa, int m, const T *B, i64 ldb, i64 sb, float *dst, int ks, float *sums) {
        TileProb q = tile_prob(TILE_TN, m, r, M, A, m, B, ldb, dst, r);
        if (slices > 1 && B == dT) q.B = mid, q.bslices = slices, q.sstride = (i64)G * M * r;
        q.nb = G;
        q.sa = sa;
        q.sb = sb;
        q.sc = (i64)m * r;
        q.ssums = m;
        q.o.f32 = 1;
        q.o.accumulate = accumulate;
        q.o.sums = sums;
        float *psum = part;
        const i64 n = (i64)G * m * r, nsum = (i64)G * m;
        if (ks > 1) {
            q.o.accumulate = 0;
            q.o.C = part;
            q.o.split_stride = n;
            part += ks * n;
            part += (64 - ((uintptr_t)part / 4) % 64) % 64; // partial sums start 256-byte aligned
            if (sums) {
                psum = part;
                q.o.sums = psum;
                q.o.sums_stride = nsum;
                part += ks * nsum;
                part += (64 - ((uintptr_t)part / 4) % 64) % 64;
            }
        }
        tile_add(a, sh, d->dtype, q, ks);
        if (ks > 1) {
            const int got = a.p[a.n - 1].ksplit;
            split_sum_add(ss, SplitSum{(const float *)q.o.C, dst, n, n, got, accumulate, nullptr, 0, 0});
            if (sums) split_sum_add(ss, SplitSum{psum, sums, nsum, nsum, got, accumulate, nullptr, 0, 0});
        }
    };
    if (dU)
        grad(dY, (i64)M * out, out, T_saved ? T_saved : Tws, r, (i64)M * r, dU, p.grads.ksplit[1], want_db ? dbias : nullptr);
    if (dV) grad(X, 0, in, dT, ldd, sd, dV, p.grads.ksplit[2], nullptr);
    st = launch_tiles_linear(s, "linear_dX,dU,dV", d->dtype, sh, a);
    if (st == PF_OK) st = launch_split_sums(s, ss);
    for (int g = 0; st == PF_OK && want_db && !dU && g < G; ++g)
        st = launch_colsum<T>(s, dY + (i64)g * M * out, part, dbias + (i64)g * out, M, out, out, accumulate);
    return st;
}

// ------------------------------------------------------------- fused (bf16)
// Y = (X V) U^T + bias on the two-stage chain kernel: stage 1 weights = V^T re-ordered into MFMA fragments,
// stage 2 weights = U[out][r] read in place.
static int linear_fwd_fused(const pf_linear_desc *d, const bf16_t *X, const bf16_t *V, const bf16_t *U,
                            const bf16_t *bias, bf16_t *Y, bf16_t *T_save, Workspace &ws, hipStream_t s,
                            const LinEpilogue &ep = LinEpilogue{})
{
    const int in = (int)d->in, out = (int)d->out, r = (int)d->r;
    if (linear_chain2_supported(in, out, r)) {
        LinChainArgs c{(const uint16_t *)X, (const uint16_t *)V, (const uint16_t *)U,
                       d->has_bias ? (const uint16_t *)bias : nullptr, (uint16_t *)Y, (uint16_t *)T_save, nullptr,
                       d->M, in, out};
        c.ep_add = (const uint16_t *)ep.add;
        c.ep_relu = ep.relu;
        if (ep.used) *ep.used = true;
        return rows_fwd_pays(d->M, in, out, r) ? launch_linear_rows(s, "linear_fwd_rows", c) : launch_linear_chain2(s, "linear_fwd_fused", c);
    }
    uint16_t *w1 = ws.take<uint16_t>((size_t)(in > out ? in : out) * r);
    int st = launch_pack_chain(s, make_pack_w1((const uint16_t *)V, (uint4 *)w1, in, r, 1, 1, r, 0),
                               make_pack_w2(nullptr, nullptr, out, r, 1, 0, 0, 0, 0));
    if (st != PF_OK) return st;
    ChainArgs a{(const uint16_t *)X, (const uint4 *)w1, nullptr, (const uint16_t *)U, (uint16_t *)Y,
                (uint16_t *)T_save,  in,                out,     8,                   8,
                d->M,                d->has_bias ? bias : nullptr};
    return launch_linear_chain(s, "linear_fwd_fused", a, r);
}

// Both factor gradients in one launch, their group sums, and the bias gradient (from the column sums the chain
// kernel left, two rows per 32-row tile, or from dY).
static int linear_wgrads_fused(const pf_linear_desc *d, const LinearPlan &p, const bf16_t *X, const bf16_t *dY,
                               const bf16_t *Tt, const bf16_t *dT16, float *dU, float *dV, float *dbias,
                               const float *colsum, int accumulate, float *part, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    const bool want_db = d->has_bias && dbias;
    const int tiles = (M + 63) / 64;
    float *part_dU = part, *part_dV = part + (size_t)p.wg_groups * r * out;
    WgradArgs a1{(const uint16_t *)Tt, (const uint16_t *)dY, dU ? part_dU : nullptr, r, out, 8, 8, tiles, p.wg_ipg,
                 p.wg_groups,          d->M};
    WgradArgs a2{(const uint16_t *)dT16, (const uint16_t *)X, dV ? part_dV : nullptr, r, in, 8, 8, tiles, p.wg_ipg,
                 p.wg_groups,            d->M};
    int st = launch_linear_wgrad_pair(s, a1, a2, p.wg_cols);
    if (st != PF_OK) return st;
    WgradReduceArgs r0{part_dU, dU, p.wg_groups, 1, r, out, 1, r, 0, accumulate};
    WgradReduceArgs r1{part_dV, dV, p.wg_groups, 1, r, in, 1, r, 0, accumulate};
    const ColsumTilesArgs cs{colsum, dbias, 2 * ((M + LC_ROWS - 1) / LC_ROWS), out, accumulate};
    st = launch_wgrad_reduce(s, r0, r1, want_db && colsum ? &cs : nullptr);
    if (st != PF_OK) return st;
    if (want_db && !colsum) st = launch_colsum<bf16_t>(s, dY, part, dbias, M, out, out, accumulate);
    return st;
}

// dT = dY U, dX = dT V^T on the same kernel (stage 1 weights = U^T re-ordered, stage 2 weights = V[in][r] in
// place); then both factor gradients in one launch, their group sums, and the bias gradient.
static int linear_bwd_fused(const pf_linear_desc *d, const LinearPlan &p, const bf16_t *X, const bf16_t *V,
                            const bf16_t *U, const bf16_t *dY, const bf16_t *T_saved, bf16_t *dX, float *dU, float *dV,
                            float *dbias, int accumulate, Workspace &ws, hipStream_t s,
                            const LinEpilogue &ep = LinEpilogue{})
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    uint16_t *w1 = ws.take<uint16_t>((size_t)(in > out ? in : out) * r);
    bf16_t *dT16 = ws.take<bf16_t>(p.n_T);
    bf16_t *T16 = ws.take<bf16_t>(p.n_T);
    const size_t grads = (size_t)p.wg_groups * r * (in + out);
    float *part = ws.take<float>(grads > p.n_part ? grads : p.n_part);
    float *colsum = p.chain2 ? ws.take<float>(p.n_colsum) : nullptr;
    const bool want_db = d->has_bias && dbias;
    int st = PF_OK;
    if (dU && !T_saved) { // T was not saved: recompute it
        st = launch_gemm_generic<bf16_t, true, false>(
            "linear_T=X*V", s, GemmShape{M, r, in, 1, 1}, OpA_RowMajor<bf16_t>{X, in, 0}, OpB_KN<bf16_t>{V, r, 0, 0},
            EpiRowMajor<bf16_t, bf16_t>{T16, nullptr, r, nullptr, 0});
        if (st != PF_OK) return st;
    }
    if (p.chain2) {
        LinChainArgs c{(const uint16_t *)dY, (const uint16_t *)U, (const uint16_t *)V, nullptr, (uint16_t *)dX,
                       (uint16_t *)dT16, want_db ? colsum : nullptr, d->M, out, in};
        c.ep_add = (const uint16_t *)ep.add;
        c.ep_mask = (const uint16_t *)ep.mask;
        if (ep.used) *ep.used = true;
        st = launch_linear_chain2(s, "linear_bwd_data_fused", c);
    } else {
        st = launch_pack_chain(s, make_pack_w1((const uint16_t *)U, (uint4 *)w1, out, r, 1, 1, r, 0),
                               make_pack_w2(nullptr, nullptr, in, r, 1, 0, 0, 0, 0));
        if (st != PF_OK) return st;
        ChainArgs a{(const uint16_t *)dY, (const uint4 *)w1, nullptr, (const uint16_t *)V, (uint16_t *)dX,
                    (uint16_t *)dT16,     out,               in,      8,                   8,
                    d->M,                 nullptr};
        st = launch_linear_chain(s, "linear_bwd_data_fused", a, r);
    }
    if (st != PF_OK) return st;
    return linear_wgrads_fused(d, p, X, dY, T_saved ? T_saved : T16, dT16, dU, dV, dbias, colsum, accumulate, part, s);
}

// dT = dY U and dX = dT V^T in one launch, both factor gradients and the bias gradient in another, the sums over their splits.
static int linear_bwd_two(const pf_linear_desc *d, const LinearPlan &p, const bf16_t *X, const bf16_t *V, const bf16_t *U, const bf16_t *dY,
                          const bf16_t *T_saved, bf16_t *dX, float *dU, float *dV, float *dbias, int accumulate, Workspace &ws, hipStream_t s,
                          const LinEpilogue &ep)
{
    const int in = (int)d->in, out = (int)d->out, r = (int)d->r;
    bf16_t *Tws = ws.take<bf16_t>(p.n_T), *dT = ws.take<bf16_t>(p.n_T);
    float *part = ws.take<float>(p.n_lg > p.t.n_part_T ? p.n_lg : p.t.n_part_T);
    const bool want_db = d->has_bias && dbias;
    int st = PF_OK;
    if (dU && !T_saved) {
        st = tiles_mid<bf16_t>(s, "linear_T=X*V", p.t.T, 1, (int)d->M, r, in, X, 0, V, Tws, r, 0, part);
        if (st != PF_OK) return st;
    }
    LinTwoArgs two{d->M, out, in, r, (const uint16_t *)dY, (const uint16_t *)U, (const uint16_t *)V, nullptr, (const uint16_t *)ep.add,
                   (uint16_t *)dX, (uint16_t *)dT, 0, 1, 0, 0, 0, 0, 0, p.two_bwd_split, (const uint16_t *)ep.mask};
    if (ep.used) *ep.used = true;
    st = launch_linear_two(s, "linear_bwd_data_two", two, p.two_bwd);
    if (st != PF_OK) return st;
    LinGradArgs a{d->M, r, p.lg.splits, p.lg.per, 0, {}};
    SplitSumArgs ss = {};
    const auto take = [&](size_t n) { // partial sums start 256-byte aligned
        float *f = part;
        part += (n + 63) / 64 * 64;
        return f;
    };
    const auto grad = [&](const bf16_t *A, const bf16_t *B, int cols, float *dst, float *sums) {
        const i64 n = (i64)cols * r;
        LinGradProb &q = a.p[a.n++];
        q = LinGradProb{(const uint16_t *)A, (const uint16_t *)B, cols, take(p.lg.splits * n), sums ? take((size_t)p.lg.splits * cols) : nullptr};
        split_sum_add(ss, SplitSum{q.out, dst, n, n, p.lg.splits, accumulate, nullptr, 0, 0});
        if (sums) split_sum_add(ss, SplitSum{q.sums, sums, cols, cols, p.lg.splits, accumulate, nullptr, 0, 0});
    };
    // (for the bias gradient alone any matrix of rank r does)
    if (dU || want_db) grad(dY, !dU ? dT : T_saved ? T_saved : Tws, out, dU, want_db ? dbias : nullptr);
    if (dV) grad(X, dT, in, dV, nullptr);
    if (a.n) st = launch_linear_grad(s, a);
    return st == PF_OK ? launch_split_sums(s, ss) : st;
}

// --------------------------------------- fp32, few rows, dimensions in whole tiles
// Two launches per direction: the slices of the rank-r intermediate, then every product that reads their sum.
static int linear_fwd_small(const pf_linear_desc *d, const LinearPlan &p, const float *X, const float *V, const float *U,
                            const float *bias, float *Y, float *T_save, Workspace &ws, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    float *P = ws.take<float>(p.n_small);
    const int S = linear_small_slices(in);
    int st = launch_ls_slices(s, "linear_T_slices", LsSliceArgs{X, V, P, in, r, M, in, r, S});
    if (st != PF_OK) return st;
    LsTileArgs ta = {};
    ls_add(ta, ls_operand(P, r, LS_MK, S, (i64)M * r), ls_operand(U, r, LS_MK), M, out, r, Y, out,
           d->has_bias ? bias : nullptr, 0, T_save);
    return launch_ls_tiles(s, "linear_Y=T*Ut+b", ta);
}

static int linear_bwd_small(const pf_linear_desc *d, const LinearPlan &p, const float *X, const float *V, const float *U,
                            const float *dY, const float *T_saved, float *dX, float *dU, float *dV, float *dbias,
                            int accumulate, Workspace &ws, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    float *PdT = ws.take<float>(p.n_small), *PT = ws.take<float>(p.n_small);
    const int SdT = linear_small_slices(out), ST = linear_small_slices(in);
    const bool recompute = dU && !T_saved;
    // dT = dY U in slices and, when T was not kept, T = X V again, in one launch
    int st = launch_ls_slices(s, "linear_dT_slices", LsSliceArgs{dY, U, PdT, out, r, M, out, r, SdT},
                              recompute ? LsSliceArgs{X, V, PT, in, r, M, in, r, ST} : LsSliceArgs{});
    if (st != PF_OK) return st;
    const LsOperand dT_rows = ls_operand(PdT, r, LS_MK, SdT, (i64)M * r); // (row, rank index)
    const LsOperand dT_cols = ls_operand(PdT, r, LS_KM, SdT, (i64)M * r); // (rank index, row): contraction over rows
    const bool want_db = d->has_bias && dbias;
    LsTileArgs ta = {};
    if (dX) ls_add(ta, dT_rows, ls_operand(V, r, LS_MK), M, in, r, dX, in, nullptr, 0);
    if (dU)
        ls_add(ta, ls_operand(dY, out, LS_KM), recompute ? ls_operand(PT, r, LS_KM, ST, (i64)M * r) : ls_operand(T_saved, r, LS_KM),
               out, r, M, dU, r, nullptr, accumulate, nullptr, want_db ? dbias : nullptr);
    else if (want_db) // only the bias gradient of this product is wanted: the column sums of its left operand
        ls_add(ta, ls_operand(dY, out, LS_KM), ls_operand(dY, out, LS_KM), out, 32, M, nullptr, 0, nullptr, accumulate, nullptr,
               dbias);
    if (dV) ls_add(ta, ls_operand(X, in, LS_KM), dT_cols, in, r, M, dV, r, nullptr, accumulate);
    return launch_ls_tiles(s, "linear_dX,dU,dV,db", ta);
}

// ------------------------------------------------------------- fp32, few rows
static int linear_T_skinny(const pf_linear_desc *d, const float *X, const float *V, float *T, float *part, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, r = (int)d->r;
    SkinnyArgs a;
    skinny_one(M, X, in, V, r, in, r, part, a);
    int st = launch_skinny_gemm(s, "linear_T=X*V", a, false);
    if (st != PF_OK) return st;
    SliceSumArgs ss = {};
    ss.s[ss.nseg++] = slice_seg(a.p[0], T, r, r);
    return launch_slice_sum(s, ss);
}

static int linear_fwd_skinny(const pf_linear_desc *d, const LinearPlan &p, const float *X, const float *V, const float *U,
                             const float *bias, float *Y, float *T_save, Workspace &ws, hipStream_t s)
{
    const int M = (int)d->M, out = (int)d->out, r = (int)d->r;
    float *Tws = ws.take<float>(p.n_T);
    float *part = ws.take<float>(p.n_part_sk);
    float *T = T_save ? T_save : Tws;
    int st = linear_T_skinny(d, X, V, T, part, s);
    if (st != PF_OK) return st;
    SkinnyArgs a;
    skinny_one(M, T, r, U, r, r, out, part, a);
    st = launch_skinny_gemm(s, "linear_Y=T*Ut", a, true);
    if (st != PF_OK) return st;
    SliceSumArgs ss = {};
    ss.s[ss.nseg++] = slice_seg(a.p[0], Y, out, out, d->has_bias ? bias : nullptr);
    return launch_slice_sum(s, ss);
}

static int linear_bwd_skinny(const pf_linear_desc *d, const LinearPlan &p, const float *X, const float *V, const float *U,
                             const float *dY, const float *T_saved, float *dX, float *dU, float *dV, float *dbias,
                             int accumulate, Workspace &ws, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out, r = (int)d->r;
    float *Tws = ws.take<float>(p.n_T);
    float *dT = ws.take<float>(p.n_T);
    float *part = ws.take<float>(p.n_part_sk);
    int st = PF_OK;
    if (dU && !T_saved) { // T was not saved: recompute it
        st = linear_T_skinny(d, X, V, Tws, part, s);
        if (st != PF_OK) return st;
    }
    const float *T = T_saved ? T_saved : Tws;
    SkinnyArgs a;
    skinny_one(M, dY, out, U, r, out, r, part, a);
    st = launch_skinny_gemm(s, "linear_dT=dY*U", a, false);
    if (st != PF_OK) return st;
    SliceSumArgs ss = {};
    ss.s[ss.nseg++] = slice_seg(a.p[0], dT, r, r);
    st = launch_slice_sum(s, ss);
    if (st != PF_OK) return st;
    ss = SliceSumArgs{};
    if (dX) {
        skinny_one(M, dT, r, V, r, r, in, part, a);
        st = launch_skinny_gemm(s, "linear_dX=dT*Vt", a, true);
        if (st != PF_OK) return st;
        ss.s[ss.nseg++] = slice_seg(a.p[0], dX, in, in);
    }
    // factor gradients are rank-M updates; the slice sums of dX ride along
    RankArgs ra = {};
    ra.M = M;
    ra.accumulate = accumulate;
    rank_add(ra, dY, out, T, r, dU, r, out, r);
    rank_add(ra, X, in, dT, r, dV, r, in, r);
    if (d->has_bias && dbias) rank_add(ra, dY, out, nullptr, 0, dbias, 1, out, 1);
    return launch_rank_update(s, "linear_grads", ra, ss);
}

// ------------------------------------------------------------------ dense
struct DensePlan {
    int ks;
    size_t n_part, bytes;
};
static DensePlan plan_dense_linear(const pf_linear_desc *d)
{
    DensePlan p;
    p.ks = choose_ksplit(d->out, d->in, d->M);
    size_t a = (size_t)p.ks * d->out * d->in, b = (size_t)colsum_chunks(d->M) * d->out;
    p.n_part = a > b ? a : b;
    p.bytes = align_up(p.n_part * sizeof(float));
    return p;
}

template <typename T>
static int dense_linear_fwd_t(const pf_linear_desc *d, const T *X, const T *W, const T *bias, T *Y, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out;
    return launch_gemm_generic<T, true, true>("dense_linear_Y=X*Wt", s, GemmShape{M, out, in, 1, 1},
                                              OpA_RowMajor<T>{X, in, 0}, OpB_NK<T>{W, in, 0},
                                              EpiRowMajor<T, T>{Y, nullptr, out, d->has_bias ? bias : nullptr, 0});
}

template <typename T>
static int dense_linear_bwd_t(const pf_linear_desc *d, const T *X, const T *W, const T *dY, T *dX, float *dW,
                              float *dbias, int accumulate, Workspace &ws, hipStream_t s)
{
    const int M = (int)d->M, in = (int)d->in, out = (int)d->out;
    const DensePlan p = plan_dense_linear(d);
    float *part = ws.take<float>(p.n_part);
    int st = PF_OK;
    if (M == 0) {
        if (!accumulate) {
            st = launch_zero_f32(s, dW, (i64)out * in);
            if (st == PF_OK && d->has_bias) st = launch_zero_f32(s, dbias, out);
        }
        return st;
    }
    if (dX) {
        st = launch_gemm_generic<T, true, false>("dense_linear_dX=dY*W", s, GemmShape{M, in, out, 1, 1},
                                                 OpA_RowMajor<T>{dY, out, 0}, OpB_KN<T>{W, in, 0, 0},
                                                 EpiRowMajor<T, T>{dX, nullptr, in, nullptr, 0});
        if (st != PF_OK) return st;
    }
    if (dW) {
        st = launch_gemm_generic<T, false, false>("dense_linear_dW=dYt*X", s, GemmShape{out, in, M, 1, p.ks},
                                                  OpA_ColMajor<T>{dY, out, 0}, OpB_KN<T>{X, in, 0, 0},
                                                  EpiPartial{part, in, (i64)out * in});
        if (st == PF_OK) st = launch_splitk_reduce(s, part, dW, (i64)out * in, p.ks, accumulate);
        if (st != PF_OK) return st;
    }
    if (d->has_bias && dbias) st = launch_colsum<T>(s, dY, part, dbias, M, out, out, accumulate);
    return st;
}

// ------------------------------------------------- projections that share their input
template <typename T>
__global__ void add_into_kernel(T *dst, const T *src, i64 count)
{
    const i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dst[i] = from_float<T>(to_float(dst[i]) + to_float(src[i]));
}

template <typename T>
static int launch_add_into(hipStream_t s, T *dst, const T *src, i64 count)
{
    int st = PF_OK;
    if (count <= 0) return st;
    PF_LAUNCH(st, "add_into", add_into_kernel<T>, dim3((unsigned)((count + 255) / 256)), dim3(256), s, dst, src, count);
    return st;
}

struct SharedPlan {
    pf_linear_desc one; // one of the G layers
    LinearPlan p;
    bool fused_fwd; // the groups run inside one launch of the chain kernel
    int two_fwd, two_split; // ... or of the two-stage kernel (rows per workgroup, shares of the outputs), 0: not
    LinearTiles t;  // otherwise, and backward, side by side on the tiled products
    size_t fwd_bytes, bwd_bytes;
};

static int check_shared_desc(const pf_linear_shared_desc *d, pf_linear_desc *one)
{
    if (!d) return PF_ERR_NULL;
    *one = pf_linear_desc{d->M, d->n_in, d->n_out, d->r, d->dtype, PF_F32, d->has_bias};
    int st = check_linear_desc(one);
    if (st != PF_OK) return st;
    if (d->groups <= 0 || d->groups > 64) return PF_ERR_SHAPE;
    const i64 lim = 0x7fffffffLL;
    if (d->groups * d->M * d->n_out > (lim << 4)) return PF_ERR_SHAPE;
    return PF_OK;
}

static SharedPlan make_shared_plan(const pf_linear_shared_desc *d, const pf_linear_desc &one)
{
    SharedPlan sp;
    sp.one = one;
    sp.p = plan_linear(&one);
    const int G = d->groups;
    sp.fused_fwd = d->dtype == PF_BF16 && sp.p.chain2 && d->M > 0 && G > 1 && G <= LC_MAX_GROUPS &&
                   (chain_shared_fwd_pays(d->M, d->n_in) || rows_fwd_pays(d->M, d->n_in, d->n_out, d->r, G));
    sp.two_fwd = d->dtype == PF_BF16 ? two_fwd_rows(d->M, d->n_in, d->n_out, d->r, G, sp.two_split) : 0;
    if (sp.two_fwd && sp.fused_fwd && plain_chain_pays(d->M, d->n_in, d->n_out, d->r, G)) sp.two_fwd = 0;
    if (sp.two_fwd) sp.fused_fwd = false;
    const size_t el = d->dtype == PF_BF16 ? 2 : 4;
    sp.fwd_bytes = sp.p.fwd_bytes;
    // one layer's workspace, then one more dX (layer by layer)
    sp.bwd_bytes = sp.p.bwd_bytes + align_up((size_t)(d->M * d->n_in) * el);
    sp.t = make_linear_tiles(&one, G);
    if (sp.t.fwd_bytes > sp.fwd_bytes) sp.fwd_bytes = sp.t.fwd_bytes;
    if (sp.t.bwd_bytes > sp.bwd_bytes) sp.bwd_bytes = sp.t.bwd_bytes;
    return sp;
}

static const SharedPlan &plan_shared(const pf_linear_shared_desc *d, const pf_linear_desc &one)
{
    static thread_local PlanCache<PlanKey<7>, SharedPlan> cache;
    return cache.get(PlanKey<7>{{d->M, d->n_in, d->n_out, d->r, d->groups, d->dtype, d->has_bias}},
                     [&] { return make_shared_plan(d, one); });
}

// Alignment a layer's slice of the stacked operands is held to: 16 bytes where the 16-byte-load kernels may run
// (their shapes make every slice a multiple of 16 bytes anyway), else that of an element or of the 4-byte loads
// of the few-row fp32 kernels.
static int layer_align(const SharedPlan &sp, size_t el) { return sp.p.fused ? 16 : (int)(el < 4 ? el : 4); }

template <typename T>
static int shared_bwd_loop(const pf_linear_shared_desc *d, const SharedPlan &sp, const T *X, const T *V, const T *U,
                           const T *dY, const T *T_saved, T *dX, float *dU, float *dV, float *dbias, int accumulate,
                           void *workspace, size_t workspace_bytes, hipStream_t s)
{
    // layer by layer; the input gradients of the layers after the first go to a spare buffer and are added
    const i64 M = d->M, in = d->n_in, out = d->n_out, r = d->r;
    T *spare = (T *)((char *)workspace + sp.p.bwd_bytes);
    int st = PF_OK;
    for (int g = 0; g < d->groups && st == PF_OK; ++g) {
        T *dXg = !dX ? nullptr : g == 0 ? dX : spare;
        st = linear_bwd_entry(&sp.one, X, V + g * in * r, U + g * out * r, dY + g * M * out,
                              T_saved ? T_saved + g * M * r : nullptr, dXg, dU ? dU + g * out * r : nullptr,
                              dV ? dV + g * in * r : nullptr, dbias ? dbias + g * out : nullptr, accumulate, workspace,
                              workspace_bytes, s, layer_align(sp, sizeof(T)));
        if (st == PF_OK && dX && g > 0) st = launch_add_into<T>(s, dX, spare, M * in);
    }
    return st;
}

} // namespace pf

using namespace pf;

// `align`: what the data pointers must be multiples of (16 for callers; the layers of a shared-input call may
// start anywhere an element does when their shape is one the element-wise kernels take)
int pf::linear_fwd_entry(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *bias,
                         void *Y, void *T_save, void *workspace, size_t workspace_bytes, void *stream, int align,
                         const LinEpilogue *ep)
{
    int st = check_linear_desc(d);
    if (st != PF_OK) return st;
    if (!V || !U || (d->has_bias && !bias)) return PF_ERR_NULL;
    if (d->M > 0 && (!X || !Y)) return PF_ERR_NULL;
    if (any_misaligned({X, V, U, bias, Y, T_save}, align)) return PF_ERR_UNSUPPORTED;
    const LinearPlan &p = plan_linear(d);
    const size_t need = p.fwd_bytes;
    if (need > 0 && (!workspace || workspace_bytes < need)) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    if (d->M == 0) return PF_OK;
    Workspace ws(workspace, workspace_bytes);
    hipStream_t s = (hipStream_t)stream;
    if (d->dtype == PF_F32 && p.small_fwd)
        return linear_fwd_small(d, p, (const float *)X, (const float *)V, (const float *)U,
                                (const float *)bias, (float *)Y, (float *)T_save, ws, s);
    if (d->dtype == PF_F32 && p.skinny_fwd)
        return linear_fwd_skinny(d, p, (const float *)X, (const float *)V, (const float *)U,
                                 (const float *)bias, (float *)Y, (float *)T_save, ws, s);
    if (d->dtype == PF_F32 && p.t.ok)
        return linear_fwd_tiles<float>(d, p.t, 1, (const float *)X, (const float *)V, (const float *)U,
                                       (const float *)bias, (float *)Y, (float *)T_save, ws, s, ep ? *ep : LinEpilogue{});
    if (d->dtype == PF_F32)
        return linear_fwd_generic<float>(d, (const float *)X, (const float *)V, (const float *)U, (const float *)bias,
                                         (float *)Y, (float *)T_save, ws, s);
    const bool plain = !ep || (!ep->add && !ep->relu);
    if (p.two_fwd && !(plain && p.plain_chain)) {
        if (ep && ep->used) *ep->used = true;
        return launch_linear_two(s, "linear_fwd_two",
                                 LinTwoArgs{d->M, (int)d->in, (int)d->out, (int)d->r, (const uint16_t *)X, (const uint16_t *)V, (const uint16_t *)U,
                                            d->has_bias ? (const uint16_t *)bias : nullptr, ep ? (const uint16_t *)ep->add : nullptr, (uint16_t *)Y,
                                            (uint16_t *)T_save, ep ? ep->relu : 0, 1, 0, 0, 0, 0, 0, p.two_split},
                                 p.two_fwd);
    }
    if (p.chain_fwd)
        return linear_fwd_fused(d, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U, (const bf16_t *)bias,
                                (bf16_t *)Y, (bf16_t *)T_save, ws, s, ep ? *ep : LinEpilogue{});
    if (p.t.ok)
        return linear_fwd_tiles<bf16_t>(d, p.t, 1, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U,
                                        (const bf16_t *)bias, (bf16_t *)Y, (bf16_t *)T_save, ws, s,
                                        ep ? *ep : LinEpilogue{});
    return linear_fwd_generic<bf16_t>(d, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U,
                                      (const bf16_t *)bias, (bf16_t *)Y, (bf16_t *)T_save, ws, s);
}

int pf::linear_bwd_entry(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *dY,
                         const void *T_saved, void *dX, void *dU, void *dV, void *dbias, int accumulate,
                         void *workspace, size_t workspace_bytes, void *stream, int align, const LinEpilogue *ep)
{
    int st = check_linear_desc(d);
    if (st != PF_OK) return st;
    if (!V || !U) return PF_ERR_NULL;
    if (d->M > 0 && (!X || !dY)) return PF_ERR_NULL;
    if (any_misaligned({X, V, U, dY, T_saved, dX}, align) || any_misaligned({dU, dV, dbias}, 4)) return PF_ERR_UNSUPPORTED;
    const LinearPlan &p = plan_linear(d);
    const size_t need = p.bwd_bytes;
    if (need > 0 && (!workspace || workspace_bytes < need)) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    Workspace ws(workspace, workspace_bytes);
    hipStream_t s = (hipStream_t)stream;
    if (d->dtype == PF_F32 && p.small_bwd)
        return linear_bwd_small(d, p, (const float *)X, (const float *)V, (const float *)U,
                                (const float *)dY, (const float *)T_saved, (float *)dX, (float *)dU, (float *)dV,
                                (float *)dbias, accumulate, ws, s);
    if (d->dtype == PF_F32 && p.skinny_bwd)
        return linear_bwd_skinny(d, p, (const float *)X, (const float *)V, (const float *)U,
                                 (const float *)dY, (const float *)T_saved, (float *)dX, (float *)dU, (float *)dV,
                                 (float *)dbias, accumulate, ws, s);
    if (d->dtype == PF_F32 && p.t.ok)
        return linear_bwd_tiles<float>(d, p.t, 1, (const float *)X, (const float *)V, (const float *)U,
                                       (const float *)dY, (const float *)T_saved, (float *)dX, (float *)dU, (float *)dV,
                                       (float *)dbias, accumulate, ws, s, ep ? *ep : LinEpilogue{});
    if (d->dtype == PF_F32)
        return linear_bwd_generic<float>(d, (const float *)X, (const float *)V, (const float *)U, (const float *)dY,
                                         (const float *)T_saved, (float *)dX, (float *)dU, (float *)dV,
                                         (float *)dbias, accumulate, ws, s);
    if (p.two_bwd && dX)
        return linear_bwd_two(d, p, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U, (const bf16_t *)dY, (const bf16_t *)T_saved,
                              (bf16_t *)dX, (float *)dU, (float *)dV, (float *)dbias, accumulate, ws, s, ep ? *ep : LinEpilogue{});
    if (p.chain_bwd && dX)
        return linear_bwd_fused(d, p, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U, (const bf16_t *)dY,
                                (const bf16_t *)T_saved, (bf16_t *)dX, (float *)dU, (float *)dV, (float *)dbias,
                                accumulate, ws, s, ep ? *ep : LinEpilogue{});
    if (p.t.ok)
        return linear_bwd_tiles<bf16_t>(d, p.t, 1, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U, (const bf16_t *)dY,
                                        (const bf16_t *)T_saved, (bf16_t *)dX, (float *)dU, (float *)dV, (float *)dbias,
                                        accumulate, ws, s, ep ? *ep : LinEpilogue{});
    return linear_bwd_generic<bf16_t>(d, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U,
                                      (const bf16_t *)dY, (const bf16_t *)T_saved, (bf16_t *)dX, (float *)dU,
                                      (float *)dV, (float *)dbias, accumulate, ws, s);
}

extern "C" {

size_t pf_lowrank_linear_fwd_workspace_bytes(const pf_linear_desc *d)
{
    if (check_linear_desc(d) != PF_OK) return 0;
    return plan_linear(d).fwd_bytes;
}

size_t pf_lowrank_linear_bwd_workspace_bytes(const pf_linear_desc *d)
{
    if (check_linear_desc(d) != PF_OK) return 0;
    return plan_linear(d).bwd_bytes;
}

int pf_lowrank_linear_fwd(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *bias,
                          void *Y, void *T_save, void *workspace, size_t workspace_bytes, void *stream)
{
    return pf::linear_fwd_entry(d, X, V, U, bias, Y, T_save, workspace, workspace_bytes, stream, 16);
}

int pf_lowrank_linear_bwd(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *dY,
                          const void *T_saved, void *dX, void *dU, void *dV, void *dbias, int accumulate,
                          void *workspace, size_t workspace_bytes, void *stream)
{
    return pf::linear_bwd_entry(d, X, V, U, dY, T_saved, dX, dU, dV, dbias, accumulate, workspace, workspace_bytes,
                                stream, 16);
}

} // extern "C"

// ---------------------------------------------------- library-owned scratch
// Backward for callers that cannot allocate: the partial sums of the factor gradients, the rank-r gradient dT
// and a recomputed T live in this array instead of a caller's workspace.  Every GPU the library runs on holds
// its own copy at its own address until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; kernels are given the address that call returns.
static __device__ __align__(256) unsigned char scratch[PF_STATIC_SCRATCH_BYTES];

namespace pf {
constexpr int SCRATCH_MAX_DEVICES = 64;
static void *g_scratch_addr[SCRATCH_MAX_DEVICES]; // per device, looked up once
static std::mutex g_scratch_lock;

// Device address of `scratch` on the current device (no allocation: the array came with the code object).
static int scratch_on_current_device(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= SCRATCH_MAX_DEVICES)
        return set_hip_error(e != hipSuccess ? e : hipErrorInvalidDevice);
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_addr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return set_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol);
        g_scratch_addr[dev] = ptr;
    }
    *out = g_scratch_addr[dev];
    return PF_OK;
}
} // namespace pf

extern "C" {

size_t pf_static_scratch_bytes(void) { return (size_t)PF_STATIC_SCRATCH_BYTES; }

int pf_lowrank_linear_bwd_static(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *dY,
                                 const void *T_saved, void *dX, void *dU, void *dV, void *dbias, int accumulate,
                                 void *stream)
{
    int st = check_linear_desc(d);
    if (st != PF_OK) return st;
    if (plan_linear(d).bwd_bytes > (size_t)PF_STATIC_SCRATCH_BYTES) return PF_ERR_WORKSPACE;
    void *ptr = nullptr;
    st = scratch_on_current_device(&ptr);
    if (st != PF_OK) return st;
    // nothing in the backward pass reads scratch memory before writing it, so what the last call left is harmless
    return pf::linear_bwd_entry(d, X, V, U, dY, T_saved, dX, dU, dV, dbias, accumulate, ptr,
                                (size_t)PF_STATIC_SCRATCH_BYTES, stream, 16);
}

size_t pf_dense_linear_workspace_bytes(const pf_linear_desc *d)
{
    if (check_linear_desc(d) != PF_OK) return 0;
    return plan_dense_linear(d).bytes;
}

int pf_dense_linear_fwd(const pf_linear_desc *d, const void *X, const void *W, const void *bias, void *Y,
                        void *workspace, size_t workspace_bytes, void *stream)
{
    (void)workspace;
    (void)workspace_bytes;
    int st = check_linear_desc(d);
    if (st != PF_OK) return st;
    if (!W || (d->has_bias && !bias)) return PF_ERR_NULL;
    if (d->M == 0) return PF_OK;
    if (!X || !Y) return PF_ERR_NULL;
    hipStream_t s = (hipStream_t)stream;
    if (d->dtype == PF_F32)
        return dense_linear_fwd_t<float>(d, (const float *)X, (const float *)W, (const float *)bias, (float *)Y, s);
    return dense_linear_fwd_t<bf16_t>(d, (const bf16_t *)X, (const bf16_t *)W, (const bf16_t *)bias, (bf16_t *)Y, s);
}

int pf_dense_linear_bwd(const pf_linear_desc *d, const void *X, const void *W, const void *dY, void *dX, void *dW,
                        void *dbias, int accumulate, void *workspace, size_t workspace_bytes, void *stream)
{
    int st = check_linear_desc(d);
    if (st != PF_OK) return st;
    if (!W) return PF_ERR_NULL;
    if (d->M > 0 && (!X || !dY)) return PF_ERR_NULL;
    const size_t need = plan_dense_linear(d).bytes;
    if (!workspace || workspace_bytes < need) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    Workspace ws(workspace, workspace_bytes);
    hipStream_t s = (hipStream_t)stream;
    if (d->dtype == PF_F32)
        return dense_linear_bwd_t<float>(d, (const float *)X, (const float *)W, (const float *)dY, (float *)dX,
                                         (float *)dW, (float *)dbias, accumulate, ws, s);
    return dense_linear_bwd_t<bf16_t>(d, (const bf16_t *)X, (const bf16_t *)W, (const bf16_t *)dY, (bf16_t *)dX,
                                      (float *)dW, (float *)dbias, accumulate, ws, s);
}

size_t pf_lowrank_linear_shared_fwd_workspace_bytes(const pf_linear_shared_desc *d)
{
    pf_linear_desc one;
    if (check_shared_desc(d, &one) != PF_OK) return 0;
    return plan_shared(d, one).fwd_bytes;
}

size_t pf_lowrank_linear_shared_bwd_workspace_bytes(const pf_linear_shared_desc *d)
{
    pf_linear_desc one;
    if (check_shared_desc(d, &one) != PF_OK) return 0;
    return plan_shared(d, one).bwd_bytes;
}

int pf_lowrank_linear_shared_fwd(const pf_linear_shared_desc *d, const void *X, const void *V, const void *U,
                                 const void *bias, void *Y, void *T_save, void *workspace, size_t workspace_bytes,
                                 void *stream)
{
    pf_linear_desc one;
    int st = check_shared_desc(d, &one);
    if (st != PF_OK) return st;
    if (!V || !U || (d->has_bias && !bias)) return PF_ERR_NULL;
    if (d->M > 0 && (!X || !Y)) return PF_ERR_NULL;
    if (any_misaligned({X, V, U, bias, Y, T_save}, 16)) return PF_ERR_UNSUPPORTED;
    const SharedPlan sp = plan_shared(d, one);
    if (sp.fwd_bytes > 0 && (!workspace || workspace_bytes < sp.fwd_bytes)) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    if (d->M == 0) return PF_OK;
    const i64 M = d->M, in = d->n_in, out = d->n_out, r = d->r;
    hipStream_t s = (hipStream_t)stream;
    if (sp.fused_fwd) {
        LinChainArgs c{(const uint16_t *)X, (const uint16_t *)V, (const uint16_t *)U,
                       d->has_bias ? (const uint16_t *)bias : nullptr, (uint16_t *)Y, (uint16_t *)T_save, nullptr,
                       M, (int)in, (int)out};
        c.groups = d->groups;
        c.gs_W1 = in * r;
        c.gs_W2 = out * r;
        c.gs_bias = out;
        c.gs_out = M * out;
        c.gs_mid = M * r;
        return rows_fwd_pays(M, in, out, r, d->groups) ? launch_linear_rows(s, "linear_shared_fwd_rows", c)
                                                       : launch_linear_chain2(s, "linear_shared_fwd_fused", c);
    }
    if (sp.two_fwd)
        return launch_linear_two(s, "linear_shared_fwd_two",
                                 LinTwoArgs{M, (int)in, (int)out, (int)r, (const uint16_t *)X, (const uint16_t *)V, (const uint16_t *)U,
                                            d->has_bias ? (const uint16_t *)bias : nullptr, nullptr, (uint16_t *)Y, (uint16_t *)T_save, 0, d->groups,
                                            in * r, out * r, out, M * out, M * r, sp.two_split},
                                 sp.two_fwd);
    if (sp.t.ok) {
        Workspace ws(workspace, workspace_bytes);
        if (d->dtype == PF_F32)
            return linear_fwd_tiles<float>(&one, sp.t, d->groups, (const float *)X, (const float *)V, (const float *)U,
                                           (const float *)bias, (float *)Y, (float *)T_save, ws, s, LinEpilogue{});
        return linear_fwd_tiles<bf16_t>(&one, sp.t, d->groups, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U,
                                        (const bf16_t *)bias, (bf16_t *)Y, (bf16_t *)T_save, ws, s, LinEpilogue{});
    }
    const size_t el = d->dtype == PF_BF16 ? 2 : 4;
    for (int g = 0; g < d->groups && st == PF_OK; ++g)
        st = linear_fwd_entry(&one, X, (const char *)V + g * in * r * el, (const char *)U + g * out * r * el,
                              bias ? (const char *)bias + g * out * el : nullptr, (char *)Y + g * M * out * el,
                              T_save ? (char *)T_save + g * M * r * el : nullptr, workspace, workspace_bytes, stream,
                              layer_align(sp, el));
    return st;
}

int pf_lowrank_linear_shared_bwd(const pf_linear_shared_desc *d, const void *X, const void *V, const void *U,
                                 const void *dY, const void *T_saved, void *dX, void *dU, void *dV, void *dbias,
                                 int accumulate, void *workspace, size_t workspace_bytes, void *stream)
{
    pf_linear_desc one;
    int st = check_shared_desc(d, &one);
    if (st != PF_OK) return st;
    if (!V || !U) return PF_ERR_NULL;
    if (d->M > 0 && (!X || !dY)) return PF_ERR_NULL;
    if (any_misaligned({X, V, U, dY, T_saved, dX}, 16) || any_misaligned({dU, dV, dbias}, 4)) return PF_ERR_UNSUPPORTED;
    const SharedPlan sp = plan_shared(d, one);
    if (!workspace || workspace_bytes < sp.bwd_bytes) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    hipStream_t s = (hipStream_t)stream;
    const int G = d->groups;
    if (sp.t.ok) {
        Workspace ws(workspace, workspace_bytes);
        if (d->dtype == PF_F32)
            return linear_bwd_tiles<float>(&one, sp.t, G, (const float *)X, (const float *)V, (const float *)U,
                                           (const float *)dY, (const float *)T_saved, (float *)dX, (float *)dU,
                                           (float *)dV, (float *)dbias, accumulate, ws, s, LinEpilogue{});
        return linear_bwd_tiles<bf16_t>(&one, sp.t, G, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U,
                                        (const bf16_t *)dY, (const bf16_t *)T_saved, (bf16_t *)dX, (float *)dU,
                                        (float *)dV, (float *)dbias, accumulate, ws, s, LinEpilogue{});
    }
    if (d->dtype == PF_F32)
        return shared_bwd_loop<float>(d, sp, (const float *)X, (const float *)V, (const float *)U, (const float *)dY,
                                      (const float *)T_saved, (float *)dX, (float *)dU, (float *)dV,
                                      (float *)dbias, accumulate, workspace, workspace_bytes, s);
    return shared_bwd_loop<bf16_t>(d, sp, (const bf16_t *)X, (const bf16_t *)V, (const bf16_t *)U,
                                   (const bf16_t *)dY, (const bf16_t *)T_saved, (bf16_t *)dX, (float *)dU,
                                   (float *)dV, (float *)dbias, accumulate, workspace, workspace_bytes, s);
}

} // extern "C"

// ------------------------------------------------ entry points with an epilogue
// (the element-wise part is applied by the caller when *fused stays false)
int pf::linear_fwd_entry_ep(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *bias,
                            const void *residual, int act, void *Y, void *T_save, void *workspace,
                            size_t workspace_bytes, void *stream, bool *fused)
{
    *fused = false;
    const LinEpilogue ep{residual, nullptr, act == PF_ACT_RELU ? 1 : 0, fused};
    return pf::linear_fwd_entry(d, X, V, U, bias, Y, T_save, workspace, workspace_bytes, stream, 16, &ep);
}

int pf::linear_bwd_entry_ep(const pf_linear_desc *d, const void *X, const void *V, const void *U, const void *dZ,
                            const void *T_saved, const void *dX_add, int x_is_relu, void *dX, void *dU, void *dV,
                            void *dbias, int accumulate, void *workspace, size_t workspace_bytes, void *stream,
                            bool *fused)
{
    *fused = false;
    const LinEpilogue ep{dX_add, x_is_relu ? X : nullptr, 0, fused};
    return pf::linear_bwd_entry(d, X, V, U, dZ, T_saved, dX, dU, dV, dbias, accumulate, workspace, workspace_bytes,
                                stream, 16, &ep);
}
