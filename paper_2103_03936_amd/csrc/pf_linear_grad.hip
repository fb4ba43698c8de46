#include "pf_linear_grad.h"

#include "pf_tile.h"

namespace pf {

// A workgroup of eight wavefronts has 128 columns and all ranks of one gradient over a run of rows.  The contraction is the slow index
// of both operands: 64 rows of both lie in LDS as in memory and the fragments come from transposing reads.  What bounds it is how
// much a compute unit has in flight towards memory, so three chunks of 64 rows (96 KB at rank 128) are in registers behind the two in
// LDS, through descriptors (BufSrc) and without a condition, so that a wait is for the oldest of them alone.  A chunk takes 2000 clocks
// where 240 workgroups load 9.2 TB/s, 5 of them from HBM (16384 x 2048 and x 512, rank 128: 27.6 us; 8192 18.3, of which 9 are launch, first
// load and 16 MB of partial sums).  Ranks above 128 are six or eight blocks (FLAT: the ranks' chunk dealt out over its run of memory).  8192 rows,
// 512 -> 2048 and 2048 -> 512: 22.0 on the kernel of pf_linear_wgrad.hip with two tiles in flight.
template <int RB>
struct LinGradCfg {
    static constexpr int NT = 512, KC = 64, R = 32 * RB, RING = 3;
    // 64 columns by 64 ranks; of three wavefronts across the ranks two without any
    static constexpr int WM = 2, WN = RB > 1 ? RB / 2 : 1, WK = 8 / (WM * WN), NB = RB > 1 ? 2 : 1, STEPS = KC / 16;
    static constexpr int AP = 128 + 8, BP = R + 8, ABYTES = KC * AP * 2, BBYTES = KC * BP * 2, BUF = ABYTES + BBYTES;
    static constexpr int ACH = KC * 16 / NT, BPIECES = KC * RB * 4, BCH = BPIECES / NT > 0 ? BPIECES / NT : 1; // pieces per thread
    static constexpr bool FLAT = RB > 4; // the ranks' chunk, one run of memory, is dealt out piece by piece
    static constexpr int SP = R + 4, SBYTES = WK * 128 * SP * 4;
    static constexpr int BYTES = (2 * BUF > SBYTES ? 2 * BUF : SBYTES) + 8 * 128 * 4;
    static_assert(STEPS % WK == 0 && BYTES <= 160 * 1024, "");
};

template <int RB>
__global__ __launch_bounds__(512, 2) void linear_grad_kernel(LinGradArgs a)
{
    typedef LinGradCfg<RB> F;
    __shared__ __attribute__((aligned(16))) unsigned char smem[F::BYTES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hi = lane >> 5;
    const int first = (a.p[0].cols + 127) / 128, split = blockIdx.x % a.splits, tile = blockIdx.x / a.splits;
    const bool second = tile >= first;
    const LinGradProb &p = a.p[second];
    const int M = (int)a.M, r = a.r, cols = p.cols, col0 = (second ? tile - first : tile) * 128;
    const int begin = split * a.per * F::KC, end = min(M, begin + a.per * F::KC), chunks = (end - begin + F::KC - 1) / F::KC;
    const BufSrc sA(p.A, 2LL * M * cols), sB(p.B, 2LL * M * r);
    const int arow = tid / 16, acol = tid % 16 * 8, brow = tid / (RB * 4), bcol = tid % (RB * 4) * 8;
    constexpr int ASTEP = F::NT / 16, BSTEP = F::NT / (RB * 4);
    uint4 ar[F::RING][F::ACH], br[F::RING][F::BCH];
    const bool ain = col0 + acol < cols, bin = bcol < r && brow < F::KC;
    const int per = r / 8;
    int flat[F::BCH]; // where a thread's pieces of the ranks' chunk lie in LDS
#pragma unroll
    for (int u = 0; u < F::BCH; ++u)
        flat[u] = F::FLAT ? (tid + F::NT * u) / per * (F::BP * 2) + (tid + F::NT * u) % per * 16 : (brow + BSTEP * u) * (F::BP * 2) + bcol * 2;
    const auto load = [&](int q, uint4 (&x)[F::ACH], uint4 (&y)[F::BCH]) __attribute__((always_inline)) {
        const int row = begin + q * F::KC;
#pragma unroll
        for (int u = 0; u < F::ACH; ++u) {
            const int i = row + arow + ASTEP * u;
            x[u] = sA.load((ain & (i < end)) ? 2u * ((uint32_t)i * (uint32_t)cols + col0 + acol) : BUF_OUT);
        }
#pragma unroll
        for (int u = 0; u < F::BCH; ++u) {
            if constexpr (F::FLAT) {
                const int at = row * r + (tid + F::NT * u) * 8; // (a run's rows times r: below 2^30)
                y[u] = sB.load(((tid + F::NT * u < F::KC * per) & (at < end * r)) ? 2u * (uint32_t)at : BUF_OUT);
                continue;
            }
            const int i = row + brow + BSTEP * u;
            y[u] = sB.load((bin & (i < end)) ? 2u * ((uint32_t)i * (uint32_t)r + bcol) : BUF_OUT);
        }
    };
    float colsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const bool want = p.sums != nullptr;
    const auto store = [&](const uint4 (&x)[F::ACH], const uint4 (&y)[F::BCH], unsigned char *buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < F::ACH; ++u) {
            *(uint4 *)(buf + (arow + ASTEP * u) * (F::AP * 2) + acol * 2) = x[u];
            if (want) {
                float f[8];
                piece_floats<bf16_t>(x[u], f);
#pragma unroll
                for (int e = 0; e < 8; ++e) colsum[e] += f[e];
            }
        }
#pragma unroll
        for (int u = 0; u < F::BCH; ++u)
            if (F::FLAT ? tid + F::NT * u < F::KC * per : F::BPIECES >= F::NT || brow < F::KC) *(uint4 *)(buf + F::ABYTES + flat[u]) = y[u];
    };
#pragma unroll
    for (int i = 0; i < F::RING; ++i) load(i, ar[i], br[i]);
    const int wk = wave / (F::WM * F::WN), wm = wave / F::WN % F::WM, wn = wave % F::WN;
    const bool ranks = F::WM * F::WN * F::WK == 8 || __builtin_amdgcn_readfirstlane(wave) < F::WM * F::WN * F::WK;
    f32x16_t acc[2][F::NB]; // [block of columns][block of ranks]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < F::NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    store(ar[0], br[0], smem);
    load(F::RING, ar[0], br[0]);
    const auto step = [&](int q, const unsigned char *buf, unsigned char *next, uint4 (&x)[F::ACH], uint4 (&y)[F::BCH]) __attribute__((always_inline)) {
        __syncthreads();
        const uint16_t *as = (const uint16_t *)buf, *bs = (const uint16_t *)(buf + F::ABYTES);
        if (ranks)
#pragma unroll
        for (int s = 0; s < F::STEPS / F::WK; ++s) {
            const int k0 = (wk * (F::STEPS / F::WK) + s) * 16;
            bf16x8_t fa[2], fb[F::NB];
#pragma unroll
            for (int i = 0; i < 2; ++i) fa[i] = lds_frag_tr(as, F::AP, k0, wm * 64 + i * 32, lane);
#pragma unroll
            for (int j = 0; j < F::NB; ++j) fb[j] = lds_frag_tr(bs, F::BP, k0, (wn * F::NB + j) * 32, lane);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < F::NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
        }
        store(x, y, next);
        load(q + 1 + F::RING, x, y);
    };
    unsigned char *b0 = smem, *b1 = smem + F::BUF;
    for (int q = 0;;) { // (buffer and registers of a chunk are known at compile time)
        step(q, b0, b1, ar[1], br[1]);
        if (++q >= chunks) break;
        step(q, b1, b0, ar[2], br[2]);
        if (++q >= chunks) break;
        step(q, b0, b1, ar[0], br[0]);
        if (++q >= chunks) break;
        step(q, b1, b0, ar[1], br[1]);
        if (++q >= chunks) break;
        step(q, b0, b1, ar[2], br[2]);
        if (++q >= chunks) break;
        step(q, b1, b0, ar[0], br[0]);
        if (++q >= chunks) break;
    }
    // (the chunk stored last lies past the run: zeros, to the column sums as well)

    __syncthreads();
    float *ss = (float *)smem, *cs = (float *)(smem + F::BYTES - 8 * 128 * 4);
    if (ranks)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < F::NB; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const f32x4_t w = {acc[i][j][4 * k], acc[i][j][4 * k + 1], acc[i][j][4 * k + 2], acc[i][j][4 * k + 3]};
                *(f32x4_t *)&ss[(wk * 128 + wm * 64 + i * 32 + (lane & 31)) * F::SP + (wn * F::NB + j) * 32 + 8 * k + 4 * hi] = w;
            }
    if (want) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            colsum[e] += __shfl_xor(colsum[e], 16);
            colsum[e] += __shfl_xor(colsum[e], 32);
            if (lane < 16) cs[wave * 128 + acol + e] = colsum[e];
        }
    }
    __syncthreads();
    float *out = p.out + (i64)split * cols * r;
#pragma unroll 4
    for (int i = tid; i < 128 * RB * 8; i += F::NT) {
        const int c = i / (RB * 8), k = i % (RB * 8) * 4;
        f32x4_t w = *(const f32x4_t *)&ss[c * F::SP + k];
#pragma unroll
        for (int x = 1; x < F::WK; ++x) w += *(const f32x4_t *)&ss[(x * 128 + c) * F::SP + k];
        if (col0 + c < cols && k < r) *(f32x4_t *)&out[(i64)(col0 + c) * r + k] = w;
    }
    if (want && tid < 128 && col0 + tid < cols) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) v += cs[w * 128 + tid];
        p.sums[(i64)split * cols + col0 + tid] = v;
    }
}

bool linear_grad_supported(i64 M, i64 in, i64 out, i64 r)
{
    const i64 lim = 1LL << 30; // (descriptors of less than 2^31 bytes: of both matrices)
    return M >= 64 && in >= 8 && out >= 8 && in % 8 == 0 && out % 8 == 0 && r >= 8 && r <= 256 && r % 8 == 0 && M * in < lim && M * out < lim && M * r < lim;
}

// One workgroup to a compute unit, in one round, of at least two chunks.
LinGradPlan plan_linear_grad(i64 M, i64 in, i64 out, i64 r)
{
    const i64 tiles = (in + 127) / 128 + (out + 127) / 128, chunks = (M + 63) / 64;
    if (!linear_grad_supported(M, in, out, r) || tiles > 128) return LinGradPlan{0, 0};
    i64 splits = 256 / tiles;
    if (splits > 32) splits = 32;
    i64 per = (chunks + splits - 1) / splits;
    if (per < 2) per = 2;
    return LinGradPlan{(int)((chunks + per - 1) / per), (int)per};
}

int launch_linear_grad(hipStream_t s, const LinGradArgs &a)
{
    int st = PF_OK, tiles = 0;
    for (int i = 0; i < a.n; ++i) {
        if (!linear_grad_supported(a.M, a.p[i].cols, a.p[i].cols, a.r)) return PF_ERR_UNSUPPORTED;
        tiles += (a.p[i].cols + 127) / 128;
    }
    const i64 chunks = (a.M + 63) / 64;
    if (a.n < 1 || a.per < 1 || a.splits < 1 || (i64)a.splits * a.per < chunks || (i64)(a.splits - 1) * a.per >= chunks) return PF_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)(tiles * a.splits)), block(512);
    if (a.r <= 32) PF_LAUNCH(st, "linear_grads", linear_grad_kernel<1>, grid, block, s, a);
    else if (a.r <= 64) PF_LAUNCH(st, "linear_grads", linear_grad_kernel<2>, grid, block, s, a);
    else if (a.r <= 128) PF_LAUNCH(st, "linear_grads", linear_grad_kernel<4>, grid, block, s, a);
    else if (a.r <= 192) PF_LAUNCH(st, "linear_grads", linear_grad_kernel<6>, grid, block, s, a);
    else PF_LAUNCH(st, "linear_grads", linear_grad_kernel<8>, grid, block, s, a);
    return st;
}

} // namespace pf
