// Filter gradients of the factorized convolution from pixel-major tiles: dUk from dT and X seen through the taps, dVp (and the sums
// of dZ over the pixels) from T and dZ, both in one launch, as partial sums over runs of tiles.
#include "pf_conv_px_dev.h"

namespace pf {

// The contraction runs over the pixels, which is the slow direction of a pixel-major tile: fragments of both operands come from the
// transposing LDS reads, and a tap is again another row, here of dT: G(tap) = sum over p of dT[p - tap] X[p], so that X, which has more
// channels, needs no halo and a fragment of it serves several taps.  Groups of eight pixels of dT lie one after the other in LDS; the
// rows of a tile's pixels through all taps are looked up in a table that is written once per tile (computed per fragment, they took
// twice as long as the products), a row of zeros standing for what lies outside the plane.
// A workgroup of eight wavefronts owns all ranks x SC channels x the taps, in two LDS buffers with the next tile's operands in registers.
// With nine taps a wavefront has 32 ranks, 64 channels and a group of the taps; where eight are not used up so, and with one tap, they
// split a tile's eight steps of 16 pixels and their sums meet in LDS at the end.
// 128 images of 128 x 16 x 16, rank 32, 3 x 3: 15 us (the halo on X and nine taps per wavefront 19: the sums of four wavefronts that split
// the pixels met in LDS, 295 KB in and out); a tile takes 1800 clocks of products and their LDS reads, 2000 of addresses, table and stores,
// the partial sums of a workgroup 4500, which is the rate at which the chip writes them.
template <typename T, int KK, int RB>
struct PxWgCfg {
    static constexpr int V = PxEl<T>::V, PC = PxEl<T>::PC, F4 = sizeof(T) == 4;
    static constexpr int NT = 512, P = 128, SC = KK == 9 ? (RB == 4 ? 32 : 64) : F4 ? 64 : 128, CB = SC / 32;
    // one tap: a wavefront has MB rank blocks of one channel block
    static constexpr int MB = KK == 1 && RB == 4 ? 2 : 1, MW = RB / MB, NB = KK == 9 ? CB : 1, CW = CB / NB; // (RB blocks of ranks)
    static constexpr int TG = KK == 1 ? 1 : RB == 4 ? 2 : 4, KS = 8 / (CW * MW * TG);
    static constexpr int NTAP = (KK + TG - 1) / TG, TW = KK == 1 ? 0 : TG == 4 ? 4 : 8, TROW = TG * TW; // taps of a wavefront, words of the table per pixel pair
    static constexpr int NA = KK == 9 ? NTAP : MB;
    static constexpr int AROWS = KK == 9 ? PX_WG_ROWS : 136, APANEL = AROWS * 128, APANELS = (32 * RB + PC - 1) / PC, ABYTES = APANELS * APANEL, ZERO = AROWS - 1;
    static constexpr int BROWS = 136, BPANEL = BROWS * 128, BBYTES = (SC + PC - 1) / PC * BPANEL;
    static constexpr int TABLE = 64 * TROW * 4, BUF = ABYTES + BBYTES + TABLE;
    static constexpr int AO = 32 * RB / V, BO = SC / V, GS = V == 8 ? 4 : 5, BLOCKS = ((AO + BO) * (2 << GS) + NT - 1) / NT; // pieces, groups of a tile (log2), blocks per thread
    static constexpr int OPITCH = SC * KK + 4, OROWS = 32 * RB, OBYTES = KS * OROWS * OPITCH * 4;
    static constexpr int BYTES = 2 * BUF > OBYTES ? 2 * BUF : OBYTES;
    static __host__ __device__ constexpr int tap0(int tg) { return TG == 4 ? (tg ? 2 * tg + 1 : 0) : 5 * tg; } // first tap of a group (3, 2, 2, 2 or 5, 4)
    static_assert(BYTES + 16 <= 160 * 1024 && KS * TG * CW * MW == 8 && (KK == 9 || KS <= 4) && SC / V * 32 == (KK == 9 ? SC / V * 32 : NT), "");
};

// Float, one tap: products of one tile, 32 ranks x 32 channels over a wavefront's share of the pixels, in runs of 32 pixels with sums of their
// own.  A row holds 32 ranks or channels, which is what the lanes of an operand want: plain reads, free of conflicts.
template <typename F>
__device__ __forceinline__ void px_wgrad_f32(const unsigned char *as, const unsigned char *bs, int ks, f32x16_t &acc)
{
    const int lane = threadIdx.x & 63, hi = lane >> 5;
    // pixel 8 st + e + 4 hi of a run: where its piece lies in the row depends on st and e through their exclusive or only
    uint32_t own[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) own[z] = 4 * hi * 128 + ((hi << 4) ^ ((lane & 31) >> 2 << 4) ^ (z << 5)) + (lane & 3) * 4;
#pragma unroll
    for (int run = 0; run < 4 / F::KS; ++run) {
        const int row0 = (ks * (4 / F::KS) + run) * 32;
        f32x16_t sum;
        px_clear(sum);
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int at = (row0 + 8 * st + e) * 128 + own[e ^ st];
                sum = __builtin_amdgcn_mfma_f32_32x32x2f32(*(const float *)(as + at), *(const float *)(bs + at), sum, 0, 0, 0);
            }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] += sum[v];
    }
}

// Nine taps, channels whose X is infinite or NaN in a pixel at the edge of its plane: there a tap that reaches out of the plane multiplied
// it by the row of zeros, which is NaN for a term that does not exist.  Their gradients again, the terms that exist and no others, in runs of
// 128 pixels with sums of their own.  Such a value leaves none of its channel's sums finite, with any rank through any tap, so one sum of
// each channel is looked at (a check of all as they leave, and a barrier for it, took 0.4 of 22.5 us); what it starts takes milliseconds at
// worst and is for values that no healthy step has.
template <typename T, int SC>
__device__ __forceinline__ void px_wgrad_edges(const PxWgradArgs<T> &a, const PxGrad<T> &p, int c0, int begin, int end, float *part, uint32_t *flag)
{
    const PxPlaneOf<T> &g = a.gk;
    const int n = min(SC, p.C - c0), tid = threadIdx.x, NT = blockDim.x;
    __syncthreads(); // (what `flag` lies on has been read, and what is written again has been stored)
    for (int c = tid; c < n; c += NT) flag[c] = 0;
    __syncthreads();
    for (int i = tid; i < (end - begin) * n; i += NT) {
        const int c = i / (end - begin), px = begin + i - c * (end - begin), im = px_div(px, g.HW, g.mHW), q = px - im * g.HW, y = px_div(q, g.W, g.mW), x = q - y * g.W;
        const bool edge = y == 0 || y == g.H - 1 || x == 0 || x == g.W - 1;
        if (edge && !isfinite(px_float(p.B[(im * p.C + c0 + c) * g.HW + q]))) flag[c] = 1;
    }
    __syncthreads();
    for (int i = tid; i < a.r * n * 9; i += NT) {
        const int rank = i / (n * 9), j = i - rank * n * 9, c = j / 9, tap = j - c * 9, dy = 1 - tap / 3, dx = 1 - tap % 3;
        if (!flag[c]) continue;
        float all = 0.f;
        for (int run = begin; run < end; run += 128) {
            float sum = 0.f;
            for (int px = run; px < min(run + 128, end); ++px) {
                const int im = px_div(px, g.HW, g.mHW), q = px - im * g.HW, y = px_div(q, g.W, g.mW), x = q - y * g.W;
                if (y + dy >= 0 && y + dy < g.H && x + dx >= 0 && x + dx < g.W)
                    sum += px_float(p.A[(im * p.a_ch + rank) * g.HW + q + dy * g.W + dx]) * px_float(p.B[(im * p.C + c0 + c) * g.HW + q]);
            }
            all += sum;
        }
        part[rank * p.C * 9 + (c0 + c) * 9 + tap] = all;
    }
}

template <typename T, int KK, int RB>
__device__ __forceinline__ void px_wgrad(const PxWgradArgs<T> &a, const PxGrad<T> &p, int index, unsigned char *smem)
{
    typedef PxWgCfg<T, KK, RB> F;
    constexpr int NT = F::NT, V = F::V;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hi = lane >> 5;
    const int unit = index % p.units, group = index / p.units, c0 = unit * F::SC;
    const PxPlaneOf<T> &gt = KK == 9 ? a.gk : a.g1, &g1 = a.g1;
    const int tiles = (g1.N * g1.HW + F::P - 1) / F::P, t0 = group * p.per, t1 = min(tiles, t0 + p.per);
    // A thread's blocks: A's pieces, then B's, with as many groups of pixels as a tile can have.  Without a halo a row is a pixel of the tile.
    const int gshift = g1.HW % V == 0 ? F::GS : F::GS + 1, ashift = KK == 9 ? F::GS + 1 : gshift, nA = F::AO << ashift, nB = F::BO << gshift;
    int at[F::BLOCKS][V];
    bool live[F::BLOCKS];
    uint4 reg[F::BLOCKS][V];
    const bool whole = g1.HW % V == 0; // (rows of a block then stay the same from tile to tile)
#pragma unroll
    for (int u = 0; u < F::BLOCKS; ++u) {
        const int i = tid + NT * u;
        const bool isa = i < nA;
        const int j = isa ? i : i - nA, shift = isa ? ashift : gshift, gi = j & ((1 << shift) - 1), o = j >> shift;
#pragma unroll
        for (int e = 0; e < V; ++e) at[u][e] = (isa ? (o >> 3) * F::APANEL : F::ABYTES + (o >> 3) * F::BPANEL) + px_at(gi * V + e, o & 7);
    }
    const auto fetch = [&](int tile) __attribute__((always_inline)) {
        const PxTile ta = px_tile(gt, tile * F::P, F::P, true), tb = px_tile(g1, tile * F::P, F::P, true);
#pragma unroll
        for (int u = 0; u < F::BLOCKS; ++u) {
            const int i = tid + NT * u;
            if (i < nA + nB) {
                const bool isa = i < nA;
                const int j = isa ? i : i - nA, shift = isa ? ashift : gshift, gi = j & ((1 << shift) - 1), o = j >> shift;
                const int ch = isa ? p.a_ch : p.C, c = (isa ? 0 : c0) + V * o;
                const T *src = isa ? p.A : p.B;
                int n, q;
                live[u] = KK == 9 && isa ? px_group(gt, ta, gi, n, q) : px_group(g1, tb, gi, n, q);
                if (!live[u]) n = q = 0;
                // (channels past the last are sums that nobody stores)
                const int off = (n * ch + min(c, ch - 1)) * g1.HW + q, most = max(ch - 1 - c, 0) * g1.HW;
#pragma unroll
                for (int k = 0; k < V; ++k) reg[u][k] = px_load(src, off + min(k * g1.HW, most));
                if (!whole && !(KK == 9 && isa)) {
                    const int s0 = n * g1.HW + q - tb.p0, base = isa ? (o >> 3) * F::APANEL : F::ABYTES + (o >> 3) * F::BPANEL;
#pragma unroll
                    for (int e = 0; e < V; ++e) at[u][e] = base + px_at(s0 + e >= 0 && s0 + e < tb.p1 - tb.p0 ? s0 + e : F::BROWS - 1, o & 7);
                }
            }
        }
    };
    const auto store = [&](unsigned char *buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < F::BLOCKS; ++u)
            if (tid + NT * u < nA + nB && live[u]) {
#pragma unroll
                for (int e = 0; e < V; ++e) *(uint4 *)(buf + at[u][e]) = px_turn(reg[u], e);
            }
    };
    // rows of dT for pixels 8 j + e and 8 j + e + 4 of the tile and every tap
    const auto table = [&](int tile, unsigned char *buf) __attribute__((always_inline)) {
        const PxTile t = px_tile(gt, tile * F::P, F::P, true);
        if (tid < 64 * 6) {
            const int j = tid / 6, dy = 1 - tid % 6 / 2, half = tid & 1, p = t.p0 + (j >> 2) * 8 + (j & 3) + 4 * half;
            const int n = px_div(p, gt.HW, gt.mHW), q = p - n * gt.HW, y = px_div(q, gt.W, gt.mW), x = q - y * gt.W;
            const bool row = p < t.p1 && y + dy >= 0 && y + dy < gt.H;
            uint16_t *to = (uint16_t *)(buf + F::ABYTES + F::BBYTES) + j * (2 * F::TROW) + half;
#pragma unroll
            for (int d = 0; d < 3; ++d) { // tap (1 - dy, d) reaches back to (y + dy, x + 1 - d)
                const bool in = row && x + 1 - d >= 0 && x + 1 - d < gt.W;
                const int tap = (1 - dy) * 3 + d, tg = F::TG == 4 ? (tap < 3 ? 0 : (tap - 1) / 2) : tap / 5;
                to[2 * (tg * F::TW + tap - F::tap0(tg))] = (uint16_t)px_at(in ? px_linear(gt, t, n, q + dy * gt.W + 1 - d) : F::ZERO, 0);
            }
        }
    };
    // the last tile: no pixel where there is none
    const auto ragged = [&](int tile, unsigned char *buf) __attribute__((always_inline)) {
        if ((tile + 1) * F::P > g1.N * g1.HW) {
            __syncthreads();
            for (int i = tid; i < ((KK == 1 ? F::ABYTES : 0) + F::BBYTES) / 16; i += NT) ((uint4 *)(buf + (KK == 1 ? 0 : F::ABYTES)))[i] = px_zero();
            __syncthreads();
        }
    };
    const int ci = wave % F::CW, mi = wave / F::CW % F::MW, w2 = wave / (F::CW * F::MW), tg = w2 % F::TG, ks = w2 / F::TG;
    f32x16_t acc[F::NA][F::NB];
#pragma unroll
    for (int i = 0; i < F::NA; ++i)
#pragma unroll
        for (int j = 0; j < F::NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    float sum[KK == 1 ? V : 1];
#pragma unroll
    for (int e = 0; e < (KK == 1 ? V : 1); ++e) sum[e] = 0.f;
    // this lane's part of a transposing read: row and, in bytes, octet and half of a block of 32 channels
    const int trow = 8 * hi + (lane >> 2 & 3), toct = (lane >> 4 & 1) * 2 + (lane >> 1 & 1), thalf = (lane & 1) * 8;
    typedef __attribute__((address_space(3))) bf16x4_t *lds_ptr;
    const auto frag = [&](const unsigned char *x, const unsigned char *y) __attribute__((always_inline)) {
        const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)x), up = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)y);
        bf16x8_t r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = lo[e], r[4 + e] = up[e];
        return r;
    };
    if (KK == 9 && tid == 0) *(uint32_t *)(smem + F::BYTES) = 0; // (read at the very end)
    if (t0 < t1) {
        fetch(t0);
        if (KK == 9) {
            if (tid < 16 * F::APANELS) *(uint4 *)(smem + (tid & 1) * F::BUF + (tid >> 4) * F::APANEL + F::ZERO * 128 + (tid >> 1 & 7) * 16) = px_zero();
            table(t0, smem);
        }
        ragged(t0, smem);
        store(smem);
    }
    for (int tile = t0; tile < t1; ++tile) {
        unsigned char *buf = smem + (tile - t0 & 1) * F::BUF, *next = smem + (tile + 1 - t0 & 1) * F::BUF;
        const unsigned char *bs = buf + F::ABYTES;
        __syncthreads();
        if (tile + 1 < t1) {
            fetch(tile + 1);
            if (KK == 9) table(tile + 1, next);
        }
        if constexpr (F::F4) px_wgrad_f32<F>(buf + mi * F::APANEL, bs + ci * F::BPANEL, ks, acc[0][0]);
#pragma unroll
        for (int q = 0; q < (F::F4 ? 0 : 8 / F::KS); ++q) {
            const int step = ks * (8 / F::KS) + q, row = step * 16 + trow;
            bf16x8_t b[F::NB];
#pragma unroll
            for (int j = 0; j < F::NB; ++j) {
                const int cb = ci * F::NB + j, oct = (cb & 1) * 4 + toct;
                const unsigned char *panel = bs + (cb >> 1) * F::BPANEL + thalf;
                b[j] = frag(panel + px_at(row, oct), panel + px_at(row + 4, oct));
            }
            if constexpr (KK == 9) {
                const uint32_t *e = (const uint32_t *)(bs + F::BBYTES) + (step * 8 + hi * 4 + (lane >> 2 & 3)) * F::TROW + tg * F::TW;
                uint32_t tab[8];
#pragma unroll
                for (int t = 0; t < F::NTAP; t += 4) {
                    const uint4 v = *(const uint4 *)(e + t);
                    tab[t] = v.x, tab[t + 1] = v.y, tab[t + 2] = v.z, tab[t + 3] = v.w;
                }
                const uint32_t x = (((mi & 1) * 4 + toct) << 4) + thalf;
                const unsigned char *panel = buf + (mi >> 1) * F::APANEL;
#pragma unroll
                for (int t = 0; t < F::NTAP; ++t) {
                    if (t == F::NTAP - 1 && tg > 0) break; // (the first group has a tap more)
                    const uint32_t w = tab[t] ^ (x | x << 16);
                    const bf16x8_t f = frag(panel + (w & 0xffffu), panel + (w >> 16));
#pragma unroll
                    for (int j = 0; j < F::NB; ++j) acc[t][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, b[j], acc[t][j], 0, 0, 0);
                }
            } else {
#pragma unroll
                for (int i = 0; i < F::MB; ++i) {
                    const int rb = mi * F::MB + i, oct = (rb & 1) * 4 + toct;
                    const unsigned char *panel = buf + (rb >> 1) * F::APANEL + thalf;
                    acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(panel + px_at(row, oct), panel + px_at(row + 4, oct)), b[0], acc[i][0], 0, 0, 0);
                }
            }
        }
        if (KK == 1 && p.sums) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float v[V];
                px_unpack<T>(*(const uint4 *)(bs + (tid >> 8) * F::BPANEL + px_at((tid & 31) + 32 * k, tid >> 5 & 7)), v);
#pragma unroll
                for (int e = 0; e < V; ++e) sum[KK == 1 ? e : 0] += v[e];
            }
        }
        if (tile + 1 < t1) {
            ragged(tile + 1, next);
            store(next);
        }
    }
    // whole rows out, summed over the wavefronts that shared a block
    float *os = (float *)smem;
    float *part = p.part + (i64)group * a.r * p.C * KK;
    const int cols = min(F::SC, p.C - c0) * KK;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < F::NA; ++i) {
        const int tap = KK == 9 ? F::tap0(tg) + i : 0, row0 = (mi * F::MB + (KK == 9 ? 0 : i)) * 32;
        if (KK == 9 && i == F::NA - 1 && tg > 0) break;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = row0 + (v >> 2) * 8 + (v & 3) + 4 * hi;
#pragma unroll
            for (int j = 0; j < F::NB; ++j)
                os[(ks * F::OROWS + row) * F::OPITCH + ((ci * F::NB + j) * 32 + (lane & 31)) * KK + tap] = acc[i][j][v];
        }
    }
    if (KK == 9 && mi == 0) { // (a channel's sums with the first rank tell)
        float odd = 0.f;
#pragma unroll
        for (int j = 0; j < F::NB; ++j) odd = fmaf(acc[0][j][0], 0.f, odd);
        if (lane < 32 && odd != 0.f) *(uint32_t *)(smem + F::BYTES) = 1;
    }
    __syncthreads();
    constexpr int PR = F::SC * KK / 4; // pieces of four floats in a row
#pragma unroll 4
    for (int i = tid; i < F::OROWS * PR; i += NT) {
        const int rank = i / PR, col = (i - rank * PR) * 4;
        if (rank < a.r && col < cols) {
            f32x4_t v = *(const f32x4_t *)&os[rank * F::OPITCH + col];
#pragma unroll
            for (int w = 1; w < F::KS; ++w) v += *(const f32x4_t *)&os[(w * F::OROWS + rank) * F::OPITCH + col];
            *(f32x4_t *)&part[rank * p.C * KK + c0 * KK + col] = v;
        }
    }
    if constexpr (KK == 9) {
        if (*(const uint32_t *)(smem + F::BYTES)) px_wgrad_edges<T, F::SC>(a, p, c0, t0 * F::P, min(t1 * F::P, g1.N * g1.HW), part, (uint32_t *)smem);
    }
    if (KK == 1 && p.sums) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float v = sum[KK == 1 ? e : 0];
#pragma unroll
            for (int d = 1; d < 32; d <<= 1) v += __shfl_xor(v, d, 64);
            const int c = c0 + (tid >> 5) * V + e;
            if ((tid & 31) == 0 && c < p.C) p.sums[(i64)group * p.C + c] = v;
        }
    }
}

template <typename T, int K1, int RB>
__global__ __launch_bounds__(512, 2) void conv_px_wgrad_kernel(PxWgradArgs<T> a)
{
    constexpr int b1 = PxWgCfg<T, K1, RB>::BYTES, b2 = PxWgCfg<T, 1, RB>::BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[(b1 > b2 ? b1 : b2) + 16];
    const int first = a.p[0].units * a.p[0].groups, b = blockIdx.x;
    if (K1 == 9 && a.p[0].kk == 9 && b < first)
        px_wgrad<T, K1, RB>(a, a.p[0], b, smem);
    else
        px_wgrad<T, 1, RB>(a, b < first ? a.p[0] : a.p[1], b < first ? b : b - first, smem);
}

template <typename T>
int px_slab(int k, int r)
{
    if (sizeof(T) == 4) return 64;
    return k == 1 ? 128 : px_rank_blocks(r) == 4 ? 32 : 64;
}
template int px_slab<uint16_t>(int, int);
template int px_slab<float>(int, int);
template <typename T>
double px_wgrad_cost(int k, int r) // us per tile
{
    const int RB = px_rank_blocks(r);
    if (sizeof(T) == 4) return 1.7;
    return k == 3 ? (RB == 2 ? 6.5 : 4.6) : 3.0;
}
template double px_wgrad_cost<uint16_t>(int, int);
template double px_wgrad_cost<float>(int, int);
template <typename T>
void px_wgrad_plan(int npx, int r, int C1, int k, int C2, int (&groups)[2], int (&per)[2])
{
    const int tiles = (npx + 127) / 128, s1 = px_slab<T>(k, r), s2 = px_slab<T>(1, r);
    const int units[2] = {(C1 + s1 - 1) / s1, (C2 + s2 - 1) / s2};
    const double cost[2] = {px_wgrad_cost<T>(k, r), px_wgrad_cost<T>(1, r)};
    const double mb[2] = {4e-6 * r * C1 * k * k, 4e-6 * r * C2};
    double best = 1e30;
    // tiles per group of the first problem, from the fewest that one round of the chip allows to where they alone take longer than the best;
    // the second takes as long, or what room is left
    const int most1 = units[1] + units[0] < 256 ? (256 - units[1]) / units[0] : 1;
    for (int p1 = (tiles + most1 - 1) / most1; p1 <= tiles && p1 * cost[0] < best; ++p1) {
        const int g1 = (tiles + p1 - 1) / p1, room = 256 - units[0] * g1, most2 = room > units[1] ? room / units[1] : 1;
        int p2 = (int)(p1 * cost[0] / cost[1]), least = (tiles + most2 - 1) / most2;
        p2 = p2 < least ? least : p2 > tiles ? tiles : p2;
        const int g2 = (tiles + p2 - 1) / p2;
        const double a = p1 * cost[0], b = p2 * cost[1], t = (a > b ? a : b) + (g1 * mb[0] + g2 * mb[1]) * 1.5;
        if (t < best) {
            best = t;
            per[0] = p1, groups[0] = g1, per[1] = p2, groups[1] = g2;
        }
    }
}

template void px_wgrad_plan<uint16_t>(int, int, int, int, int, int (&)[2], int (&)[2]);
template void px_wgrad_plan<float>(int, int, int, int, int, int (&)[2], int (&)[2]);

template <typename T, int K1, int RB>
static int px_wgrad_l(hipStream_t s, const PxWgradArgs<T> &a)
{
    int st = PF_OK, blocks = 0;
    for (int i = 0; i < a.n; ++i) blocks += a.p[i].units * a.p[i].groups;
    PF_LAUNCH(st, "conv_wgrad_px", (conv_px_wgrad_kernel<T, K1, RB>), dim3(blocks), dim3(512), s, a);
    return st;
}
template <int K1>
static int px_wgrad_r(hipStream_t s, const PxWgradArgs<uint16_t> &a)
{
    return a.r <= 32 ? px_wgrad_l<uint16_t, K1, 1>(s, a) : a.r <= 64 ? px_wgrad_l<uint16_t, K1, 2>(s, a) : px_wgrad_l<uint16_t, K1, 4>(s, a);
}
template <typename T>
int launch_px_wgrad(hipStream_t s, const PxWgradArgs<T> &a)
{
    if (a.n < 1 || !px_bwd_takes<T>(a.p[0].kk == 9 ? 3 : 1, a.r)) return PF_ERR_UNSUPPORTED;
    if constexpr (sizeof(T) == 4)
        return px_wgrad_l<T, 1, 1>(s, a);
    else
        return a.p[0].kk == 9 ? px_wgrad_r<9>(s, a) : px_wgrad_r<1>(s, a);
}
template int launch_px_wgrad(hipStream_t, const PxWgradArgs<uint16_t> &);
template int launch_px_wgrad(hipStream_t, const PxWgradArgs<float> &);

} // namespace pf
