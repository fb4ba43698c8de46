#include "pf_linear_two.h"

#include "pf_tile.h"

namespace pf {

// A workgroup of eight wavefronts takes 32 MB rows through both stages.  Both factors stream through LDS as they lie in memory (the
// first one's fragments come from transposing reads): beside the products of a chunk the next one goes to LDS, piece by piece, and the one
// after that is requested.  Nothing is loaded or stored under a condition (BufSrc), so that a wait is for what is used and not for all that
// was issued since.  What bounds it: the memory pipe (19 clocks for a kilobyte of a factor, of which every workgroup reads all), and the
// chain of barrier, LDS reads, eight dependent products and the way of the outputs through LDS: 128 outputs of 32 rows take 1500 clocks,
// with all of them alone under 600 each.  2000 rows, 256 -> rank 64 -> 1024: 10.4 us on the tiled products (two or three launches),
// 6.6 before the pipelining, 5.9; 8192 x 512 -> 128 -> 512, three layers side by side 30.1 -> 19.0; 500 x 512 -> 128 -> 2048 18.8 -> 14.6.
// Backward the tiled products form dX beside the gradients (500 x 384 -> 96 -> 384: 10.7 against 13.0 with both stages here).
// Ranks from 136 to 256 in whole pieces (FLAT) have five, six or eight blocks: a wavefront per block in the first stage, up to 64 rows (32
// above rank 192: the LDS of a compute unit).  The widths of such factors are no powers of two, so their pieces are dealt out over the
// chunk, one run of memory; by rows, a fifth to a third of the loads would be of nothing.  8192 rows, tiled products / this: 640 -> 160
// -> 2560 37.4 / 20.8 us, 768 -> 192 -> 3072 40.4 / 26.1, 1024 -> 256 -> 1024 26.8 / 24.3.
// WM x WN wavefronts over (ranks, rows), WK of them split the contraction of the first stage; the second takes 128 outputs at a time.
template <int RB, int MB>
struct LinTwoCfg {
    static constexpr int NT = 512, MR = 32 * MB, Kp = 32 * RB, KC = RB == 8 || (RB == 4 && MB == 4) ? 64 : 128;
    static constexpr bool FLAT = RB > 4; // a factor's chunk, which is one run of memory, is dealt out piece by piece, and some wavefronts have no ranks
    static constexpr int WM = RB, WN = 8 / RB < MB ? 8 / RB : MB, WK = 8 / (WM * WN), NB = MB / WN, STEPS = KC / 16 / WK;
    static constexpr int VP = Kp + 8, XP = KC + 8;                                          // pitches (elements)
    static constexpr int VCH = (KC * RB * 4 + NT - 1) / NT, XCH = MR * KC / 8 / NT > 0 ? MR * KC / 8 / NT : 1; // pieces per thread
    static constexpr int VBYTES = KC * VP * 2, XBYTES = MR * XP * 2, BUF = VBYTES + XBYTES;
    static constexpr int SP = Kp + 4, SBYTES = WK > 1 ? WK * MR * SP * 4 : 0;                // sums of the first stage
    // second stage: a wavefront has 32 outputs of NB2 blocks of rows
    static constexpr int OC = 128, NB2 = MB < 4 ? 1 : 2, AP = Kp + 8, ABYTES = OC * AP * 2, ACH = (OC * RB * 4 + NT - 1) / NT;
    static constexpr int TP = Kp + 8, TBYTES = MR * TP * 2, OP = OC + 8, OBYTES = MR * OP * 2, BIAS = OC * 2;
    static constexpr int S1 = TBYTES + (2 * BUF > SBYTES ? 2 * BUF : SBYTES);
    static constexpr int O0 = 0, A0 = TBYTES > 2 * OBYTES ? TBYTES : 2 * OBYTES, B0 = A0 + 2 * ABYTES, S2 = B0 + 2 * BIAS; // (mid is gone when outputs come)
    static constexpr int BYTES = S1 > S2 ? S1 : S2;
    static_assert(KC / 16 % WK == 0 && 2 * RB % ACH == 0 && WK >= 1, "whole steps");
    static_assert(BYTES <= 160 * 1024, "LDS of a compute unit");
};

// Piece `col` (eight elements) of row `row` of [rows][r]: loaded from inside the array, put in place when it is stored.
struct LinPiece {
    int off, nv; // element wanted, elements of it that exist
    __device__ __forceinline__ LinPiece(int row, int col, int rows, int r) : off(min(row, rows - 1) * r + col * 8), nv(row < rows ? r - col * 8 : 0) {}
    __device__ __forceinline__ uint4 load(const uint16_t *p, int total) const { return ldg16((const char *)p + 2u * (uint32_t)min(off, total - 8)); }
    __device__ __forceinline__ uint4 fix(uint4 v, int total) const
    {
        if (nv >= 8) return v;
        const int s = off - min(off, total - 8);
        if (s) v = piece_shift<2>(v, min(s, 8));
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] &= nv >= 2 * j + 2 ? 0xffffffffu : nv == 2 * j + 1 ? 0xffffu : 0u;
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
};

// bf16 elements of v where those of m are above zero (as integers 1 .. 0x7f80: NaN is not)
__device__ __forceinline__ uint4 lt_kept(uint4 v, uint4 m)
{
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    const auto one = [](uint32_t x, uint32_t k) __attribute__((always_inline)) {
        const us2 left = __builtin_elementwise_sub_sat(us2{0x7f80, 0x7f80}, (us2)(__builtin_bit_cast(us2, k) - us2{1, 1})); // 0: not kept
        return x & __builtin_bit_cast(uint32_t, (us2)(us2{0, 0} - __builtin_elementwise_min(left, us2{1, 1})));
    };
    return make_uint4(one(v.x, m.x), one(v.y, m.y), one(v.z, m.z), one(v.w, m.w));
}

// EVEN: ranks in whole pieces.  Everything is then loaded and stored through descriptors without a branch.
// ADD, MASK: a residual is added; outputs are kept where `mask` is positive (its pieces are those that a thread stores).
template <int RB, int MB, bool EVEN, bool ADD, bool MASK>
__global__ __launch_bounds__(512, 2) void linear_two_kernel(LinTwoArgs a)
{
    typedef LinTwoCfg<RB, MB> F;
    constexpr int NT = F::NT, MR = F::MR, KC = F::KC, Kp = F::Kp;
    __shared__ __attribute__((aligned(16))) unsigned char lt_smem[F::BYTES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hi = lane >> 5;
    const int K = a.K, N = a.N, r = a.r, M = (int)a.M, m0 = blockIdx.x * MR;
    constexpr int TP = F::TP;
    uint16_t *ts = (uint16_t *)lt_smem;
    unsigned char *base = lt_smem + F::TBYTES;
    const i64 z = blockIdx.z;
    const uint16_t *W1 = a.W1 + z * a.s_W1, *W2 = a.W2 + z * a.s_W2, *bias = a.bias ? a.bias + z * a.s_bias : nullptr;
    uint16_t *out = a.out + z * a.s_out, *mid = a.mid ? a.mid + z * a.s_mid : nullptr;
    const int chunks = (N + F::OC - 1) / F::OC, c_begin = chunks * (int)blockIdx.y / a.osplit, c_end = chunks * ((int)blockIdx.y + 1) / a.osplit;

    // ------------------------------------------------ mid
    uint4 vr[F::VCH], xr[2][F::XCH]; // (the factors come from L2, the input from further away)
    const int steps = (K + KC - 1) / KC;
    // A thread's pieces lie in one column of the factor and one of the input.
    const BufSrc sV(W1, 2LL * K * r), sX(a.in, 2LL * M * K), sU(W2, 2LL * N * r), sB(bias, 2LL * N), sA(a.add, 2LL * M * N), sM(a.mask, 2LL * M * N), sY(out, 2LL * M * N);
    const int per = r / 8, vrow = tid / (RB * 4), vcol = tid % (RB * 4), xrow = tid / (KC / 8), xcol = tid % (KC / 8) * 8;
    constexpr int VSTEP = NT / (RB * 4), XSTEP = NT / (KC / 8);
    const bool vin = vcol * 8 < r;
    int flat[F::FLAT ? F::ACH : 1]; // where a thread's pieces of a chunk of either factor lie in LDS
    if constexpr (F::FLAT) {
        static_assert(F::VP == F::AP && F::VCH <= F::ACH, "both factors' chunks lie alike");
#pragma unroll
        for (int u = 0; u < F::ACH; ++u) flat[u] = (tid + NT * u) / per * (F::AP * 2) + (tid + NT * u) % per * 16;
    }
    uint32_t xat[F::XCH];
#pragma unroll
    for (int u = 0; u < F::XCH; ++u) xat[u] = (uint32_t)(m0 + xrow + XSTEP * u) * (uint32_t)K + xcol;
    const auto load_v = [&](int q, int u) __attribute__((always_inline)) {
        if constexpr (F::FLAT) {
            vr[u] = sV.load(tid + NT * u < KC * per ? 2u * (uint32_t)(q * KC * r + (tid + NT * u) * 8) : BUF_OUT);
            return;
        }
        const int row = q * KC + vrow + VSTEP * u;
        vr[u] = EVEN ? sV.load(vin ? 2u * (uint32_t)(row * r + vcol * 8) : BUF_OUT) : LinPiece(row, vcol, K, r).load(W1, K * r);
    };
    const auto load_x = [&](int q, int u, uint4 &x) __attribute__((always_inline)) { x = sX.load(q * KC + xcol < K ? 2u * (xat[u] + q * KC) : BUF_OUT); };
    const auto store_v = [&](int q, int u, unsigned char *buf) __attribute__((always_inline)) { // (ranks past the last are sums that nobody reads)
        if constexpr (F::FLAT) {
            if (tid + NT * u < KC * per) *(uint4 *)(buf + flat[u]) = vr[u];
            return;
        }
        *(uint4 *)(buf + (vrow + VSTEP * u) * (F::VP * 2) + vcol * 16) = EVEN ? vr[u] : LinPiece(q * KC + vrow + VSTEP * u, vcol, K, r).fix(vr[u], K * r);
    };
    const auto store_x = [&](int u, unsigned char *buf, const uint4 &x) __attribute__((always_inline)) {
        if (MR >= XSTEP || xrow < MR) *(uint4 *)(buf + F::VBYTES + (xrow + XSTEP * u) * (F::XP * 2) + xcol * 2) = x;
    };
#pragma unroll
    for (int u = 0; u < F::XCH; ++u) load_x(0, u, xr[0][u]);
#pragma unroll
    for (int u = 0; u < F::VCH; ++u) load_v(0, u);
#pragma unroll
    for (int u = 0; u < F::XCH; ++u) load_x(1, u, xr[1][u]);
    const int wk = wave / (F::WM * F::WN), wm = wave / F::WN % F::WM, wn = wave % F::WN;
    const bool ranks = !F::FLAT || __builtin_amdgcn_readfirstlane(wave) < F::WM;
    f32x16_t acc[F::NB];
#pragma unroll
    for (int j = 0; j < F::NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll
    for (int u = 0; u < F::XCH; ++u) {
        store_x(u, base, xr[0][u]);
        load_x(2, u, xr[0][u]);
    }
#pragma unroll
    for (int u = 0; u < F::VCH; ++u) {
        store_v(0, u, base);
        load_v(1, u);
    }
    // a chunk's products beside the next one's way to LDS and the one after that's from memory
    const auto step1 = [&](int q, const unsigned char *buf, unsigned char *next, uint4 (&x)[F::XCH]) __attribute__((always_inline)) {
        __syncthreads();
        bf16x8_t f[2], b[2][F::NB];
        const auto frags = [&](int s) __attribute__((always_inline)) {
            const int st = wk * F::STEPS + s;
            f[s & 1] = lds_frag_tr((const uint16_t *)buf, F::VP, st * 16, wm * 32, lane);
#pragma unroll
            for (int j = 0; j < F::NB; ++j)
                b[s & 1][j] = *(const bf16x8_t *)(buf + F::VBYTES + ((wn * F::NB + j) * 32 + (lane & 31)) * (F::XP * 2) + (st * 16 + hi * 8) * 2);
        };
        if (ranks) frags(0);
#pragma unroll
        for (int s = 0; s < F::STEPS; ++s) {
            if (ranks && s + 1 < F::STEPS) frags(s + 1);
#pragma unroll
            for (int j = 0; j < F::NB; ++j)
                if (ranks) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s & 1], b[s & 1][j], acc[j], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < F::XCH; ++u)
                if (u * F::STEPS / F::XCH == s) {
                    store_x(u, next, x[u]);
                    load_x(q + 3, u, x[u]);
                }
#pragma unroll
            for (int u = 0; u < F::VCH; ++u)
                if (u * F::STEPS / F::VCH == s) {
                    store_v(q + 1, u, next);
                    load_v(q + 2, u);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int q = 0; q < steps - 1; q += 2) {
        step1(q, base, base + F::BUF, xr[1]);
        step1(q + 1, base + F::BUF, base, xr[0]);
    }
    if (steps & 1) step1(steps - 1, base, base + F::BUF, xr[1]);

    // the sums -> LDS in bf16, zero past the last rank whatever the input holds
    if constexpr (F::WK == 1) {
        if (ranks)
#pragma unroll
        for (int j = 0; j < F::NB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) { // ranks 32 wm + 8 q + 4 hi ..
                const int left = r - (32 * wm + 8 * q + 4 * hi);
                uint2 w;
                w.x = pack_bf16x2(left > 0 ? acc[j][4 * q] : 0.f, left > 1 ? acc[j][4 * q + 1] : 0.f);
                w.y = pack_bf16x2(left > 2 ? acc[j][4 * q + 2] : 0.f, left > 3 ? acc[j][4 * q + 3] : 0.f);
                *(uint2 *)&ts[((wn * F::NB + j) * 32 + (lane & 31)) * TP + 32 * wm + 8 * q + 4 * hi] = w;
            }
    } else {
        float *ss = (float *)base;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < F::NB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4_t w = {acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
                *(f32x4_t *)&ss[(wk * MR + (wn * F::NB + j) * 32 + (lane & 31)) * F::SP + 32 * wm + 8 * q + 4 * hi] = w;
            }
        __syncthreads();
        for (int i = tid; i < MR * RB * 4; i += NT) {
            const int row = i / (RB * 4), o = i % (RB * 4);
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; e += 4) {
                f32x4_t w = *(const f32x4_t *)&ss[row * F::SP + o * 8 + e];
#pragma unroll
                for (int k = 1; k < F::WK; ++k) w += *(const f32x4_t *)&ss[(k * MR + row) * F::SP + o * 8 + e];
#pragma unroll
                for (int x = 0; x < 4; ++x) v[e + x] = o * 8 + e + x < r ? w[x] : 0.f;
            }
            *(uint4 *)&ts[row * TP + o * 8] = floats_piece<bf16_t>(v);
        }
    }

    // ------------------------------------------------ out
    // 128 at a time.  A lane of the products has four neighbouring outputs of a row in every fourth register: stored from there, 32 bytes of
    // a row side by side, a kilobyte took 65 clocks of the memory pipe, of whole rows 20.  So they pass through LDS, in bf16 and two buffers,
    // where the residual waits in the places of the outputs that it is added to; a piece of a row belongs to one thread on both ways.
    constexpr int NB2 = F::NB2, OP = F::OP;
    const int wo = wave % 4, wr = wave / 4 * NB2; // outputs, first block of rows
    const bool active = MB > 1 || __builtin_amdgcn_readfirstlane(wave) < 4;
    uint4 ar[F::ACH], add[2][ADD ? MB : 1], keep[2][MASK ? MB : 1], bs;
    const int parts = c_end - c_begin, orow = tid / 16, ocol = tid % 16 * 8; // (and every 32nd row from there)
    uint16_t *as0 = (uint16_t *)(lt_smem + F::A0), *as1 = (uint16_t *)(lt_smem + F::A0 + F::ABYTES);
    uint16_t *os0 = (uint16_t *)(lt_smem + F::O0), *os1 = (uint16_t *)(lt_smem + F::O0 + F::OBYTES);
    uint16_t *bs0 = (uint16_t *)(lt_smem + F::B0), *bs1 = (uint16_t *)(lt_smem + F::B0 + F::BIAS);
    const auto load_u = [&](int q, int u) __attribute__((always_inline)) {
        if constexpr (F::FLAT) {
            ar[u] = sU.load(tid + NT * u < F::OC * per ? 2u * (uint32_t)((c_begin + q) * F::OC * r + (tid + NT * u) * 8) : BUF_OUT);
            return;
        }
        const int row = (c_begin + q) * F::OC + vrow + VSTEP * u;
        ar[u] = EVEN ? sU.load(vin ? 2u * (uint32_t)(row * r + vcol * 8) : BUF_OUT) : LinPiece(row, vcol, N, r).load(W2, N * r);
    };
    const auto store_u = [&](int q, int u, uint16_t *as) __attribute__((always_inline)) { // (half a step past the last rank: zero)
        if constexpr (F::FLAT) {
            if (tid + NT * u < F::OC * per) *(uint4 *)((unsigned char *)as + flat[u]) = ar[u];
            return;
        }
        const int row = vrow + VSTEP * u;
        *(uint4 *)&as[row * F::AP + vcol * 8] = EVEN ? ar[u] : LinPiece((c_begin + q) * F::OC + row, vcol, N, r).fix(ar[u], N * r);
    };
    const auto out_at = [&](int q, int u) __attribute__((always_inline)) {
        const int o = (c_begin + q) * F::OC + ocol, row = m0 + orow + 32 * u;
        return ((q >= 0) & (o < N) & (row < M)) ? 2u * ((uint32_t)row * (uint32_t)N + o) : BUF_OUT;
    };
    const auto load_b = [&](int q) __attribute__((always_inline)) { bs = sB.load(tid < 16 ? 2u * (uint32_t)((c_begin + q) * F::OC + ocol) : BUF_OUT); };
#pragma unroll
    for (int u = 0; u < F::ACH; ++u) load_u(0, u);
    if (tid < 64) load_b(0);
    if constexpr (ADD) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int u = 0; u < MB; ++u) add[i][u] = sA.load(out_at(i, u));
    }
    if constexpr (MASK) {
#pragma unroll
        for (int u = 0; u < MB; ++u) keep[0][u] = sM.load(out_at(0, u)), keep[1][u] = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    bf16x8_t tf[NB2][2 * RB];
    if (active) {
#pragma unroll
        for (int j = 0; j < NB2; ++j)
#pragma unroll
            for (int st = 0; st < 2 * RB; ++st) tf[j][st] = *(const bf16x8_t *)&ts[((wr + j) * 32 + (lane & 31)) * TP + st * 16 + hi * 8];
    }
    if (mid && blockIdx.y == 0) {
        const int pieces = (r + 7) / 8;
        for (int i = tid; i < MR * pieces; i += NT) {
            const int o = i % pieces, row = i / pieces;
            if (m0 + row < M) {
                const uint4 v = *(const uint4 *)&ts[row * TP + o * 8];
                uint16_t *to = mid + (i64)(m0 + row) * r + o * 8;
                if (r - o * 8 >= 8) {
                    stg16(to, v);
                } else {
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (e < r - o * 8) to[e] = (uint16_t)(w[e / 2] >> (16 * (e & 1)));
                }
            }
        }
    }
    const bool relu = a.relu != 0;
    __syncthreads();
    if constexpr (F::FLAT) { // (zeros past the last rank, which no piece covers)
        for (int i = tid; i < 2 * F::OC * (RB * 4 - per); i += NT)
            *(uint4 *)(lt_smem + F::A0 + i / (RB * 4 - per) * (F::AP * 2) + (per + i % (RB * 4 - per)) * 16) = make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < F::ACH; ++u) {
        store_u(0, u, as0);
        load_u(1, u);
    }
    if (tid < 64) {
        if (tid < 16) *(uint4 *)&bs0[ocol] = bs;
        load_b(1);
    }
    if constexpr (ADD) {
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            *(uint4 *)&os0[(orow + 32 * u) * OP + ocol] = add[0][u];
            add[0][u] = sA.load(out_at(2, u));
        }
    }
    // 128 outputs' products, beside them the next factor rows on their way to LDS, those after them from memory, and the outputs before
    const auto step2 = [&](int q, const uint16_t *as, uint16_t *anext, uint16_t *os, uint16_t *obefore, const uint16_t *bias_s, uint16_t *bnext,
                           uint4 (&x)[ADD ? MB : 1], uint4 (&m)[MASK ? MB : 1]) __attribute__((always_inline)) {
        __syncthreads();
        uint4 before[MB];
#pragma unroll
        for (int u = 0; u < MB; ++u) before[u] = *(const uint4 *)&obefore[(orow + 32 * u) * OP + ocol];
        const auto frag = [&](int st) __attribute__((always_inline)) { return *(const bf16x8_t *)&as[(wo * 32 + (lane & 31)) * F::AP + st * 16 + hi * 8]; };
        bf16x8_t f[2];
        f32x16_t y[NB2];
        if (active) f[0] = frag(0);
        if (active) { // the sums start from the bias and the residual
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint2 b = *(const uint2 *)&bias_s[wo * 32 + 8 * k + 4 * hi];
#pragma unroll
                for (int j = 0; j < NB2; ++j) {
                    y[j][4 * k] = __uint_as_float(b.x << 16), y[j][4 * k + 1] = __uint_as_float(b.x & 0xffff0000u);
                    y[j][4 * k + 2] = __uint_as_float(b.y << 16), y[j][4 * k + 3] = __uint_as_float(b.y & 0xffff0000u);
                    if constexpr (ADD) {
                        const uint2 d = *(const uint2 *)&os[((wr + j) * 32 + (lane & 31)) * OP + wo * 32 + 8 * k + 4 * hi];
                        y[j][4 * k] += __uint_as_float(d.x << 16), y[j][4 * k + 1] += __uint_as_float(d.x & 0xffff0000u);
                        y[j][4 * k + 2] += __uint_as_float(d.y << 16), y[j][4 * k + 3] += __uint_as_float(d.y & 0xffff0000u);
                    }
                }
            }
        }
#pragma unroll
        for (int st = 0; st < 2 * RB; ++st) {
            if (active) {
                if (st + 1 < 2 * RB) f[(st + 1) & 1] = frag(st + 1);
#pragma unroll
                for (int j = 0; j < NB2; ++j) y[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[st & 1], tf[j][st], y[j], 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < F::ACH; ++u)
                if (u * 2 * RB / F::ACH == st) {
                    store_u(q + 1, u, anext);
                    load_u(q + 2, u);
                }
#pragma unroll
            for (int u = 0; u < MB; ++u)
                if (u * 2 * RB / MB == st) {
                    if constexpr (MASK) before[u] = lt_kept(before[u], m[u]), m[u] = sM.load(out_at(q + 1, u));
                    sY.store(out_at(q - 1, u), before[u]);
                    if constexpr (ADD) {
                        *(uint4 *)&obefore[(orow + 32 * u) * OP + ocol] = x[u];
                        x[u] = sA.load(out_at(q + 3, u));
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (tid < 64) {
            if (tid < 16) *(uint4 *)&bnext[ocol] = bs;
            load_b(q + 2);
        }
        if (active) {
#pragma unroll
            for (int j = 0; j < NB2; ++j) {
                if (relu) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) y[j][v] = fmaxf(y[j][v], 0.f);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *(uint2 *)&os[((wr + j) * 32 + (lane & 31)) * OP + wo * 32 + 8 * k + 4 * hi] =
                        make_uint2(pack_bf16x2(y[j][4 * k], y[j][4 * k + 1]), pack_bf16x2(y[j][4 * k + 2], y[j][4 * k + 3]));
            }
        }
    };
    const auto last = [&](int q, const uint16_t *os, const uint4 (&m)[MASK ? MB : 1]) __attribute__((always_inline)) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            const uint4 v = *(const uint4 *)&os[(orow + 32 * u) * OP + ocol];
            sY.store(out_at(q, u), MASK ? lt_kept(v, m[MASK ? u : 0]) : v);
        }
    };
    int q = 0;
    for (; q < parts - 1; q += 2) {
        step2(q, as0, as1, os0, os1, bs0, bs1, add[1], keep[1]);
        step2(q + 1, as1, as0, os1, os0, bs1, bs0, add[0], keep[0]);
    }
    if (parts & 1) {
        step2(q, as0, as1, os0, os1, bs0, bs1, add[1], keep[1]);
        last(q, os0, keep[0]);
    } else {
        last(q - 1, os1, keep[1]);
    }
}

static int lt_blocks(i64 r) { return r <= 32 ? 1 : r <= 64 ? 2 : r <= 128 ? 4 : r <= 160 ? 5 : r <= 192 ? 6 : 8; }
static int lt_most(i64 r) { return r <= 128 ? 4 : r <= 192 ? 2 : 1; } // blocks of 32 rows that a workgroup's LDS has room for

bool linear_two_supported(i64 M, i64 K, i64 N, i64 r)
{
    const i64 lim = 1LL << 30;
    return M >= 1 && K >= 8 && N >= 8 && K % 8 == 0 && N % 8 == 0 && r >= 8 && (r <= 128 || (r <= 256 && r % 8 == 0)) && M * K < lim &&
           M * N < lim && K * r < lim && N * r < lim;
}

// Fitted to times of 130 shapes (1 to 16384 rows, 128 to 4096 wide, ranks 8 to 128) with every number of rows and share of the outputs, 8 %
// rms: what a workgroup costs and 32 rows through a chunk of either stage, and what a compute unit reads and writes 12 and 14 ns per KB.
// Ranks above 128, where a chunk's products and its barrier cost more, fitted by themselves: 312 shapes of 64 to 16384 rows, 5 % rms.
double plan_linear_two(i64 M, i64 K, i64 N, i64 r, int groups, int &rows, int &osplit)
{
    double best = 1e30;
    const int RB = lt_blocks(r), chunks = (int)((N + 127) / 128);
    for (int mb = 1; mb <= lt_most(r); mb *= 2) {
        const i64 tiles = (M + 32 * mb - 1) / (32 * mb);
        const int KC = RB == 8 || (RB == 4 && mb == 4) ? 64 : 128;
        const double steps = (double)((K + KC - 1) / KC);
        for (int os = 1; os <= chunks && os <= 8; os *= 2) {
            const int per = (chunks + os - 1) / os;
            const i64 rounds = (tiles * os * groups + 255) / 256;
            const double full = tiles * os * groups < 256 ? tiles * os * groups / 256.0 : 1;
            const double kb1 = K * (r + 32.0 * mb) / 512, kb2 = per * 128.0 * (r + 32 * mb) / 512;
            const double wide = 2.53 + rounds * (2.6 + steps * (0.319 + 0.205 * mb * KC / 128) + per * (0.25 + 0.035 * mb) + 0.0026 * kb1 + 0.0119 * kb2 +
                                                 0.0024 * full * (kb1 + kb2));
            const double t = RB > 4 ? wide : 3.49 + rounds * (0.77 + 0.0392 * steps * mb + 0.0044 * per + 0.0452 * per * mb + 0.0121 * kb1 + 0.0137 * kb2 +
                                              0.0049 * full * (kb1 + kb2) + (r % 8 ? 0.33 * (steps + per) : 0));
            if (t < best) best = t, rows = 32 * mb, osplit = os;
        }
    }
    return best;
}

template <int RB, int MB>
static int lt_launch(hipStream_t s, const char *name, const LinTwoArgs &a)
{
    typedef LinTwoCfg<RB, MB> F;
    int st = PF_OK;
    const dim3 grid((unsigned)((a.M + F::MR - 1) / F::MR), a.osplit, a.groups);
    const bool even = a.r % 8 == 0;
    if constexpr (MB < 4)
        if (even && a.add && a.mask) {
            PF_LAUNCH(st, name, (linear_two_kernel<RB, MB, true, true, true>), grid, dim3(F::NT), s, a);
            return st;
        }
    if (even && a.mask) PF_LAUNCH(st, name, (linear_two_kernel<RB, MB, true, false, true>), grid, dim3(F::NT), s, a);
    else if (even && a.add) PF_LAUNCH(st, name, (linear_two_kernel<RB, MB, true, true, false>), grid, dim3(F::NT), s, a);
    else if (even) PF_LAUNCH(st, name, (linear_two_kernel<RB, MB, true, false, false>), grid, dim3(F::NT), s, a);
    else if (a.mask || RB > 4) return PF_ERR_UNSUPPORTED; // (backward and ranks above 128 take ranks in whole pieces)
    else if constexpr (RB <= 4) {
        if (a.add) PF_LAUNCH(st, name, (linear_two_kernel<RB, MB, false, true, false>), grid, dim3(F::NT), s, a);
        else PF_LAUNCH(st, name, (linear_two_kernel<RB, MB, false, false, false>), grid, dim3(F::NT), s, a);
    }
    return st;
}
template <int RB>
static int lt_rows(hipStream_t s, const char *name, const LinTwoArgs &a, int rows)
{
    if constexpr (RB > 4) {
        if constexpr (RB < 8)
            if (rows == 64) return lt_launch<RB, 2>(s, name, a);
        return rows == 32 ? lt_launch<RB, 1>(s, name, a) : PF_ERR_UNSUPPORTED;
    }
    if (rows == 128 && a.add && a.mask) rows = 64; // (both arrays' pieces beside the sums of 128 rows do not fit the registers)
    if constexpr (RB <= 4)
        return rows == 128  ? lt_launch<RB, 4>(s, name, a)
               : rows == 64 ? lt_launch<RB, 2>(s, name, a)
               : rows == 32 ? lt_launch<RB, 1>(s, name, a)
                            : PF_ERR_UNSUPPORTED;
}
int launch_linear_two(hipStream_t s, const char *name, const LinTwoArgs &a, int rows)
{
    if (!linear_two_supported(a.M, a.K, a.N, a.r) || a.osplit < 1 || a.osplit > (a.N + 127) / 128) return PF_ERR_UNSUPPORTED;
    switch (lt_blocks(a.r)) {
    case 1: return lt_rows<1>(s, name, a, rows);
    case 2: return lt_rows<2>(s, name, a, rows);
    case 4: return lt_rows<4>(s, name, a, rows);
    case 5: return lt_rows<5>(s, name, a, rows);
    case 6: return lt_rows<6>(s, name, a, rows);
    default: return lt_rows<8>(s, name, a, rows);
    }
}

} // namespace pf
