#include "pf_linear_two.h"

#include "pf_tile.h"

namespace pf {

// A workgroup of eight wavefronts takes 32 MB rows through both stages.  Both factors stream through LDS as they lie in memory (the
// first one's fragments come from transposing reads), two parts of about 32 KB in flight in registers beside two in LDS: what bounds
// the kernel is latency (a chunk of 40 KB takes 1500 clocks, of which its loads are 700 at the 58 bytes a clock that a compute unit takes
// in with 32 KB outstanding, its LDS traffic 830) and, for many rows, the factors read again by every workgroup.  2000 rows, 256 ->
// rank 64 -> 1024: 10.4 us on the tiled products (two or three launches), 6.6; 500 x 384 -> 96 -> 384: 9.2 -> 7.0; 8192 x 384 -> 96 ->
// 1536: 23.7 -> 17.5.  Rank 128 and widths in multiples of 256 have a kernel of their own (8192 x 512 -> 512: 9.6, here 12.7), above
// rank 128 the tiled products are faster (8192 x 768 -> 192 -> 768: 22.4 against 23.3, 1000 x 1024 -> 256 -> 1024 12.7 against 19), and
// backward they form dX beside the gradients (500 x 384 -> 96 -> 384: 10.7 against 13.0 with both stages here).
// WM x WN wavefronts over (ranks, rows), WK of them split the contraction of the first stage; the second takes 128 outputs at a time.
template <int RB, int MB>
struct LinTwoCfg {
    static constexpr int NT = 512, MR = 32 * MB, Kp = 32 * RB, KC = RB == 4 && MB == 4 ? 64 : 128;
    static constexpr int WM = RB, WN = 8 / RB < MB ? 8 / RB : MB, WK = 8 / (WM * WN), NB = MB / WN;
    static constexpr int VP = Kp + 8, XP = KC + 8;                                          // pitches (elements)
    static constexpr int VCH = KC * RB * 4 / NT, XCH = MR * KC / 8 / NT > 0 ? MR * KC / 8 / NT : 1; // pieces per thread
    static constexpr int VBYTES = KC * VP * 2, XBYTES = MR * XP * 2, BUF = VBYTES + XBYTES;
    static constexpr int SP = Kp + 4, SBYTES = WK > 1 ? WK * MR * SP * 4 : 0;                // sums of the first stage
    static constexpr int OC = 128, ON = MB < 2 ? 1 : 2, NB2 = MB / ON, WK2 = 8 / (4 * ON);
    static constexpr int AP = Kp + 8, ABYTES = OC * AP * 2, ACH = OC * RB * 4 / NT, ABUF = RB == 4 && MB == 4 ? 1 : 2;
    static constexpr int CP = OC + 4, CBYTES = WK2 * MR * CP * 4, OUT = MR * OC / 8 / NT;
    static_assert(KC / 16 % WK == 0 && 2 * RB % WK2 == 0, "whole steps");
    static constexpr int TP = Kp + 8, TBYTES = MR * TP * 2;
    static constexpr int S1 = 2 * BUF > SBYTES ? 2 * BUF : SBYTES, S2 = ABUF * ABYTES + CBYTES, BYTES = TBYTES + (S1 > S2 ? S1 : S2);
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

template <int RB, int MB>
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
    uint4 vr[2][F::VCH], xr[2][F::XCH];
    const int steps = (K + KC - 1) / KC;
    // A thread's pieces lie in one column of the factor and one of the input.  Ranks in whole pieces: nothing to put in place.
    const bool even = r % 8 == 0;
    const int vrow = tid / (RB * 4), vcol = tid % (RB * 4), xrow = tid / (KC / 8), xcol = tid % (KC / 8) * 8;
    constexpr int VSTEP = NT / (RB * 4), XSTEP = NT / (KC / 8);
    const bool vin = vcol * 8 < r;
    uint32_t xat[F::XCH];
#pragma unroll
    for (int u = 0; u < F::XCH; ++u) xat[u] = (uint32_t)min(m0 + xrow + XSTEP * u, M - 1) * (uint32_t)K + xcol;
    const auto load1 = [&](int q, uint4 (&v)[F::VCH], uint4 (&x)[F::XCH]) __attribute__((always_inline)) {
        const int k0 = q * KC;
        if (even && k0 + KC <= K) {
#pragma unroll
            for (int u = 0; u < F::VCH; ++u) v[u] = ldg16((const char *)(W1 + (i64)k0 * r) + 2u * (uint32_t)(vin ? (vrow + VSTEP * u) * r + vcol * 8 : 0));
#pragma unroll
            for (int u = 0; u < F::XCH; ++u) x[u] = ldg16((const char *)(a.in + k0) + 2u * xat[u]);
            return;
        }
#pragma unroll
        for (int u = 0; u < F::VCH; ++u) v[u] = LinPiece(k0 + vrow + VSTEP * u, vcol, K, r).load(W1, K * r);
#pragma unroll
        for (int u = 0; u < F::XCH; ++u) x[u] = ldg16((const char *)a.in + 2u * (xat[u] + (uint32_t)(min(k0 + xcol, K - 8) - xcol)));
    };
    const auto store1 = [&](int q, unsigned char *buf, const uint4 (&v)[F::VCH], const uint4 (&x)[F::XCH]) __attribute__((always_inline)) {
        const int k0 = q * KC;
        unsigned char *vb = buf + vrow * (F::VP * 2) + vcol * 16, *xb = buf + F::VBYTES + xrow * (F::XP * 2) + xcol * 2;
        if (even && k0 + KC <= K) { // (ranks past the last are sums that nobody reads)
#pragma unroll
            for (int u = 0; u < F::VCH; ++u) *(uint4 *)(vb + VSTEP * u * (F::VP * 2)) = v[u];
#pragma unroll
            for (int u = 0; u < F::XCH; ++u)
                if (MR >= XSTEP || xrow < MR) *(uint4 *)(xb + XSTEP * u * (F::XP * 2)) = x[u];
            return;
        }
#pragma unroll
        for (int u = 0; u < F::VCH; ++u) *(uint4 *)(vb + VSTEP * u * (F::VP * 2)) = LinPiece(k0 + vrow + VSTEP * u, vcol, K, r).fix(v[u], K * r);
        const bool in = k0 + xcol < K;
#pragma unroll
        for (int u = 0; u < F::XCH; ++u)
            if (MR >= XSTEP || xrow < MR) {
                const uint4 w = x[u];
                *(uint4 *)(xb + XSTEP * u * (F::XP * 2)) = make_uint4(in ? w.x : 0u, in ? w.y : 0u, in ? w.z : 0u, in ? w.w : 0u);
            }
    };
    load1(0, vr[0], xr[0]);
    if (steps > 1) load1(1, vr[1], xr[1]);
    const int wk = wave / (F::WM * F::WN), wm = wave / F::WN % F::WM, wn = wave % F::WN;
    f32x16_t acc[F::NB];
#pragma unroll
    for (int j = 0; j < F::NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    for (int q0 = 0; q0 < steps; q0 += 2) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int q = q0 + p;
            if (q < steps) {
                unsigned char *buf = base + p * F::BUF;
                store1(q, buf, vr[p], xr[p]);
                if (q + 2 < steps) load1(q + 2, vr[p], xr[p]);
                __syncthreads();
#pragma unroll
                for (int s = 0; s < KC / 16 / F::WK; ++s) {
                    const int st = wk * (KC / 16 / F::WK) + s;
                    if (q * KC + st * 16 >= K) break;
                    const bf16x8_t f = lds_frag_tr((const uint16_t *)buf, F::VP, st * 16, wm * 32, lane);
#pragma unroll
                    for (int j = 0; j < F::NB; ++j) {
                        const bf16x8_t b = *(const bf16x8_t *)(buf + F::VBYTES + ((wn * F::NB + j) * 32 + (lane & 31)) * (F::XP * 2) + (st * 16 + hi * 8) * 2);
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, b, acc[j], 0, 0, 0);
                    }
                }
            }
        }
    }

    // the sums -> LDS in bf16, zero past the last rank whatever the input holds
    if constexpr (F::WK == 1) {
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
    uint4 ar[2][F::ACH];
    const int parts = c_end - c_begin;
    const auto load2 = [&](int q, uint4 (&to)[F::ACH]) __attribute__((always_inline)) {
        const int o0 = (c_begin + q) * F::OC;
        if (even && o0 + F::OC <= N) {
#pragma unroll
            for (int u = 0; u < F::ACH; ++u) to[u] = ldg16((const char *)(W2 + (i64)o0 * r) + 2u * (uint32_t)(vin ? (vrow + VSTEP * u) * r + vcol * 8 : 0));
            return;
        }
#pragma unroll
        for (int u = 0; u < F::ACH; ++u) to[u] = LinPiece(o0 + vrow + VSTEP * u, vcol, N, r).load(W2, N * r);
    };
    load2(0, ar[0]);
    if (parts > 1) load2(1, ar[1]);
    uint4 add[F::OUT], bs;
    const int orow = tid / 16, ocol = tid % 16 * 8; // (and every 32nd row from there)
    const auto load_ep = [&](int o0) __attribute__((always_inline)) {
        const int o = min(o0 + ocol, N - 8);
        bs = bias ? ldg16((const char *)bias + 2u * (uint32_t)o) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < F::OUT; ++u) {
            const uint32_t at = (uint32_t)min(m0 + orow + 32 * u, M - 1) * (uint32_t)N + o;
            if (a.add) add[u] = ldg16((const char *)a.add + 2u * at);
        }
    };
    load_ep(c_begin * F::OC);
    __syncthreads();
    if (mid && blockIdx.y == 0) {
        const int per = (r + 7) / 8;
        for (int i = tid; i < MR * per; i += NT) {
            const int o = i % per, row = i / per;
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
    const int om = wave % 4, on = wave / 4 % F::ON, wk2 = wave / (4 * F::ON);
    float *cs = (float *)(base + F::ABUF * F::ABYTES);
    f32x16_t y[F::NB2];
#pragma unroll
    for (int j = 0; j < F::NB2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) y[j][v] = 0.f;
    for (int q0 = 0; q0 < parts; q0 += 2) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int q = q0 + p, o0 = (c_begin + q) * F::OC;
            if (q < parts) {
                uint16_t *as = (uint16_t *)(base + (F::ABUF == 2 ? p * F::ABYTES : 0));
                if (F::ABUF == 1) __syncthreads();
                if (even && o0 + F::OC <= N) { // (half a step past the last rank: zero)
#pragma unroll
                    for (int u = 0; u < F::ACH; ++u) {
                        const uint4 w = ar[p][u];
                        *(uint4 *)&as[(vrow + VSTEP * u) * F::AP + vcol * 8] = make_uint4(vin ? w.x : 0u, vin ? w.y : 0u, vin ? w.z : 0u, vin ? w.w : 0u);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < F::ACH; ++u)
                        *(uint4 *)&as[(vrow + VSTEP * u) * F::AP + vcol * 8] = LinPiece(o0 + vrow + VSTEP * u, vcol, N, r).fix(ar[p][u], N * r);
                }
                if (q + 2 < parts) load2(q + 2, ar[p]);
                __syncthreads();
#pragma unroll
                for (int s = 0; s < 2 * RB / F::WK2; ++s) {
                    const int st = wk2 * (2 * RB / F::WK2) + s;
                    if (st * 16 >= r) break;
                    const bf16x8_t f = *(const bf16x8_t *)&as[(om * 32 + (lane & 31)) * F::AP + st * 16 + hi * 8];
#pragma unroll
                    for (int j = 0; j < F::NB2; ++j) {
                        const bf16x8_t b = *(const bf16x8_t *)&ts[((on * F::NB2 + j) * 32 + (lane & 31)) * TP + st * 16 + hi * 8];
                        y[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, b, y[j], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int j = 0; j < F::NB2; ++j)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const f32x4_t w = {y[j][4 * k], y[j][4 * k + 1], y[j][4 * k + 2], y[j][4 * k + 3]};
                        *(f32x4_t *)&cs[(wk2 * MR + (on * F::NB2 + j) * 32 + (lane & 31)) * F::CP + om * 32 + 8 * k + 4 * hi] = w;
#pragma unroll
                        for (int e = 0; e < 4; ++e) y[j][4 * k + e] = 0.f;
                    }
                __syncthreads();
                if (o0 + ocol < N) {
                    float b[8];
                    piece_floats<bf16_t>(bs, b);
#pragma unroll
                    for (int u = 0; u < F::OUT; ++u) {
                        const int row = orow + 32 * u;
                        float v[8], f[8];
#pragma unroll
                        for (int e = 0; e < 8; e += 4) {
                            f32x4_t w = *(const f32x4_t *)&cs[row * F::CP + ocol + e];
                            if (F::WK2 == 2) w += *(const f32x4_t *)&cs[(MR + row) * F::CP + ocol + e];
#pragma unroll
                            for (int x = 0; x < 4; ++x) v[e + x] = w[x] + b[e + x];
                        }
                        if (a.add) {
                            piece_floats<bf16_t>(add[u], f);
#pragma unroll
                            for (int e = 0; e < 8; ++e) v[e] += f[e];
                        }
                        if (a.relu) {
#pragma unroll
                            for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f);
                        }
                        if (m0 + row < M) stg16((char *)out + 2u * ((uint32_t)(m0 + row) * (uint32_t)N + o0 + ocol), floats_piece<bf16_t>(v));
                    }
                }
                if (q + 1 < parts) load_ep(o0 + F::OC);
            }
        }
    }
}

static int lt_blocks(i64 r) { return r <= 32 ? 1 : r <= 64 ? 2 : 4; }

bool linear_two_supported(i64 M, i64 K, i64 N, i64 r)
{
    const i64 lim = 1LL << 30;
    return M >= 1 && K >= 8 && N >= 8 && K % 8 == 0 && N % 8 == 0 && r >= 8 && r <= 128 && M * K < lim && M * N < lim && K * r < lim && N * r < lim;
}

// Fitted to times of 108 shapes (1 to 16384 rows, 128 to 4096 wide, ranks 16 to 128) with every number of rows and share of the outputs, 10 %
// rms: a chunk of the first stage costs 0.21 us, 128 outputs 0.12 per 32 rows, and what a compute unit reads 17 and 31 ns per KB.
double plan_linear_two(i64 M, i64 K, i64 N, i64 r, int groups, int &rows, int &osplit)
{
    double best = 1e30;
    const int RB = lt_blocks(r), chunks = (int)((N + 127) / 128);
    for (int mb = 1; mb <= 4; mb *= 2) {
        const i64 tiles = (M + 32 * mb - 1) / (32 * mb);
        const double steps = (double)((K + (RB == 4 && mb == 4 ? 63 : 127)) / (RB == 4 && mb == 4 ? 64 : 128));
        for (int os = 1; os <= chunks && os <= 16; os *= 2) {
            const int per = (chunks + os - 1) / os;
            const i64 rounds = (tiles * os * groups + 255) / 256;
            const double full = tiles * os * groups < 256 ? tiles * os * groups / 256.0 : 1;
            const double kb1 = K * (r + 32.0 * mb) / 512, kb2 = per * 128.0 * (r + 32 * mb) / 512;
            const double t = 3.8 + rounds * (0.21 * steps + 0.116 * per * mb + 0.0172 * kb1 + 0.0312 * kb2 + 0.0026 * full * (kb1 + kb2) +
                                             (r % 8 ? 0.37 * (steps + per) : 0));
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
    PF_LAUNCH(st, name, (linear_two_kernel<RB, MB>), dim3((unsigned)((a.M + F::MR - 1) / F::MR), a.osplit, a.groups), dim3(F::NT), s, a);
    return st;
}
template <int RB>
static int lt_rows(hipStream_t s, const char *name, const LinTwoArgs &a, int rows)
{
    return rows == 128 ? lt_launch<RB, 4>(s, name, a) : rows == 64 ? lt_launch<RB, 2>(s, name, a) : rows == 32 ? lt_launch<RB, 1>(s, name, a) : PF_ERR_UNSUPPORTED;
}
int launch_linear_two(hipStream_t s, const char *name, const LinTwoArgs &a, int rows)
{
    if (!linear_two_supported(a.M, a.K, a.N, a.r) || a.osplit < 1 || a.osplit > (a.N + 127) / 128) return PF_ERR_UNSUPPORTED;
    return lt_blocks(a.r) == 1 ? lt_rows<1>(s, name, a, rows) : lt_blocks(a.r) == 2 ? lt_rows<2>(s, name, a, rows) : lt_rows<4>(s, name, a, rows);
}

} // namespace pf
