// Both data gradients of the factorized convolution in one launch: dT = (scale Vp)^T dZ, dX = sum over the taps of Uk^T dT, plus the
// gradient of a skip connection, masked by a ReLU input.
#include "pf_conv_px_dev.h"

namespace pf {

// A workgroup forms dT for the 32 PB pixels of its tile and for their halo (again for pixels that neighbouring tiles share: their share
// of the first stage is cheaper than a launch of its own and dT's way through memory), keeps it in LDS, pixel-major and with zeros
// outside the planes, and takes the taps as row offsets.  dZ passes in chunks, the 1 x 1 filters as they lie in memory (transposing
// reads), the thin ones re-ordered (PxPack), TPP taps of MC channels at a time.  128 images of 128 x 16 x 16, rank 32, 3 x 3: 14 us for
// what took two launches and a third of another (6.5 us for dT, most of 39 for dX with the filter gradients).  Float (one tap): 226 images of
// 64 x 14 x 14, rank 16, with the filter gradients 67.9 -> 44.6 us, 12 of 96 x 14 x 14, rank 24 26.7 -> 23.5.
template <typename T, int KK, int RB, int PB, int NT>
struct PxBwdCfg {
    typedef PxRows<T, PB, NT> R;
    static constexpr int V = PxEl<T>::V, ES = sizeof(T), F4 = ES == 4, WAVES = NT / 64, P = 32 * PB;
    static constexpr int HB = KK == 1 ? PB : (R::rows + 31) / 32;               // pixel blocks of the first stage
    static constexpr int WPX = HB < WAVES ? HB : WAVES, NB1 = (HB + WPX - 1) / WPX;
    static constexpr int WRB = WAVES / WPX < RB ? WAVES / WPX : RB, MB1 = (RB + WRB - 1) / WRB;
    static constexpr int VROWS = R::CH < 128 ? R::CH : 128;                     // rows of Vp in a part
    static constexpr int VPARTS = R::CH / VROWS, VPITCH = 32 * RB + V, RP = 32 * RB / V;          // (elements)
    static constexpr int VCH = VROWS * RP / NT, VBYTES = VROWS * VPITCH * ES;
    // second stage
    static constexpr int MC = (NT == 512 ? 128 : 64) * (PB == 1 ? 2 : 1);       // channels at a time
    static constexpr int OM = MC / 32, ON = WAVES / OM, NB = PB / ON;
    static constexpr int TPP = KK == 1 || RB == 4 || (RB == 2 && PB == 1) ? 1 : 3, PARTS = KK / TPP;
    static constexpr int PPR = TPP * RP, APITCH = PPR * 16 + 16, ABYTES = MC * APITCH, ACH = MC * PPR / NT;
    static constexpr int RING = PARTS == 1 ? 1 : NT == 512 ? (ACH > 4 ? 1 : 3) : 1;
    static constexpr int TP = (32 * RB + PxEl<T>::PC - 1) / PxEl<T>::PC, TBYTES = TP * R::panel, CP = P + 4, CBYTES = MC * CP * 4;
    static constexpr int ABUF = NT == 512 && !(PB == 1 && RB == 4) ? 2 : 1;
    static constexpr int s1 = R::bytes + VBYTES, s2 = TBYTES + (ABUF * ABYTES > CBYTES ? ABUF * ABYTES : CBYTES);
    static constexpr int BYTES = s1 > s2 ? s1 : s2;
    static_assert(OM * ON == WAVES && PB % ON == 0 && MC * PPR % NT == 0 && VROWS * RP % NT == 0, "whole rounds");
    static_assert(PARTS % RING == 0, "a part's registers are known at compile time");
    static_assert(BYTES <= (NT == 512 ? 160 : 80) * 1024, "LDS of a compute unit, or of half of one");
};

// The fragment of 2 V output channels (from `k0` on) x 32 ranks (from m0 on) out of rows of ranks.
template <typename T>
__device__ __forceinline__ uint4 px_frag_v(const T *vs, int pitch, int k0, int m0, int lane)
{
    if constexpr (sizeof(T) == 2) {
        union {
            bf16x8_t v;
            uint4 u;
        } f;
        f.v = lds_frag_tr(vs, pitch, k0, m0, lane);
        return f.u;
    } else {
        const T *p = vs + (k0 + 4 * (lane >> 5)) * pitch + m0 + (lane & 31);
        return make_uint4(__float_as_uint(p[0]), __float_as_uint(p[pitch]), __float_as_uint(p[2 * pitch]), __float_as_uint(p[3 * pitch]));
    }
}

template <typename T, int KK, int RB, int PB, int NT>
__global__ __launch_bounds__(NT, 2) void conv_px_bwd_kernel(PxBwdArgs<T> a)
{
    typedef PxBwdCfg<T, KK, RB, PB, NT> F;
    typedef typename F::R R;
    constexpr int V = F::V, RP = F::RP;
    __shared__ __attribute__((aligned(16))) unsigned char smem[F::BYTES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hi = lane >> 5;
    const PxPlaneOf<T> &g = a.g;

    // ------------------------------------------------ dT of the tile and its halo
    unsigned char *zs = smem;
    T *vs = (T *)(smem + R::bytes);
    uint4 vr[F::VCH], zr[R::BL][V];
    float vscale[F::VCH];
    const int total_v = a.Cout * a.r;
    const auto load_v = [&](int o0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < F::VCH; ++u) {
            const int i = tid + NT * u, row = i / RP, col = i % RP;
            vr[u] = px_row_piece(a.Vp, (o0 + row) * a.r + col * V, o0 + row < a.Cout ? min(V, a.r - col * V) : 0, total_v);
            vscale[u] = a.scale ? a.scale[min(o0 + row, a.Cout - 1)] : 1.f;
        }
    };
    load_v(0);
    const PxTile t = px_tile(g, blockIdx.x * F::P, F::P);
    PxBlocks<T, PB, NT> blk;
    blk.init(g, t, 1, a.Cout);
    blk.load(a.dZ, g, a.Cout, 0, zr);
    const int w1 = wave % F::WPX, r1 = wave / F::WPX; // pixel blocks and rank blocks of the first stage (r1 >= WRB: none)
    const int npx = t.pb - t.pa;
    int slot1[F::NB1];
#pragma unroll
    for (int j = 0; j < F::NB1; ++j) slot1[j] = px_slot(g, min(t.pa + (w1 + j * F::WPX) * 32 + (lane & 31), t.pb - 1)) - t.base;
    PxSum<T, F::NB1> sum1[F::MB1];
#pragma unroll
    for (int i = 0; i < F::MB1; ++i) sum1[i].clear();
    for (int c0 = 0; c0 < a.Cout; c0 += R::CH) {
        if (c0) __syncthreads();
        blk.store(zs, zr);
        blk.load(a.dZ, g, a.Cout, c0 + R::CH, zr); // (zeros past the last channel)
#pragma unroll
        for (int part = 0; part < F::VPARTS; ++part) {
            const int o0 = c0 + part * F::VROWS;
            if (o0 < a.Cout) {
                if (part) __syncthreads();
#pragma unroll
                for (int u = 0; u < F::VCH; ++u) {
                    const int i = tid + NT * u, row = i / RP, col = i % RP;
                    uint4 v = vr[u];
                    if (a.scale) {
                        float f[V];
                        px_unpack<T>(v, f);
#pragma unroll
                        for (int e = 0; e < V; ++e) f[e] *= vscale[u];
                        v = px_piece<T>(f);
                    }
                    *(uint4 *)(vs + row * F::VPITCH + col * V) = v;
                }
                if (o0 + F::VROWS < a.Cout) load_v(o0 + F::VROWS);
                __syncthreads();
                if (r1 < F::WRB) {
#pragma unroll
                    for (int st = 0; st < F::VROWS / (2 * V); ++st) {
                        const int cs = part * (F::VROWS / (2 * V)) + st;
                        if (o0 + 2 * V * st < a.Cout) {
                            uint4 f[F::MB1];
#pragma unroll
                            for (int i = 0; i < F::MB1; ++i) f[i] = px_frag_v(vs, F::VPITCH, st * 2 * V, (r1 * F::MB1 + i) * 32, lane);
#pragma unroll
                            for (int j = 0; j < F::NB1; ++j) {
                                const uint4 b = *(const uint4 *)(zs + (cs >> 2) * R::panel + (px_at(slot1[j], hi) ^ ((cs & 3) << 5)));
#pragma unroll
                                for (int i = 0; i < F::MB1; ++i) px_mma<T>(sum1[i].at(j), f[i], b);
                            }
                        }
                        if (st % 2 == 1) {
#pragma unroll
                            for (int i = 0; i < F::MB1; ++i) sum1[i].flush();
                        }
                    }
                }
            }
        }
    }

    // ------------------------------------------------ dT -> LDS, memory
    unsigned char *ts = smem, *as = smem + F::TBYTES;
    constexpr int Kp = 32 * RB;
    uint4 ar[F::RING][F::ACH];
    // filters of part q: channels c0 .., taps (q % PARTS) TPP ..
    const auto load_a = [&](int q, uint4 (&to)[F::ACH]) __attribute__((always_inline)) {
        const int c0 = q / F::PARTS * F::MC, tap0 = q % F::PARTS * F::TPP;
#pragma unroll
        for (int u = 0; u < F::ACH; ++u) {
            const int i = tid + NT * u, row = i / F::PPR, col = i - row * F::PPR, tap = col / RP, k = col - tap * RP;
            const int c = min(c0 + row, a.C - 1);
            to[u] = px_load(a.Wb, ((tap0 + tap) * a.C + c) * Kp + k * V);
        }
    };
#pragma unroll
    for (int i = 0; i < F::RING; ++i) load_a(i, ar[i]);
    __syncthreads();
    if (KK > 1) {
        for (int i = tid; i < F::TBYTES / 16; i += NT) ((uint4 *)ts)[i] = px_zero();
        __syncthreads();
    }
    if (r1 < F::WRB) {
#pragma unroll
        for (int j = 0; j < F::NB1; ++j)
            if ((w1 + j * F::WPX) * 32 + (lane & 31) < npx) {
#pragma unroll
                for (int i = 0; i < F::MB1; ++i) {
                    const int rb = r1 * F::MB1 + i;
#pragma unroll
                    for (int q = 0; q < 4; ++q) { // ranks 32 rb + 8 q + 4 hi ..
                        // (past the last rank: zero, whatever dZ holds)
                        const int left = a.r - (32 * rb + 8 * q + 4 * hi);
                        f32x4_t w;
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[e] = left > e ? sum1[i].acc[j][4 * q + e] : 0.f;
                        if (rb < RB) {
                            if constexpr (F::F4)
                                *(f32x4_t *)(ts + rb * R::panel + px_at(slot1[j], 2 * q + hi)) = w;
                            else
                                *(uint2 *)(ts + (rb >> 1) * R::panel + px_at(slot1[j], (rb & 1) * 4 + q) + 8 * hi) =
                                    make_uint2(pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]));
                        }
                    }
                }
            }
    }
    constexpr int PG = F::P / V;
    const PxOut out = px_out(g, t);
    const int rest = px_out_rest(g, out);
    PxPieceOut po;
    po.init(g, t, out, tid % PG);
    const int slot_out = po.live ? px_slot(g, po.n, po.q) - t.base : 0; // (a row of the plane may end within the group: below)
    const int on = wave % F::ON, om = wave / F::ON;
    int baddr[KK][F::NB];
#pragma unroll
    for (int nb = 0; nb < F::NB; ++nb) {
        const int p = min(t.p0 + (on * F::NB + nb) * 32 + (lane & 31), t.p1 - 1), s = px_slot(g, p) - t.base;
#pragma unroll
        for (int tap = 0; tap < KK; ++tap) baddr[tap][nb] = px_at(s + (KK == 9 ? (tap / 3 - 1) * g.Wp + tap % 3 - 1 : 0), hi);
    }
    __syncthreads();
    if (a.dT) {
        const int rv = px_ranks<T>(a.r);
        for (int q = tid; q < rv / V * PG; q += NT) {
            const int oc = q / PG;
            if (po.live) {
                uint4 v[V];
                const int y = px_div(po.q, g.W, g.mW);
                int x = po.q - y * g.W, s = slot_out;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    v[e] = *(const uint4 *)(ts + (oc >> 3) * R::panel + px_at(s, oc & 7));
                    ++s;
                    if (++x == g.W) x = 0, s += g.h;
                }
#pragma unroll
                for (int e = 0; e < V; ++e) px_save(a.dT, (po.n * rv + oc * V + e) * g.HW + po.q, px_turn(v, e));
            }
        }
        for (int q = tid; q < rv * rest; q += NT) {
            int n, px;
            const int row = q / rest;
            px_out_pixel(g, out, q - row * rest, n, px);
            a.dT[(n * rv + row) * g.HW + px] =
                *(const T *)(ts + row / PxEl<T>::PC * R::panel + px_at(px_slot(g, n, px) - t.base, row / V & 7) + row % V * F::ES);
        }
    }

    // ------------------------------------------------ dX
    float *cs = (float *)(smem + F::TBYTES);
    constexpr int CP = F::CP, OUT = F::MC * PG / NT;
    const bool whole = g.HW % V == 0;
    const int parts = (a.C + F::MC - 1) / F::MC * F::PARTS;
    for (int q0 = 0; q0 < parts; q0 += F::PARTS) {
        const int c0 = q0 / F::PARTS * F::MC;
        uint4 add[OUT], mask[OUT];
        PxSum<T, F::NB> sum;
        sum.clear();
#pragma unroll
        for (int k = 0; k < F::PARTS; ++k) {
            unsigned char *ab = as + (F::ABUF == 2 ? (k & 1) * F::ABYTES : 0);
            if (k == 0 || F::ABUF == 1) __syncthreads(); // (the sums of the channels before, or this buffer, may still be read)
#pragma unroll
            for (int u = 0; u < F::ACH; ++u) {
                const int i = tid + NT * u, row = i / F::PPR, col = i - row * F::PPR;
                *(uint4 *)(ab + row * F::APITCH + col * 16) = ar[k % F::RING][u];
            }
            if (q0 + k + F::RING < parts) load_a(q0 + k + F::RING, ar[k % F::RING]);
            __syncthreads();
            if (k == F::PARTS - 1) {
#pragma unroll
                for (int u = 0; u < OUT; ++u) {
                    const int c = min(c0 + (tid + NT * u) / PG, a.C - 1);
                    add[u] = px_fetch(g, po, a.C, c, a.ep.add);
                    mask[u] = px_fetch(g, po, a.C, c, a.ep.mask);
                }
            }
#pragma unroll
            for (int tt = 0; tt < F::TPP; ++tt)
#pragma unroll
                for (int st = 0; st < RP / 2; ++st) {
                    const uint4 f = *(const uint4 *)(ab + (om * 32 + (lane & 31)) * F::APITCH + (tt * RP + st * 2 + hi) * 16);
#pragma unroll
                    for (int j = 0; j < F::NB; ++j)
                        px_mma<T>(sum.at(j), f, *(const uint4 *)(ts + (st >> 2) * R::panel + (baddr[k * F::TPP + tt][j] ^ ((st & 3) << 5))));
                    if (st % 4 == 3) sum.flush();
                }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < F::NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                cs[(om * 32 + (v >> 2) * 8 + 4 * hi + (v & 3)) * CP + (on * F::NB + j) * 32 + (lane & 31)] = sum.acc[j][v];
        __syncthreads();
        if (po.live) {
#pragma unroll
            for (int u = 0; u < OUT; ++u) {
                const int row = (tid + NT * u) / PG, c = c0 + row;
                if (c < a.C) {
                    float v[V];
                    px_read<V>(cs + row * CP + po.col, whole, v);
                    px_put(g, po, a.C, c, a.dX, a.ep, v, add[u], mask[u]);
                }
            }
        }
        if (rest) px_put_rest<T, NT>(g, t, out, rest, cs, CP, F::MC, a.C, c0, a.dX, a.ep);
    }
}

template <typename T, int KK, int RB, int NT>
static int px_bwd_p(hipStream_t s, const PxBwdArgs<T> &a, int P)
{
    int st = PF_OK;
    const int npx = a.g.N * a.g.HW;
    const dim3 grid((npx + P - 1) / P);
    if (P == 128) PF_LAUNCH(st, "conv_bwd_px", (conv_px_bwd_kernel<T, KK, RB, 4, NT>), grid, dim3(NT), s, a);
    if (P == 64) PF_LAUNCH(st, "conv_bwd_px", (conv_px_bwd_kernel<T, KK, RB, 2, NT>), grid, dim3(NT), s, a);
    if (P == 32) PF_LAUNCH(st, "conv_bwd_px", (conv_px_bwd_kernel<T, KK, RB, 1, NT>), grid, dim3(NT), s, a);
    return st;
}
template <typename T, int KK, int RB>
static int px_bwd_t(hipStream_t s, const PxBwdArgs<T> &a, int P, int threads)
{
    if constexpr (sizeof(T) == 2 && RB <= 2) {
        if (threads == 256) return px_bwd_p<T, KK, RB, 256>(s, a, P);
    }
    return threads == 512 ? px_bwd_p<T, KK, RB, 512>(s, a, P) : PF_ERR_UNSUPPORTED;
}
template <int KK>
static int px_bwd_r(hipStream_t s, const PxBwdArgs<uint16_t> &a, int P, int threads)
{
    return a.r <= 32 ? px_bwd_t<uint16_t, KK, 1>(s, a, P, threads) : a.r <= 64 ? px_bwd_t<uint16_t, KK, 2>(s, a, P, threads)
                                                                                : px_bwd_t<uint16_t, KK, 4>(s, a, P, threads);
}
template <typename T>
int launch_px_bwd(hipStream_t s, const PxBwdArgs<T> &a, int k, int P, int threads)
{
    if ((P != 128 && P != 64 && P != 32) || !px_bwd_takes<T>(k, a.r)) return PF_ERR_UNSUPPORTED;
    if constexpr (sizeof(T) == 4)
        return px_bwd_t<T, 1, 1>(s, a, P, threads);
    else
        return k == 3 ? px_bwd_r<9>(s, a, P, threads) : px_bwd_r<1>(s, a, P, threads);
}
template int launch_px_bwd(hipStream_t, const PxBwdArgs<uint16_t> &, int, int, int);
template int launch_px_bwd(hipStream_t, const PxBwdArgs<float> &, int, int, int);

} // namespace pf
