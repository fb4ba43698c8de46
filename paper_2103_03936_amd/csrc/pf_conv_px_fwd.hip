// The whole factorized convolution forward in one launch: T = Uk * X over the taps, Y = act(scale (Vp T) + shift + residual).
#include "pf_chain_pack.h"
#include "pf_conv_px_dev.h"

namespace pf {

// A workgroup takes 32 PB pixels through both stages.  X passes through LDS in chunks (pixel-major, halo included), the
// thin filters in parts of 2 V STEPS channels with all their taps, as they lie in memory: channel and tap are fast there, so nine
// 16-byte pieces hold the nine taps of V channels, and a wavefront picks the fragment of a tap out of them (four v_perm in bf16).
// T stays in LDS, pixel-major again, and the 1 x 1 filters pass 64 output channels at a time.
// What bounds it: a compute unit's loads (a wavefront's 16 bytes per lane every 25 to 30 clocks: 128 x 128 channels of 16 x 16 planes,
// rank 32, 110 KB for a tile of 128 pixels, 4500 of 23000 clocks), LDS reads (a fragment of X per product at rank 32: 1700 clocks a part
// whose products take 1150) and, for one tile per compute unit, the chain of start, loads, products, T and output.  128 images of
// 128 x 16 x 16, rank 32, 3 x 3, with residual input and ReLU: 26.8 us on the tiled products (two launches), 12.3; 16 images of
// 64 x 16 x 16, rank 16: 18.6 -> 7.0; 256 x 192 x 32 x 32, rank 48: 310 -> 146.  Workgroups of 512 threads keep two parts of the filters
// in flight and have twice the channels per chunk; of 256 threads, two per compute unit, they cover each other's start and output: the
// faster ones where the channels are few.
// Float takes four products per step of the matrix unit, at a sixteenth of the rate, which bounds it from rank 33 on: 168 images of
// 144 x 11 x 11, rank 46 104.8 -> 70.2 us; 168 of 128 x 6 x 6, rank 32 29.2 -> 16.0; 88 of 64 x 13 x 10, rank 16, one tap 17.9 -> 10.2.
// With stride (SD) a tile's pixels lie apart, so that 32 of them fill 256 rows, and of one tap the rows that nobody sees are not loaded:
// 126 images of 240 x 16 x 16, rank 27, stride 2, bf16 34.3 -> 10.9; 128 of 128 x 16 x 16, rank 64, float 19 us less of
// 123 for both directions; the tiled products take two launches or three and a gathering load.
// WM x WN wavefronts over (rank, pixels), WK of them share a block and split the channel steps.
template <typename T, int KK, int RB, int PB, int NT, bool SD>
struct PxFwdCfg {
    typedef PxRows<T, PB, NT, SD> R;
    static constexpr int V = PxEl<T>::V, ES = sizeof(T), WAVES = NT / 64;
    static constexpr int WM = RB, WN = PB == 1 || (RB == 4 && WAVES == 4) ? 1 : 2, WK4 = (WAVES == 4 && WN == 2 ? 2 : 4) / RB, WK = WK4 > 0 ? WK4 : 1;
    static constexpr int NB = PB / WN;
    static constexpr int STEPS = KK == 1 ? (NT == 512 ? 8 : 4) : 4 / RB, PW = 2 * V * STEPS; // steps in a part of the filters, its channels
    static constexpr int P = 32 * PB;
    static constexpr int PPR = STEPS * 2 * KK;                                     // 16-byte pieces in a row of a part
    static constexpr int WPITCH = PPR * 16 + 16;                                   // odd number of pieces
    static constexpr int PIECES = 32 * RB * PPR, WCH = (PIECES + NT - 1) / NT;     // pieces per thread
    static constexpr int PARTS = R::CH / PW;                                       // of a chunk
    static constexpr int RING = NT == 512 && PARTS % 2 == 0 ? 2 : 1, XRING = KK == 1 ? 2 : 1; // parts, chunks in flight
    static constexpr int WBUF = NT == 512 ? 2 : 1, WBYTES = 32 * RB * WPITCH;
    // second stage
    static constexpr int OC = px_outputs(RB, P, NT);
    static constexpr int OM = OC / 32, ON = WAVES / OM, ONB = PB / ON; // wavefronts over (channels, pixels)
    static constexpr int RP = 32 * RB / V, TP = (32 * RB + PxEl<T>::PC - 1) / PxEl<T>::PC; // pieces of all ranks, panels
    static constexpr int CP = P + 4;                                   // pitch of float tiles
    static constexpr int TR = 32 * RB;
    static constexpr int TBYTES = TP * P * 128, APITCH = TR * ES + 16, ABYTES = OC * APITCH, CBYTES = OC * CP * 4;
    static constexpr int ACH = OC * RP / NT;
    static constexpr int TS = NT == 512 || RB < 4 || PB < 4 ? TR : 64; // ranks at a time on their way from sums to T
    static constexpr int s1 = R::bytes + WBUF * WBYTES, s2 = TBYTES + WK * TS * CP * 4, s3 = TBYTES + ABYTES + CBYTES;
    static constexpr int BYTES = s1 > s2 ? (s1 > s3 ? s1 : s3) : (s2 > s3 ? s2 : s3);
    static_assert(OM * ON == WAVES && PB % ON == 0 && WM * WN * WK <= WAVES, "wavefronts");
    static_assert(OC * RP % NT == 0 && STEPS % WK == 0 && PARTS >= 1, "whole rounds");
    static_assert(BYTES <= (NT == 512 ? 160 : 80) * 1024, "LDS of a compute unit, or of half of one");
};

// element i of what nine (or one) pieces hold
template <typename T, int KK>
__device__ __forceinline__ uint4 px_tap(const uint4 (&raw)[KK], int tap)
{
    const auto word = [&](int k) { return px_word(raw[k >> 2], k & 3); };
    if constexpr (KK == 1) {
        return raw[0];
    } else if constexpr (sizeof(T) == 4) { // channels 0 .. 3 of the tap
        return make_uint4(word(tap), word(KK + tap), word(2 * KK + tap), word(3 * KK + tap));
    } else {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { // channels 2 j and 2 j + 1
            const int e0 = 2 * j * KK + tap, e1 = e0 + KK;
            w[j] = __builtin_amdgcn_perm(word(e1 >> 1), word(e0 >> 1), (e0 & 1 ? 0x0302u : 0x0100u) | (e1 & 1 ? 0x07060000u : 0x05040000u));
        }
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
}

template <typename T, int KK, int RB, int PB, int NT, bool SD>
__global__ __launch_bounds__(NT, 2) void conv_px_fwd_kernel(PxFwdArgs<T> a)
{
    typedef PxFwdCfg<T, KK, RB, PB, NT, SD> F;
    typedef typename F::R R;
    constexpr int NB = F::NB, V = F::V;
    __shared__ __attribute__((aligned(16))) unsigned char smem[F::BYTES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wk = wave / (F::WM * F::WN), wm = wave / F::WN % F::WM, wn = wave % F::WN; // (wk == WK: none)
    const PxPlaneOf<T> &gx = a.g, &g = SD ? a.o : a.g;
    const int stride = SD ? a.stride : 1;
    unsigned char *xs = smem, *ws = smem + R::bytes;
    const int tiles = (g.N * g.HW + F::P - 1) / F::P;
    if ((int)blockIdx.x >= tiles) {
        if (a.pack.to) {
            px_pack<T, NT>(a.pack, blockIdx.x - tiles);
            return;
        }
        const int i = (blockIdx.x - tiles) * NT + tid;
        if (i < a.chain1.n)
            pack_w1_item(a.chain1, i);
        else if (i - a.chain1.n < a.chain2.n)
            pack_w2_item(a.chain2, i - a.chain1.n);
        return;
    }

    // ------------------------------------------------ stage 1
    uint4 xr[F::XRING][R::BL][V], wr[F::RING][F::WCH];
    const int rowlen = a.C * KK; // elements of a filter
    const auto load_w = [&](int c0, uint4 (&to)[F::WCH]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < F::WCH; ++u) {
            const int i = tid + NT * u, row = i / F::PPR, col = i - row * F::PPR;
            const bool in = i < F::PIECES && row < a.r && col * V < (a.C - c0) * KK;
            to[u] = px_zero();
            if (in) to[u] = px_load(a.Uk, row * rowlen + c0 * KK + col * V);
        }
    };
#pragma unroll
    for (int i = 0; i < F::RING; ++i) load_w(F::PW * i, wr[i]);
    const PxTile t = px_tile(gx, g, stride, blockIdx.x * F::P, F::P);
    PxBlocks<T, PB, NT, SD> blk;
    blk.init(gx, t, stride, a.C);
#pragma unroll
    for (int i = 0; i < F::XRING; ++i) blk.load(a.X, gx, a.C, i * R::CH, xr[i]);
    int baddr[KK][NB]; // this lane's pixel of every block through every tap, piece lane / 32
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int p = min(t.p0 + (wn * NB + nb) * 32 + (lane & 31), t.p1 - 1), s = px_slot(gx, g, stride, p) - t.base;
#pragma unroll
        for (int tap = 0; tap < KK; ++tap)
            baddr[tap][nb] = px_at(s + (KK == 9 ? (tap / 3 - 1) * gx.Wp + tap % 3 - 1 : 0), lane >> 5);
    }
    PxSum<T, NB> sum;
    sum.clear();
    if (KK > 1) // (the slots that stand for what lies outside the planes)
        for (int i = tid; i < R::bytes / 16; i += NT) ((uint4 *)xs)[i] = px_zero();
    // (a chunk's and a part's registers are known at compile time)
    constexpr int U = F::XRING > 1 || F::PARTS % F::RING ? 2 : 1, PW = F::PW;
    static_assert(U * F::PARTS % F::RING == 0 && U % F::XRING == 0, "");
    for (int cc = 0; cc < a.C; cc += R::CH * U) {
#pragma unroll
        for (int k = 0; k < U * F::PARTS; ++k) {
            const int ck = k / F::PARTS, part = k % F::PARTS, c0 = cc + ck * R::CH, c1 = c0 + part * PW, c2 = c1 + F::RING * PW;
            if (c1 < a.C) {
                if (part == 0) {
                    __syncthreads();
                    blk.store(xs, xr[ck % F::XRING]);
                    if (c0 + F::XRING * R::CH < a.C) blk.load(a.X, gx, a.C, c0 + F::XRING * R::CH, xr[ck % F::XRING]);
                }
                unsigned char *wb = ws + (F::WBUF == 2 ? (c1 / PW & 1) * F::WBYTES : 0);
                if (F::WBUF == 1 && part) __syncthreads();
#pragma unroll
                for (int u = 0; u < F::WCH; ++u) {
                    const int i = tid + NT * u, row = i / F::PPR, col = i - row * F::PPR;
                    if (F::PIECES % NT == 0 || i < F::PIECES) *(uint4 *)(wb + row * F::WPITCH + col * 16) = wr[k % F::RING][u];
                }
                if (c2 < a.C) load_w(c2, wr[k % F::RING]);
                __syncthreads();
                if (wk < F::WK) {
#pragma unroll
                    for (int q = 0; q < F::STEPS / F::WK; ++q) {
                        const int st = wk * (F::STEPS / F::WK) + q, cs = part * F::STEPS + st; // step of the part, of the chunk
                        {
                            uint4 raw[KK];
#pragma unroll
                            for (int j = 0; j < KK; ++j)
                                raw[j] = *(const uint4 *)(wb + (wm * 32 + (lane & 31)) * F::WPITCH + ((st * 2 + (lane >> 5)) * KK + j) * 16);
                            const unsigned char *xp = xs + (cs >> 2) * R::panel;
#pragma unroll
                            for (int tap = 0; tap < KK; ++tap) {
                                const uint4 f = px_tap<T, KK>(raw, tap);
#pragma unroll
                                for (int j = 0; j < NB; ++j)
                                    px_mma<T>(sum.at(j), f, *(const uint4 *)(xp + (baddr[tap][j] ^ ((cs & 3) << 5))));
                                if (KK == 9 && tap % 3 == 2) sum.flush();
                            }
                        }
                    }
                    if (KK == 1) sum.flush();
                }
                if (part == F::PARTS - 1) sum.fold();
            }
        }
    }
    sum.total();
    __syncthreads();

    // ------------------------------------------------ T: sums -> memory and, pixel-major, LDS
    unsigned char *ts = smem, *as = smem + F::TBYTES;
    float *cs = (float *)(smem + F::TBYTES);
    constexpr int CP = F::CP, PG = F::P / V, RP = F::RP;
    const PxOut out = px_out(g, t);
    const int rest = px_out_rest(g, out);
    PxPieceOut po;
    po.init(g, t, out, tid % PG);
    const int hi = 4 * (lane >> 5);
    // what the second stage reads first: its filters, the residual input, scale and shift of the thread's output pieces
    constexpr int OUT = F::OC * PG / NT;
    const int total_v = a.Cout * a.r;
    uint4 ar[F::ACH], add[OUT];
    float sc[OUT], sh[OUT];
    const auto load_a = [&](int o0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < F::ACH; ++u) {
            const int i = tid + NT * u, row = i / RP, col = i % RP;
            ar[u] = px_row_piece(a.Vp, (o0 + row) * a.r + col * V, o0 + row < a.Cout ? min(V, a.r - col * V) : 0, total_v);
        }
    };
    const auto load_ep = [&](int o0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < OUT; ++u) {
            const int ch = min(o0 + (tid + NT * u) / PG, a.Cout - 1);
            add[u] = px_fetch(g, po, a.Cout, ch, a.ep.add);
            sc[u] = a.ep.scale ? a.ep.scale[ch] : 1.f;
            sh[u] = a.ep.shift ? a.ep.shift[ch] : 0.f;
        }
    };
    load_a(0);
    load_ep(0);
#pragma unroll
    for (int r0 = 0; r0 < F::TR; r0 += F::TS) {
        if (r0 > 0) __syncthreads();
        if (wk < F::WK && (F::TS == F::TR || (wm * 32 >= r0 && wm * 32 < r0 + F::TS))) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    cs[(wk * F::TS + wm * 32 - r0 + (v >> 2) * 8 + hi + (v & 3)) * CP + (wn * NB + j) * 32 + (lane & 31)] = sum.acc[j][v];
        }
        __syncthreads();
        for (int q = tid; q < F::TS / V * F::P; q += NT) {
            const int px = q % F::P, oc = q / F::P, rp = r0 / V + oc;
            float v[V];
#pragma unroll
            for (int e = 0; e < V; ++e) {
                v[e] = cs[(oc * V + e) * CP + px];
#pragma unroll
                for (int w = 1; w < F::WK; ++w) v[e] += cs[(w * F::TS + oc * V + e) * CP + px];
                if (r0 + oc * V + e >= a.r) v[e] = 0.f; // (whatever X holds)
            }
            *(uint4 *)(ts + rp / 8 * F::P * 128 + px_at(px, rp & 7)) = px_piece<T>(v);
        }
    }
    __syncthreads();
    if (a.mid) { // V ranks of V pixels per thread
        for (int q = tid; q < RP * PG; q += NT) {
            const int oc = q / PG;
            if (po.live && oc * V < a.r) {
                uint4 v[V];
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] = *(const uint4 *)(ts + (oc >> 3) * F::P * 128 + px_at(po.col + e, oc & 7));
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (oc * V + e < a.r) px_save(a.mid, (po.n * a.r + oc * V + e) * g.HW + po.q, px_turn(v, e));
            }
        }
        for (int q = tid; q < a.r * rest; q += NT) {
            int n, px;
            const int row = q / rest;
            px_out_pixel(g, out, q - row * rest, n, px);
            a.mid[(n * a.r + row) * g.HW + px] =
                *(const T *)(ts + row / PxEl<T>::PC * F::P * 128 + px_at(n * g.HW + px - t.p0, row / V & 7) + row % V * (int)sizeof(T));
        }
    }

    // ------------------------------------------------ stage 2
    cs = (float *)(smem + F::TBYTES + F::ABYTES);
    const bool whole = g.HW % V == 0; // groups start at whole pieces
    const int om = wave / F::ON, on = wave % F::ON;
    for (int o0 = 0; o0 < a.Cout; o0 += F::OC) {
#pragma unroll
        for (int u = 0; u < F::ACH; ++u) {
            const int i = tid + NT * u, row = i / RP, col = i % RP;
            *(uint4 *)(as + row * F::APITCH + col * 16) = ar[u];
        }
        __syncthreads();
        if (o0 + F::OC < a.Cout) load_a(o0 + F::OC);
        PxSum<T, F::ONB> y;
        y.clear();
#pragma unroll
        for (int st = 0; st < RP / 2; ++st) {
            const uint4 f = *(const uint4 *)(as + (om * 32 + (lane & 31)) * F::APITCH + (st * 2 + (lane >> 5)) * 16);
#pragma unroll
            for (int j = 0; j < F::ONB; ++j) {
                const int px = (on * F::ONB + j) * 32 + (lane & 31);
                px_mma<T>(y.at(j), f, *(const uint4 *)(ts + st / 4 * F::P * 128 + px_at(px, (st & 3) * 2 + (lane >> 5))));
            }
            if (st % 4 == 3) y.flush();
        }
#pragma unroll
        for (int j = 0; j < F::ONB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                cs[(om * 32 + (v >> 2) * 8 + hi + (v & 3)) * CP + (on * F::ONB + j) * 32 + (lane & 31)] = y.acc[j][v];
        __syncthreads();
        if (po.live) {
#pragma unroll
            for (int u = 0; u < OUT; ++u) {
                const int row = (tid + NT * u) / PG, ch = o0 + row;
                if (ch < a.Cout) {
                    float v[V];
                    px_read<V>(cs + row * CP + po.col, whole, v);
#pragma unroll
                    for (int e = 0; e < V; ++e) v[e] = v[e] * sc[u] + sh[u];
                    px_put(g, po, a.Cout, ch, a.Y, a.ep, v, add[u], px_zero());
                }
            }
        }
        if (rest) px_put_rest<T, NT>(g, t, out, rest, cs, CP, F::OC, a.Cout, o0, a.Y, a.ep);
        if (o0 + F::OC < a.Cout) load_ep(o0 + F::OC);
    }
}

template <typename T>
static dim3 px_fwd_grid(const PxFwdArgs<T> &a, int P, int NT)
{
    return dim3((a.o.N * a.o.HW + P - 1) / P + (a.pack.to ? px_pack_blocks(a.pack, NT) : (a.chain1.n + a.chain2.n + NT - 1) / NT));
}
template <typename T, int KK, int RB>
static int px_fwd_strided(hipStream_t s, const PxFwdArgs<T> &a, int P)
{
    int st = P == 32 || (KK == 1 && P == 64) ? PF_OK : PF_ERR_UNSUPPORTED;
    const dim3 grid = px_fwd_grid(a, P, 512), nt(512);
    if constexpr (KK == 1) {
        if (P == 64) PF_LAUNCH(st, "conv_fwd_px_s", (conv_px_fwd_kernel<T, KK, RB, 2, 512, true>), grid, nt, s, a);
    }
    if (P == 32) PF_LAUNCH(st, "conv_fwd_px_s", (conv_px_fwd_kernel<T, KK, RB, 1, 512, true>), grid, nt, s, a);
    return st;
}
template <typename T, int KK, int RB, int NT>
static int px_fwd_p(hipStream_t s, const PxFwdArgs<T> &a, int P)
{
    int st = PF_OK;
    if (a.stride > 1) {
        if constexpr (NT == 512) return px_fwd_strided<T, KK, RB>(s, a, P);
        return PF_ERR_UNSUPPORTED;
    }
    const dim3 grid = px_fwd_grid(a, P, NT);
    if (P == 128) PF_LAUNCH(st, "conv_fwd_px", (conv_px_fwd_kernel<T, KK, RB, 4, NT, false>), grid, dim3(NT), s, a);
    if (P == 64) PF_LAUNCH(st, "conv_fwd_px", (conv_px_fwd_kernel<T, KK, RB, 2, NT, false>), grid, dim3(NT), s, a);
    if (P == 32) PF_LAUNCH(st, "conv_fwd_px", (conv_px_fwd_kernel<T, KK, RB, 1, NT, false>), grid, dim3(NT), s, a);
    return st;
}
template <typename T, int KK, int RB>
static int px_fwd_t(hipStream_t s, const PxFwdArgs<T> &a, int P, int threads)
{
    if constexpr (sizeof(T) == 2 && RB <= 2) {
        if (threads == 256) return px_fwd_p<T, KK, RB, 256>(s, a, P);
    }
    return threads == 512 ? px_fwd_p<T, KK, RB, 512>(s, a, P) : PF_ERR_UNSUPPORTED;
}
template <typename T, int KK>
static int px_fwd_r(hipStream_t s, const PxFwdArgs<T> &a, int P, int threads)
{
    if constexpr (sizeof(T) == 2) {
        if (a.r > 64) return px_fwd_t<T, KK, 4>(s, a, P, threads);
    }
    return a.r <= 32 ? px_fwd_t<T, KK, 1>(s, a, P, threads) : px_fwd_t<T, KK, 2>(s, a, P, threads);
}
template <typename T>
int launch_px_fwd(hipStream_t s, const PxFwdArgs<T> &a, int k, int P, int threads)
{
    if ((P != 128 && P != 64 && P != 32) || a.r > (sizeof(T) == 2 ? 128 : 64) || (k != 1 && k != 3)) return PF_ERR_UNSUPPORTED;
    return k == 3 ? px_fwd_r<T, 9>(s, a, P, threads) : px_fwd_r<T, 1>(s, a, P, threads);
}
template int launch_px_fwd(hipStream_t, const PxFwdArgs<uint16_t> &, int, int, int);
template int launch_px_fwd(hipStream_t, const PxFwdArgs<float> &, int, int, int);

template <typename T>
__global__ __launch_bounds__(256) void px_pack_kernel(PxPack<T> p) { px_pack<T, 256>(p, blockIdx.x); }
template <typename T>
int launch_px_pack(hipStream_t s, const PxPack<T> &p)
{
    int st = PF_OK;
    PF_LAUNCH(st, "conv_px_pack", px_pack_kernel<T>, dim3(px_pack_blocks(p, 256)), dim3(256), s, p);
    return st;
}
template int launch_px_pack(hipStream_t, const PxPack<uint16_t> &);
template int launch_px_pack(hipStream_t, const PxPack<float> &);

template <typename T>
bool px_fits(int N, int C, int H, int W, int Cout, int r, int k, int stride, int pad, int Ho, int Wo)
{
    constexpr int V = PxEl<T>::V;
    if ((k != 1 && k != 3) || stride < 1 || pad != k / 2 || Ho != (H - 1) / stride + 1 || Wo != (W - 1) / stride + 1) return false;
    if (N < 1 || Ho * Wo < V || C % V || Cout % V || r > 16 * V || (i64)Cout * r < V) return false;
    const i64 px = (i64)N * H * W, lim = (1LL << 31) / (i64)sizeof(T); // 32-bit byte offsets
    return px * C < lim && px * Cout < lim && px * (r + V) < lim && (i64)px_pack_elems(C, r, k) < lim && (i64)Cout * r < lim;
}
template bool px_fits<uint16_t>(int, int, int, int, int, int, int, int, int, int, int);
template bool px_fits<float>(int, int, int, int, int, int, int, int, int, int, int);

// Have all tiles at most `slots` slots and `groups` groups?  A plan asks this for each tile size in both directions, so it is answered from a
// bound where that will do: `all` pixels on R rows more than one of n planes have all + h R + h Wp (n - 1) slots and the reach of the taps,
// and no more groups than (pixels + (V - 1) n) / V.  Otherwise from tiles: how far one reaches depends on where in the plane it starts,
// on a multiple of `step`, and inside a plane on the column alone (with stride, on the row within V as well), so the first rows and
// the end of a plane stand for all.  A plan takes 1 to 3 us so, where trying every tile took 42 (16 x 16 pixels) to 7700 (225 x 225).
template <int S>
static bool px_tiles_fit(const PxPlane<S> &g, const PxPlane<S> &o, int stride, int P, int slots, int groups, bool loose = false)
{
    constexpr int V = 1 << S;
    const auto gcd_with = [](int p, int n) { return n % p ? n & -n : p; }; // of a power of two and n
    const i64 npx = (i64)o.N * o.HW, tiles = (npx + P - 1) / P;
    const int step = gcd_with(P, o.HW), all = npx < P ? (int)npx : P;
    if (stride == 1) {
        const int planes = (o.HW - step + all - 1) / o.HW, rows = (o.W - gcd_with(step, o.W) + all - 1) / o.W; // (more than one)
        const int range = all + 2 * g.h * (g.W + 1);
        const int most = g.HW % V == 0 ? (range + (g.h ? 2 : 1) * (V - 1)) / V : (range + (V - 1) * (planes + 1)) / V;
        if (all + g.h * (rows + planes * g.Wp + 2 * (g.Wp + 1)) <= slots && most <= groups) return true;
    }
    const auto fits = [&](i64 p0) {
        const PxTile t = px_tile(g, o, stride, (int)p0, P, loose);
        return t.slots <= slots && px_groups(g, t) <= groups;
    };
    const i64 period = (i64)step * (o.W / gcd_with(step, o.W)) * (stride > 1 ? V : 1); // of the column (and the row within V)
    const i64 head = period + 4 * o.W, tail = (o.HW - 4 * o.W - P) / step * step;
    if (tiles <= 256 || head >= tail) {
        for (i64 i = 0; i < tiles && i < o.HW / step; ++i) // (i P mod HW takes every position)
            if (!fits(i * P)) return false;
        return true;
    }
    for (i64 q = 0; q < o.HW; q += step) { // (more than 256 tiles: the end of a plane is followed by another, if it can be)
        if (q >= head && q < tail) q = tail;
        if (!fits(q)) return false;
    }
    return true;
}
template <int S>
bool px_tile_fits(const PxPlane<S> &g, const PxPlane<S> &o, int stride, int P)
{
    typedef typename std::conditional<S == 3, uint16_t, float>::type T;
    typedef PxRows<T, 4, 256> R4;
    typedef PxRows<T, 2, 256> R2;
    typedef PxRows<T, 1, 256> R1;
    if (P == 128 || stride > 1) return px_tiles_fit(g, o, stride, P, R4::rows - 1, R4::groups);
    return P == 64 ? px_tiles_fit(g, o, 1, P, R2::rows - 1, R2::groups) : px_tiles_fit(g, o, 1, P, R1::rows - 1, R1::groups);
}
template bool px_tile_fits(const PxPlane<3> &, const PxPlane<3> &, int, int);
template bool px_tile_fits(const PxPlane<2> &, const PxPlane<2> &, int, int);
template <int S>
bool px_wgrad_fits(const PxPlane<S> &g) { return px_tiles_fit(g, g, 1, 128, 1 << 30, (PX_WG_ROWS - 8) >> S, true); }
template bool px_wgrad_fits(const PxPlane<3> &);
template bool px_wgrad_fits(const PxPlane<2> &);

} // namespace pf
