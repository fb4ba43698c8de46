// The tiled products' kernels, convolutions (one translation unit per element type).
#pragma once

#include "pf_tile_put.h"

namespace pf {

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

// WG: the launch has weight gradients (tiles of CFGW).  Launches without run kernels without their registers.
template <typename CT, class CFG, class CFGW, bool GATHER, bool WG>
__global__ __launch_bounds__(TILE_THREADS, sizeof(CT) == 2 && CFG::BM * CFG::BN <= 64 * 64 ? 3 : 2) void
tile_conv_kernel(TileArgs by_value)
{
    const TileArgs &a = tile_args(by_value);
    constexpr int BM = CFG::BM, BN = CFG::BN, BK = TileEl<CT>::BK;
    typedef LoadKC<CT, BM> AK;
    typedef LoadMC<CT, BM, false, true> AS;
    typedef LoadPixMC<CT, BN, false> BP;
    typedef LoadPixMC<CT, BN, true> BPG;
    typedef LoadPixKC<CT, CFGW::BM, false, true> AW;
    typedef LoadPixKC<CT, CFGW::BM, false> AWT;
    typedef LoadPixKC<CT, CFGW::BN, false> BW;
    typedef LoadPixKC<CT, CFGW::BN, false, true> BWT;
    typedef LoadPixKC<CT, CFGW::BN, true> BWG;
    constexpr int s1 = TileSize<CT, CFG, AK, BP>::bytes, s2 = TileSize<CT, CFG, AS, BP>::bytes,
                  s3 = TileSize<CT, CFGW, AW, BW>::bytes;
    constexpr int s12 = s1 > s2 ? s1 : s2, bytes = WG && s3 > s12 ? s3 : s12;
    __shared__ __attribute__((aligned(16))) unsigned char smem[bytes];
    extern __shared__ __attribute__((aligned(16))) unsigned char tile_tables[];
    const int tid = threadIdx.x;
    const TileAt t = find_tile<CFG>(a);
    if (!t.live) return;
    const TileProb &p = a.p[t.prob];
    const int kbeg = t.ks * p.kper, nch = (min(p.K, kbeg + p.kper) - kbeg + BK - 1) / BK; // (not TILE_WG)
    constexpr bool STRIDED = GATHER && !WG; // (a strided input is the right operand of launches without weight gradients only)
    if (p.type == TILE_CONV || (STRIDED && p.type == TILE_CONVG)) {
        AK la;
        la.init(p.A, p.lda, p.M, p.K, t.m0, kbeg, tid);
        if (STRIDED && p.type == TILE_CONVG) {
            typename std::conditional<STRIDED, BPG, BP>::type lb;
            lb.init(p.pb, t.n0, kbeg, tid, tile_tables);
            tile_product<CT, CFG>(la, lb, nch, smem, tid);
        } else {
            BP lb;
            lb.init(p.pb, t.n0, kbeg, tid, tile_tables);
            tile_product<CT, CFG>(la, lb, nch, smem, tid);
            if constexpr (GATHER && PairOut<CT, CFG>::TAKEN) {
                if (p.pair) {
                    const TileProb &p2 = a.p[t.prob + 1];
                    PairOut<CT, CFG> both;
                    both.keep(smem, tid);
                    __syncthreads();
                    la.init(p2.A, p2.lda, p2.M, p2.K, t.m0, 0, tid);
                    lb.init(p2.pb, t.n0, 0, tid, tile_tables);
                    tile_product<CT, CFG>(la, lb, (p2.K + BK - 1) / BK, smem, tid);
                    both.put(p, t.m0, t.n0, smem, tid);
                    return;
                }
            }
        }
        put_planes<CT, CFG>(p, t.ks, t.zb, t.m0, t.n0, smem, tid);
    } else if (p.type == TILE_CONVT) {
        AS la;
        BP lb;
        la.init(p.A, p.lda, p.M, p.K, t.m0, kbeg, tid, p.ascale);
        lb.init(p.pb, t.n0, kbeg, tid, tile_tables);
        tile_product<CT, CFG>(la, lb, nch, smem, tid);
        put_planes<CT, CFG>(p, t.ks, t.zb, t.m0, t.n0, smem, tid);
    } else if (p.type == TILE_PACK) {
        pack_filters<CT>(p, t.index, tid);
    } else if constexpr (WG) {
        const TileAt u = find_tile<CFGW>(a);
        const int img0 = u.ks * p.kper, img1 = min(p.pa.N, img0 + p.kper);
        const int pieces = (img1 - img0) * p.pa.HC, n = (pieces + BK / TileEl<CT>::V - 1) / (BK / TileEl<CT>::V);
        unsigned char *tb = tile_tables + (AW::table_bytes(p.pa) + 15) / 16 * 16;
        if (p.type == TILE_WGT) {
            AWT la;
            BWT lb;
            la.init(p.pa, u.m0, img0, img1, tid, tile_tables);
            lb.init(p.pb, u.n0, img0, img1, tid, tb);
            __syncthreads();
            tile_product<CT, CFGW>(la, lb, n, smem, tid);
            finish<CT, CFGW, BWT>(p, u.ks, u.zb, u.m0, u.n0, lb, u.n0, p.N, p.o.sums && u.m0 == 0, smem, tid);
        } else {
            AW la;
            la.init(p.pa, u.m0, img0, img1, tid, tile_tables);
            if (GATHER && p.type == TILE_WGG) {
                BWG lb;
                lb.init(p.pb, u.n0, img0, img1, tid, tb);
                __syncthreads();
                tile_product<CT, CFGW>(la, lb, n, smem, tid);
            } else {
                BW lb;
                lb.init(p.pb, u.n0, img0, img1, tid, tb);
                __syncthreads();
                tile_product<CT, CFGW>(la, lb, n, smem, tid);
            }
            finish<CT, CFGW, AW>(p, u.ks, u.zb, u.m0, u.n0, la, u.m0, p.M, p.o.sums && u.n0 == 0, smem, tid);
        }
    }
}

// FORMS: which of the kernel's four forms a launch of these shapes can be, a bit each (strided input or paired pixels, weight gradients)
enum { CONV_PLAIN = 1, CONV_WG = 2, CONV_GATHER = 4, CONV_GATHER_WG = 8, CONV_ALL = 15 };
template <typename CT, class CFG, class CFGW, int FORMS>
static int launch_conv(hipStream_t s, const char *name, const TileArgs &a)
{
    typedef LoadPixMC<CT, CFG::BN, false> BP;
    int st = PF_OK, tab = 0;
    bool gather = false, wg = false;
    for (int i = 0; i < a.n; ++i) {
        const TileProb &p = a.p[i];
        if (p.pair && !PairOut<CT, CFG>::TAKEN) return PF_ERR_UNSUPPORTED;
        int b = BP::TAB;
        if (p.type == TILE_WG || p.type == TILE_WGT) b = (LoadPixKC<CT, 64, false>::table_bytes(p.pa) + 15) / 16 * 16 + LoadPixKC<CT, 64, false>::table_bytes(p.pb);
        if (p.type == TILE_WGG) b = (LoadPixKC<CT, 64, false>::table_bytes(p.pa) + 15) / 16 * 16 + LoadPixKC<CT, 64, true>::table_bytes(p.pb);
        if (b > tab) tab = b;
        wg = wg || p.type == TILE_WG || p.type == TILE_WGG || p.type == TILE_WGT;
        gather = gather || p.type == TILE_CONVG || p.type == TILE_WGG || p.pair;
    }
    tab = (tab + 15) / 16 * 16;
#define PF_TILE_CONV(G, W)                                                                                              \
    if constexpr (FORMS >> (2 * G + W) & 1)                                                                             \
        if (gather == G && wg == W) {                                                                                   \
            PF_LAUNCH_LDS(st, name, (tile_conv_kernel<CT, CFG, CFGW, G, W>), dim3(a.blocks), dim3(TILE_THREADS), tab, s, a); \
            return st;                                                                                                  \
        }
    PF_TILE_CONV(false, false)
    PF_TILE_CONV(false, true)
    PF_TILE_CONV(true, false)
    PF_TILE_CONV(true, true)
#undef PF_TILE_CONV
    return PF_ERR_UNSUPPORTED;
}
template <typename CT>
int launch_conv_t(hipStream_t s, const char *name, TileShape shape, TileShape wg, const TileArgs &a)
{
    typedef TileCfg<64, 64, 2, 2, 2> S64;
    typedef TileCfg<32, 64, 1, 2, 4> S32;
    typedef TileCfg<32, 128, 1, 4, 2> W32;
    // (half-height tiles beside weight gradients are those of dX in float with unit stride; the widest have Y alone)
    constexpr int BESIDE = sizeof(CT) == 4 ? CONV_WG : 0;
    switch (shape) {
    case TS_32x64: {
        bool grads = false;
        for (int i = 0; i < a.n; ++i) grads = grads || a.p[i].type == TILE_WG || a.p[i].type == TILE_WGT;
        if (grads && wg == TS_64) return launch_conv<CT, S32, S64, BESIDE>(s, name, a);
        if (grads && wg != TS_32x128) return PF_ERR_UNSUPPORTED;
        return launch_conv<CT, S32, W32, CONV_PLAIN | CONV_GATHER | BESIDE>(s, name, a);
    }
    case TS_64: return wg == TS_32x128 ? launch_conv<CT, S64, W32, CONV_ALL>(s, name, a) : launch_conv<CT, S64, S64, CONV_ALL>(s, name, a);
    case TS_128x64: return launch_conv<CT, TileCfg<128, 64, 2, 2, 2>, S64, CONV_PLAIN>(s, name, a);
    default: return PF_ERR_UNSUPPORTED;
    }
}

} // namespace pf
