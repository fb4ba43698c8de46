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
    if (!t.live) return;
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
        pack_filters<CT>(p, t.index, tid);
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
int launch_conv_t(hipStream_t s, const char *name, TileShape shape, const TileArgs &a)
{
    switch (shape) {
    case TS_32x64: return launch_conv<CT, TileCfg<32, 64, 1, 2, 4>>(s, name, a);
    case TS_64: return launch_conv<CT, TileCfg<64, 64, 2, 2, 4>>(s, name, a);
    case TS_128x64: return launch_conv<CT, TileCfg<128, 64, 2, 2, 2>>(s, name, a);
    default: return PF_ERR_UNSUPPORTED;
    }
}

} // namespace pf
