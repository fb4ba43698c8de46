// The tiled products' kernels, plain matrices (one translation unit per element type).
#pragma once

#include "pf_tile_put.h"

namespace pf {

// SLICES: left operands of TILE_NT and right ones of TILE_TN may be partial sums (the registers of four slices: two wavefronts a SIMD)
template <typename CT, class CFG, bool SLICES>
__global__ __launch_bounds__(TILE_THREADS * CFG::DEEP, SLICES ? 2 : CFG::template OCC<CT>) void tile_linear_kernel(TileArgs by_value)
{
    const TileArgs &a = tile_args(by_value);
    constexpr int BM = CFG::BM, BN = CFG::BN, DEEP = CFG::DEEP, BK = TileEl<CT>::BK * DEEP;
    typedef LoadKC<CT, BM, false, DEEP> AK;
    typedef LoadKC<CT, BM, true, DEEP> AKS;
    typedef LoadMC<CT, BM, true, false, DEEP> AM;
    typedef LoadKC<CT, BN, true, DEEP> BKC;
    typedef LoadMC<CT, BN, false, false, DEEP> BMC;
    constexpr int s1 = TileSize<CT, CFG, AK, BKC>::bytes, s2 = TileSize<CT, CFG, AK, BMC>::bytes,
                  s3 = TileSize<CT, CFG, AM, BMC>::bytes;
    constexpr int bytes = s1 > s2 ? (s1 > s3 ? s1 : s3) : (s2 > s3 ? s2 : s3);
    __shared__ __attribute__((aligned(16))) unsigned char smem[bytes];
    const int tid = threadIdx.x;
    const TileAt t = find_tile<CFG>(a);
    if (!t.live) return;
    const TileProb &p = a.p[t.prob];
    const int kbeg = t.ks * p.kper, kend = min(p.K, kbeg + p.kper), nch = (kend - kbeg + BK - 1) / BK;
    typedef typename TileEl<CT>::elem elem;
    const elem *A = (const elem *)p.A + t.zb * p.sa, *B = (const elem *)p.B + t.zb * p.sb;
    if (p.type == TILE_NT) {
        BKC lb;
        lb.init(B, p.ldb, p.N, p.K, t.n0, kbeg, tid);
        lb.seg = p.bseg;
        lb.jump = p.bjump;
        if (SLICES && p.aslices > 1) {
            LoadKCS<CT, BM, DEEP> la;
            elem *copy = p.acopy && t.n0 == 0 ? (elem *)p.acopy + t.zb * p.sa : nullptr;
            la.init((const float *)p.A + t.zb * p.sa, p.lda, p.M, p.K, t.m0, kbeg, tid, p.aslices, p.sstride, p.aseg, p.ajump, copy);
            tile_product<CT, CFG>(la, lb, nch, smem, tid);
        } else {
            AKS la;
            la.init(A, p.lda, p.M, p.K, t.m0, kbeg, tid);
            la.seg = p.aseg;
            la.jump = p.ajump;
            tile_product<CT, CFG>(la, lb, nch, smem, tid);
        }
        tile_pieces<CT, CFG>(smem, tid, [&](int m, int n, float *v) {
            put_piece<CT, TileEl<CT>::V>(p, t.ks, t.zb, t.m0 + m, t.n0 + n, v);
        });
    } else if (p.type == TILE_NN) {
        AK la;
        BMC lb;
        la.init(A, p.lda, p.M, p.K, t.m0, kbeg, tid);
        lb.init(B, p.ldb, p.N, p.K, t.n0, kbeg, tid);
        tile_product<CT, CFG>(la, lb, nch, smem, tid);
        tile_pieces<CT, CFG>(smem, tid, [&](int m, int n, float *v) {
            put_piece<CT, TileEl<CT>::V>(p, t.ks, t.zb, t.m0 + m, t.n0 + n, v);
        });
    } else {
        AM la;
        la.init(A, p.lda, p.M, p.K, t.m0, kbeg, tid);
        if (SLICES && p.bslices > 1) {
            LoadMCS<CT, BN, DEEP> lb;
            lb.init((const float *)p.B + t.zb * p.sb, p.ldb, p.N, p.K, t.n0, kbeg, tid, p.bslices, p.sstride);
            tile_product<CT, CFG>(la, lb, nch, smem, tid);
        } else {
            BMC lb;
            lb.init(B, p.ldb, p.N, p.K, t.n0, kbeg, tid);
            tile_product<CT, CFG>(la, lb, nch, smem, tid);
        }
        finish<CT, CFG, AM>(p, t.ks, t.zb, t.m0, t.n0, la, t.m0, p.M, p.o.sums && t.n0 == 0, smem, tid);
    }
}

template <typename CT, class CFG>
static int launch_linear(hipStream_t s, const char *name, const TileArgs &a)
{
    int st = PF_OK;
    bool slices = false;
    for (int i = 0; i < a.n; ++i) {
        const TileProb &p = a.p[i];
        if (p.aslices > TILE_MAX_SLICES || p.bslices > TILE_MAX_SLICES || (p.aslices > 1 && p.type != TILE_NT) || (p.bslices > 1 && p.type != TILE_TN))
            return PF_ERR_UNSUPPORTED;
        slices = slices || p.aslices > 1 || p.bslices > 1;
    }
    const dim3 grid(a.blocks), block(TILE_THREADS * CFG::DEEP);
    if constexpr (CFG::BM * CFG::BN <= 32 * 32) {
        if (slices) PF_LAUNCH(st, name, (tile_linear_kernel<CT, CFG, true>), grid, block, s, a);
        else PF_LAUNCH(st, name, (tile_linear_kernel<CT, CFG, false>), grid, block, s, a);
    } else {
        if (slices) return PF_ERR_UNSUPPORTED; // (they take the registers of a larger tile's sums)
        PF_LAUNCH(st, name, (tile_linear_kernel<CT, CFG, false>), grid, block, s, a);
    }
    return st;
}
template <typename CT>
int launch_linear_t(hipStream_t s, const char *name, TileShape shape, const TileArgs &a)
{
    switch (shape) {
    // (two chunks in flight: with four, float 1280 tiles of 8 chunks take 18.6 us instead of 14.8, a third of the code more)
    case TS_32: return launch_linear<CT, TileCfg<32, 32, 1, 1, 2>>(s, name, a);
    case TS_32D: return launch_linear<CT, TileCfg<32, 32, 1, 1, 2, 2>>(s, name, a);
    case TS_64: return launch_linear<CT, TileCfg<64, 64, 2, 2, 2>>(s, name, a);
    case TS_128x64: return launch_linear<CT, TileCfg<128, 64, 2, 2, 2>>(s, name, a);
    case TS_128: return launch_linear<CT, TileCfg<128, 128, 2, 2, 2>>(s, name, a);
    default: return PF_ERR_UNSUPPORTED;
    }
}

} // namespace pf
