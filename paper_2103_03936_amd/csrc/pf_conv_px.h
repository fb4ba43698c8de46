// Convolutions of bf16 on pixel-major tiles: unit stride, planes of equal size in and out, 1 x 1 or 3 x 3 taps.
//
// The activations lie in memory with the pixel fast and are multiplied with the channel as the contraction.  The tiled products
// (pf_tile.h) keep that direction in LDS, so a tap is a shifted, masked copy of the operand: nine loads, masks and LDS writes of
// every element.  Here eight channels of eight pixels at a time are turned in registers (one v_perm per word) on their way to
// LDS, where a pixel is a row of channels; a tap is then an offset of the row (pf_conv_px_index.h) and nothing is loaded, masked or
// stored twice.
#pragma once

#include "pf_conv_chain.h"
#include "pf_conv_px_index.h"

namespace pf {

struct PxEpilogue {
    const float *scale, *shift; // per output channel
    const uint16_t *add, *mask; // like the output: added before the ReLU / kept where mask > 0
    int relu;
};

// Thin filters [r][C][k k] as the backward kernel reads them: [mirrored tap][C][ranks, zeros up to 32, 64 or 128].
struct PxPack {
    const uint16_t *Uk;
    uint16_t *to; // NULL: not wanted
    int C, r, kk;
};
inline int px_rank_blocks(int r) { return r <= 32 ? 1 : r <= 64 ? 2 : 4; }
inline size_t px_pack_elems(int C, int r, int k) { return (size_t)k * k * C * 32 * px_rank_blocks(r); }

struct PxFwdArgs {
    PxPlane g;
    int C, Cout, r;
    const uint16_t *X, *Uk, *Vp;
    uint16_t *Y, *T; // T may be NULL
    PxEpilogue ep;
    PxPack pack;     // in extra workgroups: for the backward kernel here,
    PackW1 chain1;   // or for the chain kernel's backward direction
    PackW2 chain2;
};

// dT = (scale Vp)^T dZ, kept with its ranks padded to eights [N][(r + 7) / 8 8][HW], and dX from it.
struct PxBwdArgs {
    PxPlane g;
    int C, Cout, r;
    const uint16_t *dZ, *Vp, *Wb; // Wb: PxPack::to
    uint16_t *dX, *dT;
    const float *scale;
    PxEpilogue ep; // of dX
};

// Filter gradients, partial sums over runs of 128-pixel tiles: G[group][rank][channel][tap] = sum over pixels of A[rank][p] B[channel][p + tap].
struct PxGrad {
    const uint16_t *A, *B; // [N][a_ch][HW], [N][C][HW]
    int a_ch, C, kk;       // a_ch: channels A has in memory (at least the rank)
    int units, groups, per; // workgroups: units (of px_slab channels) x groups of `per` tiles
    float *part, *sums;    // sums (one tap; may be NULL): [group][C], B's sums over the pixels
};
// rows that a 128-pixel tile with its halo may take in that kernel, groups of eight pixels one after the other
constexpr int PX_WG_ROWS = 232;
struct PxWgradArgs {
    PxPlane g1, gk; // the planes under one tap and under the thin filters'
    int r;
    int n;          // problems
    PxGrad p[2]; // the first one may have nine taps
};

// Shapes the kernels take (bf16): sizes, alignment of the rows, 32-bit offsets.  `slots` and `groups`: the largest of any tile of P pixels.
bool px_fits(int N, int C, int H, int W, int Cout, int r, int k, int stride, int pad, int Ho, int Wo);
bool px_tile_fits(const PxPlane &g, int P);
bool px_wgrad_fits(const PxPlane &g);
// P pixels (128, 64 or 32) per workgroup of 256 or 512 threads
int px_slab(int k, int r); // channels of a workgroup
// groups and tiles per group of both problems for the whole chip (C1 channels under k x k taps, C2 under one)
void px_wgrad_plan(int npx, int r, int C1, int k, int C2, int (&groups)[2], int (&per)[2]);
int launch_px_wgrad(hipStream_t s, const PxWgradArgs &a);
int launch_px_pack(hipStream_t s, const PxPack &p);
int launch_px_bwd(hipStream_t s, const PxBwdArgs &a, int k, int P, int threads);
int launch_px_fwd(hipStream_t s, const PxFwdArgs &a, int k, int P, int threads);

} // namespace pf
