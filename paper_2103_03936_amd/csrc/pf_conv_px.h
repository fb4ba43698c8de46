// Convolutions on pixel-major tiles, bf16 and float, 1 x 1 or 3 x 3 taps: forward, and backward for planes of equal size.
// (The forward kernel takes any stride; calls reach it with 1 and 2, those of the tiled products, which are what it is chosen over.)
//
// The activations lie in memory with the pixel fast and are multiplied with the channel as the contraction.  The tiled products
// (pf_tile.h) keep that direction in LDS, so a tap is a shifted, masked copy of the operand: nine loads, masks and LDS writes of
// every element.  Here a square of channels and pixels at a time (eight, in float four) is turned in registers on its way to
// LDS, where a pixel is a row of channels; a tap is then an offset of the row (pf_conv_px_index.h) and nothing is loaded, masked or
// stored twice.
#pragma once

#include "pf_conv_chain.h"
#include "pf_conv_px_index.h"

namespace pf {

// Element types: uint16_t holds bf16.  V elements are a 16-byte piece, a 128-byte row of a panel PC channels; a step of the matrix unit
// takes 2 V channels (one bf16 instruction, four of float).
template <typename T>
struct PxEl;
template <>
struct PxEl<uint16_t> {
    static constexpr int S = 3, V = 8, PC = 64, dtype = PF_BF16;
};
template <>
struct PxEl<float> {
    static constexpr int S = 2, V = 4, PC = 32, dtype = PF_F32;
};
template <typename T>
using PxPlaneOf = PxPlane<PxEl<T>::S>;

template <typename T>
struct PxEpilogue {
    const float *scale, *shift; // per output channel
    const T *add, *mask;        // like the output: added before the ReLU / kept where mask > 0
    int relu;
};

// Thin filters [r][C][k k] as the backward kernel reads them: [mirrored tap][C][ranks, zeros up to 32, 64 or 128].
template <typename T>
struct PxPack {
    const T *Uk;
    T *to; // NULL: not wanted
    int C, r, kk;
};
inline int px_rank_blocks(int r) { return r <= 32 ? 1 : r <= 64 ? 2 : 4; }
inline size_t px_pack_elems(int C, int r, int k) { return (size_t)k * k * C * 32 * px_rank_blocks(r); }

template <typename T>
struct PxFwdArgs {
    PxPlaneOf<T> g, o; // planes of X, of Y
    int stride, C, Cout, r;
    const T *X, *Uk, *Vp;
    T *Y, *mid; // mid (the rank-r intermediate) may be NULL
    PxEpilogue<T> ep;
    PxPack<T> pack;  // in extra workgroups: for the backward kernel here,
    PackW1 chain1;   // or for the chain kernel's backward direction
    PackW2 chain2;
};

// dT = (scale Vp)^T dZ, kept with its ranks padded to whole pieces [N][px_ranks(r)][HW], and dX from it.
template <typename T>
__host__ __device__ inline int px_ranks(int r) { return (r + PxEl<T>::V - 1) / PxEl<T>::V * PxEl<T>::V; }
template <typename T>
struct PxBwdArgs {
    PxPlaneOf<T> g;
    int C, Cout, r;
    const T *dZ, *Vp, *Wb; // Wb: PxPack::to
    T *dX, *dT;
    const float *scale;
    PxEpilogue<T> ep; // of dX
};

// Filter gradients, partial sums over runs of 128-pixel tiles: G[group][rank][channel][tap] = sum over pixels of A[rank][p - tap] B[channel][p].
template <typename T>
struct PxGrad {
    const T *A, *B;         // [N][a_ch][HW], [N][C][HW]
    int a_ch, C, kk;        // a_ch: channels A has in memory (at least the rank)
    int units, groups, per; // workgroups: units (of px_slab channels) x groups of `per` tiles
    float *part, *sums;     // sums (one tap; may be NULL): [group][C], B's sums over the pixels
};
// rows that a 128-pixel tile with its halo may take in that kernel, groups one after the other
constexpr int PX_WG_ROWS = 232;
template <typename T>
struct PxWgradArgs {
    PxPlaneOf<T> g1, gk; // the planes under one tap and under the thin filters'
    int r;
    int n;               // problems
    PxGrad<T> p[2];      // the first one may have nine taps
};

// Output channels that the forward kernel forms at a time
constexpr int px_outputs(int rank_blocks, int P, int threads)
{
    return threads == 512 ? (P == 32 ? 256 : 128) : P == 32 ? 128 : rank_blocks * P == 512 ? 32 : 64;
}

// Shapes the kernels take: sizes, alignment of the rows, 32-bit offsets (float: ranks up to 64)
template <typename T>
bool px_fits(int N, int C, int H, int W, int Cout, int r, int k, int stride, int pad, int Ho, int Wo);
// Do all tiles of P pixels find room in LDS?
template <int S>
bool px_tile_fits(const PxPlane<S> &g, const PxPlane<S> &o, int stride, int P);
template <int S>
bool px_wgrad_fits(const PxPlane<S> &g);
// The backward kernels: float one tap and one block of ranks.  (With nine taps a wavefront's sums and their runs, the taps' rows and what is
// added and masks do not fit the registers: 40 to 60 us where the tiled products take 40.)
template <typename T>
inline bool px_bwd_takes(int k, int r)
{
    return sizeof(T) == 2 ? (k == 1 || k == 3) && r <= 128 : k == 1 && r <= 32;
}
template <typename T>
int px_slab(int k, int r); // channels of a workgroup of the filter gradients
template <typename T>
double px_wgrad_cost(int k, int r); // us that a tile takes a workgroup
// groups and tiles per group of both problems for the whole chip (C1 channels under k x k taps, C2 under one)
template <typename T>
void px_wgrad_plan(int npx, int r, int C1, int k, int C2, int (&groups)[2], int (&per)[2]);
template <typename T>
int launch_px_wgrad(hipStream_t s, const PxWgradArgs<T> &a);
template <typename T>
int launch_px_pack(hipStream_t s, const PxPack<T> &p);
// P pixels (128, 64 or 32) per workgroup of 512 threads, in bf16 up to rank 64 also 256; with stride 32, of one tap also 64 by 512
template <typename T>
int launch_px_bwd(hipStream_t s, const PxBwdArgs<T> &a, int k, int P, int threads);
template <typename T>
int launch_px_fwd(hipStream_t s, const PxFwdArgs<T> &a, int k, int P, int threads);

} // namespace pf
