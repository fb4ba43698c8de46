// Tiled matrix products for any shape, the host side: problem lists, the choice of tile and split, launches.
#pragma once

#include "pf_tile.h"

namespace pf {

// Where a tile goes.  float32: C[split][m][n] (a partial sum per split of the contraction) or, unsplit, a gradient that
// is written or added to.  Otherwise elements of the call's type, row-major, or (HC > 0) planes [image][m][pixel] with
// the column index counting padded pixels as PixView does.
struct TileOut {
    void *C;
    i64 ld;
    int f32, accumulate;
    i64 split_stride;
    float *sums; // sums over k of the left operand's rows, [split][m]: gradients of a bias or a shift
    i64 sums_stride;
    const void *bias;           // per column, the call's element type
    const float *scale, *shift; // per row
    const void *add, *mask;     // like C: added before the ReLU / the output is kept where mask > 0
    int relu;
    int N, CH, HC, HW, gW; // images, channels, pieces per image, pixels per image, pixels per row (planes)
    int s, ph, pw, H, W;   // s > 1: pixel (y, x) is element (y s + ph, x s + pw) of an H x W plane
};

enum TileType {
    TILE_NN,   // A [M][K], B [K][N]
    TILE_NT,   // A [M][K], B [N][K]
    TILE_TN,   // A [K][M], B [K][N]
    TILE_CONV, // A [M][K], B a PixView (k = (channel, tap))
    TILE_CONVG,// the same with stride
    TILE_CONVT,// A [K][M] with a scale per k, B a PixView
    TILE_WG,   // A and B PixViews, k = pixel
    TILE_WGG,  // the same, B with stride
    TILE_WGT,  // TILE_WG whose row sums are those of the right operand
    TILE_PACK, // filters [q][c][tap] -> [c][q][selected tap]
};

struct TileProb {
    int type, M, N, K;
    int pair;                         // TILE_CONV: the next problem has the odd pixels of this one's rows, and no workgroups
    int tm, tn, ksplit, kper, block0; // kper: chunk-aligned extent of a split (images for TILE_WG)
    const void *A, *B;
    i64 lda, ldb;
    int nb;                // TILE_NN / NT / TN: products of the same shape, operands and output apart by
    i64 sa, sb, sc, ssums; // sa, sb, sc elements (and ssums row sums), a bias by sbias
    i64 sbias;
    int aseg, bseg;        // TILE_NT: an operand comes in segments of this many contraction indices (0: one), each a matrix
    i64 ajump, bjump;      // of its own, this many elements after the one before
    const float *ascale;
    int aslices, bslices;  // > 1: A of TILE_NT, B of TILE_TN are that many partial sums (float) of the operand, `sstride` floats
    i64 sstride;           // apart; acopy (nullable): their sums in the call's type, rows lda apart
    void *acopy;
    PixView pa, pb;
    TileOut o;
};

constexpr int TILE_MAX_PROBS = 6;
struct TileArgs {
    int n, blocks;
    TileProb p[TILE_MAX_PROBS];
};

// Tile shapes a launch can use (TS_32D: 32 x 32 by eight wavefronts).
enum TileShape { TS_32, TS_64, TS_128x64, TS_128, TS_32x64, TS_32x128, TS_32D, TS_COUNT };

// One product: add it to a launch.  ksplit <= 0 asks for the split that plan_tiles chose.
TileProb tile_prob(int type, int M, int N, int K, const void *A, i64 lda, const void *B, i64 ldb, void *C, i64 ldc);

struct TilePlan {
    TileShape shape;
    int ksplit;
    double cost; // cycles
};
// The tile shape and k-split that should finish first, at most max_split ways.
TilePlan plan_tiles(int dtype, i64 M, i64 N, i64 K, int max_split);

// Several products in one launch (one tile shape); those marked may split their contraction.
struct TileNeed {
    i64 M, N, K;
    bool split;
    bool tn; // the contraction is the slow index of both operands
};
struct TileGroup {
    TileShape shape;
    int ksplit[6];
    double cost;
};
TileGroup plan_tile_group(int dtype, const TileNeed *need, int n);
// Clocks of a launch of tiles of that shape whose first `chains` products are few tiles with a long contraction and the others many with a
// short one, all unsplit
double tile_chain_cost(int dtype, TileShape shape, const TileNeed *need, int n, int chains);

// The same for intermediates whose readers can take their partial sums instead (TileProb::aslices, bslices): `all` bytes of them go into
// the readers' workgroups, `most` into one.  sliced: they are to do so.
struct MidGroup {
    TileGroup g;
    bool sliced;
};
MidGroup plan_mid_group(int dtype, const TileNeed *need, int n, TileShape reader, i64 all, i64 most);
struct MidPlan { // of one intermediate M x N
    TilePlan t;
    bool sliced;
};
MidPlan plan_mid(int dtype, i64 M, i64 N, i64 K, int max_split, TileShape reader, i64 all, i64 most);

void tile_add(TileArgs &a, TileShape shape, int dtype, const TileProb &p, int ksplit);
// The last problem goes with the one before it (TileProb::pair).
void tile_pair(TileArgs &a);
int launch_tiles_linear(hipStream_t s, const char *name, int dtype, TileShape shape, const TileArgs &a);
// (`wg`: the shape of the weight gradients' tiles, pixels being summed over)
int launch_tiles_conv(hipStream_t s, const char *name, int dtype, TileShape shape, TileShape wg, const TileArgs &a);

// dst (+)= sum over splits of src[split], optionally times rscale[index / rlen]; bf16: dst holds bf16 (no accumulation)
struct SplitSum {
    const float *src;
    float *dst;
    i64 count, stride;
    int splits, accumulate;
    const float *rscale;
    i64 rlen;
    int bf16;
    int tm, tn; // tn > 0: src is [tm][tn], dst its transpose (rscale per row of dst)
    int np, hw; // np > 0: src is [tm][images][np], dst the planes [image][tm][hw], hw <= np
};
struct SplitSumArgs {
    int n, blocks[5];
    SplitSum s[4];
};
void split_sum_add(SplitSumArgs &a, const SplitSum &s);
int launch_split_sums(hipStream_t s, const SplitSumArgs &a);

} // namespace pf
