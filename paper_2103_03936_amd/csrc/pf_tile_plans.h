// What linear layers, LSTM cells and LSTM stacks plan for the tiled products (pf_tile_host.h).
#pragma once

#include "pf_common.h"
#include "pf_tile_host.h"

namespace pf {

// G linear layers that share their input
struct LinearTiles {
    bool ok;               // every dimension holds a 16-byte piece
    TilePlan T, dT, Y;     // tile shapes and splits of the intermediates and the output
    bool T_sliced, dT_sliced; // their readers take the partial sums (float) and add them up
    TileGroup grads;       // dX, dU and dV in one launch
    size_t n_mid, n_part_T, n_part_g, fwd_bytes, bwd_bytes; // elements of T, partial sums (floats)
};
LinearTiles make_linear_tiles(const pf_linear_desc *d, int G);
// Few rows in float: the streaming kernels of pf_skinny.h instead, for each direction
void linear_skinny_pays(const pf_linear_desc *d, const LinearTiles &t, bool &fwd, bool &bwd);

// One step of an LSTM layer
struct LstmTilePlan {
    TileGroup z, dxh, grads;
    MidGroup T, dT;
    TileGroup last; // dx, dh_prev and all gradients in one launch
    bool one;       // ... where that is faster than two
    double bwd;     // clocks of the backward products
    size_t n_T, n_dT, n_dxh, fwd_bytes, bwd_bytes; // partial sums, floats
};
LstmTilePlan make_lstm_tile_plan(const pf_lstm_desc *d);
// Backward on the streaming kernels of pf_skinny.h instead
bool lstm_skinny_pays(const pf_lstm_desc *d);

// The products over all rows = T B of a stack of LSTM layers at once: Tx = X Vx of the first layer (and, step by step, zx = Tx Ux^T) before
// the recurrence, dTx = dz Ux and dx = dTx Vx^T after it
struct StackTall {
    TilePlan Tx, zx, dx;
    MidPlan dTx;
    size_t n_part; // partial sums, floats
};
StackTall make_tall(i64 rows, i64 din, i64 h, i64 r, int G);

} // namespace pf
