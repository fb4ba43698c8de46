// The factorized fully connected layer forward in one launch, in bf16, ranks up to 128 (256 in whole 16-byte pieces), any widths in whole pieces:
//     mid[rows][r] = in[rows][K] W1[K][r],   out[rows][N] = act(mid W2[N][r]^T + bias + add)
// and backward with in = dY, W1 = U, W2 = V, mid = dT, out = dX.
// (pf_linear_chain.h has the kernel for rank 128 and widths that are multiples of 256.)
#pragma once

#include "pf_common.h"

namespace pf {

struct LinTwoArgs {
    i64 M;
    int K, N, r;
    const uint16_t *in, *W1, *W2, *bias, *add; // bias [N] and add [M][N] may be NULL
    uint16_t *out, *mid;                       // mid may be NULL
    int relu;
    int groups;                          // layers side by side that share their input, elements from one to the next:
    i64 s_W1, s_W2, s_bias, s_out, s_mid;
    int osplit; // workgroups that share a row tile's outputs (each forms mid again)
    const uint16_t *mask; // [M][N], may be NULL (ranks in whole pieces only): outputs are kept where it is positive
};

bool linear_two_supported(i64 M, i64 K, i64 N, i64 r);
// Rows per workgroup (32, 64 or 128; above rank 128 at most 64, above 192 32) and shares of the outputs for the least time; microseconds
double plan_linear_two(i64 M, i64 K, i64 N, i64 r, int groups, int &rows, int &osplit);
int launch_linear_two(hipStream_t s, const char *name, const LinTwoArgs &a, int rows);

} // namespace pf
