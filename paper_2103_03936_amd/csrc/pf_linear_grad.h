// Both factor gradients of the fully connected layer in bf16, as partial sums over runs of rows:
//     out[split][cols][r] = A[rows of the split][cols]^T B[those rows][r]     (A, B = dY, T and X, dT)
// and A's column sums (the bias gradient) beside one of them.
#pragma once

#include "pf_common.h"

namespace pf {

struct LinGradProb {
    const uint16_t *A, *B; // [M][cols], [M][r]
    int cols;
    float *out;  // [splits][cols][r]
    float *sums; // [splits][cols] or NULL
};
struct LinGradArgs {
    i64 M;
    int r, splits, per; // rows in splits of `per` times 64
    int n;
    LinGradProb p[2];
};
struct LinGradPlan {
    int splits, per; // 0: not taken
};

// Whole 16-byte pieces, ranks up to 256
bool linear_grad_supported(i64 M, i64 in, i64 out, i64 r);
LinGradPlan plan_linear_grad(i64 M, i64 in, i64 out, i64 r);
int launch_linear_grad(hipStream_t s, const LinGradArgs &a);

} // namespace pf
