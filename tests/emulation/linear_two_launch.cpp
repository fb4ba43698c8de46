// The two-stage kernel by rows per workgroup and shares of the outputs, and the factor gradients by splits (test infrastructure).
// Built by tests/test_gpu_linear_two.py against the library, whose own calls choose them.
#include "pf_linear_grad.h"
#include "pf_linear_two.h"

using namespace pf;
typedef uint16_t *u16;

extern "C" int linear_two(long long M, int K, int N, int r, int groups, int rows, int osplit, u16 X, u16 V, u16 U, u16 bias, u16 add, int relu, u16 Y, u16 T,
                          u16 mask, hipStream_t s)
{
    return launch_linear_two(
        s, "linear_two", LinTwoArgs{M, K, N, r, X, V, U, bias, add, Y, T, relu, groups, (i64)K * r, (i64)N * r, N, M * N, M * r, osplit, mask}, rows);
}

extern "C" int linear_grad(long long M, int r, int splits, int per, int n, int cols1, u16 A1, u16 B1, float *out1, float *sums1, int cols2, u16 A2, u16 B2,
                           float *out2, hipStream_t s)
{
    return launch_linear_grad(s, LinGradArgs{M, r, splits, per, n, {{A1, B1, cols1, out1, sums1}, {A2, B2, cols2, out2, nullptr}}});
}
