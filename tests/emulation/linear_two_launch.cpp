// The two-stage forward kernel by rows per workgroup and shares of the outputs (test infrastructure).  Built by
// tests/test_gpu_linear_two.py against the library, whose own calls choose them.
#include "pf_linear_two.h"

using namespace pf;
typedef uint16_t *u16;

extern "C" int linear_two(long long M, int K, int N, int r, int groups, int rows, int osplit, u16 X, u16 V, u16 U, u16 bias, u16 add, int relu, u16 Y, u16 T,
                          hipStream_t s)
{
    return launch_linear_two(s, "linear_two", LinTwoArgs{M, K, N, r, X, V, U, bias, add, Y, T, relu, groups, (i64)K * r, (i64)N * r, N, M * N, M * r, osplit}, rows);
}
