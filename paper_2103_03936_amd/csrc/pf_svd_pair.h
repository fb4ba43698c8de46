// The decisions of the Jacobi SVD (pf_svd.hip), for device and host.
#pragma once

#include "pf_common.h"

#include <math.h>

namespace pf {

constexpr int SVD_MAX_SWEEPS = 40;
typedef __attribute__((ext_vector_type(2))) double f64x2_t;

// Device-side state of a call
struct SvdCtrl {
    unsigned arrived[3];    // grid barriers: of the preconditioner's sweeps, of B's first and of B's others
    unsigned failed;        // a barrier's wait ran out
    unsigned broken;        // a singular value is not finite: the matrix was not
    unsigned isolated;      // columns of the matrix that are orthogonal to all others, to the bit (zero columns among them)
    unsigned mixed;         // the eigenvectors of G are not orthogonal enough to be made so: the preconditioner is Jacobi's
    unsigned coarse[2];     // (per check) some column of B is farther from orthogonal than one correction takes out
    unsigned violations[2]; // pairs of B that are not orthogonal after the preconditioner, and after the first correction or sweep
    unsigned rot[3][SVD_MAX_SWEEPS + 1]; // pairs rotated per sweep: of L (in pairs of blocks with a large angle), of B first, of B then
    unsigned held[SVD_MAX_SWEEPS + 1];   // whether a sweep of B left pairs of short columns as they were
    unsigned sweeps;        // sweeps over the pairs of B, a check that found nothing included
    unsigned last;          // pairs rotated in the last of them
    double nil;             // squared norm below which a column of B is zero
    unsigned apart[64];     // (those who wait for the sweeps poll a line of their own)
    unsigned everyone;      // a barrier of all workgroups
};

// How long a workgroup polls for others before it gives up: SVD_POLLS times, counted afresh whenever those it waits for have got on.  (Two
// seconds at two polls a microsecond, far more than any round or product takes.  The sweeps of one stage may take longer: ten and more of
// seven rounds, 30 ms each for four million rows of 64 columns.)
constexpr int SVD_POLLS = 4000000;
struct SvdPatience {
    int polls = 0;
    unsigned seen = 0;
    // after a poll in vain: whether to go on; progress(): a counter that moves while the others do, asked for every 256 polls
    template <class PROGRESS>
    __host__ __device__ __forceinline__ bool goes_on(PROGRESS progress)
    {
        if (++polls % 256 == 0) {
            const unsigned now = progress();
            if (now != seen) seen = now, polls = 0;
        }
        return polls < SVD_POLLS;
    }
};

// Workgroups that sweep in a stage: the preconditioner's factorization and sweeps are by all that there are for it, those of B by one for each
// pair of blocks.  The others wait for them.
constexpr int SVD_B = 8; // columns of a block
__host__ __device__ __forceinline__ int svd_crew(int stage, int nc, int sweepers)
{
    const int pairs = ((nc + SVD_B - 1) / SVD_B + 1) / 2;
    return stage > 0 && pairs < sweepers ? pairs : sweepers;
}

// What a call reports: sweeps, rotations of the last one, and whether its outputs are worth nothing because a barrier's wait
// ran out (they are NaN then, for callers that do not ask for the report).
struct SvdOutcome {
    int sweeps, last;
    bool lost;
};
__host__ __device__ inline SvdOutcome svd_outcome(const SvdCtrl &c, int nc)
{
    if (c.failed) return SvdOutcome{SVD_MAX_SWEEPS, c.last ? (int)c.last : 1, true};
    SvdOutcome o = {0, 0, false};
    if (nc > 1) o.sweeps = (int)c.sweeps, o.last = (int)c.last;
    if (c.broken && o.last == 0) o.last = 1;
    return o;
}

// Whether singular value a of column i comes before b of column j (a total order: every column has a place)
__host__ __device__ __forceinline__ bool svd_before(double a, int i, double b, int j)
{
    const bool na = a != a, nb = b != b;
    return na != nb ? na : na || a == b ? i < j : a > b;
}

// Whether two columns with inner product gamma and squared norms alpha and beta are orthogonal to sqrt(tol2), relative.
// A column whose squared norm is below `nil` is orthogonal to any, one below `low` to others like it.
// Written so that NaN and infinity say no: a matrix that holds any never counts as converged.
__host__ __device__ __forceinline__ bool svd_orthogonal(double alpha, double beta, double gamma, double tol2, double nil = 0.0, double low = 0.0)
{
    const double g2 = gamma * gamma;
    const bool noise = nil == 0.0 ? false : (alpha < nil) | (beta < nil) | ((alpha < low) & (beta < low));
    return (g2 <= tol2 * (alpha * beta) || noise) && g2 < __builtin_huge_val();
}

// The two for columns of which the longest has squared norm `longest`.  The columns that a matrix of lower rank leaves over are rounding
// noise, smaller with every sweep, but never orthogonal to one another: there is no room for them, and what a sweep takes out of one
// the rotation against another brings back.  Below 2^-280 of the longest, less than any float is of another, a column is zero.
// From 2^-100 down columns are held back from one another until the longer ones take no more rotations: noise is gone by then,
// and what a graded matrix has of singular values so small is still separated.  (Sweeps for 576 x 64 of rank 40: 13, 7 now; of rank 20,
// where a limit of 2^-160 and no holding back takes 24 or more: 18 at most.)
struct SvdShort {
    double nil, low;
};
__host__ __device__ __forceinline__ SvdShort svd_short(double longest)
{
    return longest < __builtin_huge_val() ? SvdShort{0x1p-560 * longest, 0x1p-200 * longest} : SvdShort{0.0, 0.0};
}

// 1 / sqrt(q) and 1 / q to a few units of the last place: a float approximation (23 bits) and two Newton steps in double.
__host__ __device__ __forceinline__ double svd_rsqrt(double q)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double y = (double)__builtin_amdgcn_rsqf((float)q);
#else
    double y = (double)(1.0f / sqrtf((float)q));
#endif
    y = y * (1.5 - 0.5 * q * y * y);
    return y * (1.5 - 0.5 * q * y * y);
}
__host__ __device__ __forceinline__ double svd_rcp(double q)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double y = (double)__builtin_amdgcn_rcpf((float)q);
#else
    double y = (double)(1.0f / (float)q);
#endif
    y = y * (2.0 - q * y);
    return y * (2.0 - q * y);
}

// x over the power of two that brings y into [1/2, 1)
__host__ __device__ __forceinline__ double svd_scaled(double x, double y)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ldexp(x, -__builtin_amdgcn_frexp_exp(y));
#else
    int e;
    (void)frexp(y, &e);
    return ldexp(x, -e);
#endif
}

// The rotation (c, s) that takes gamma out of [[alpha, gamma], [gamma, beta]], all in double: s / c = t solves
// t^2 + 2 z t - 1 = 0, z = (beta - alpha) / (2 gamma), |t| <= 1.  With d = beta - alpha and g = 2 gamma that is
// t = +-g / (|d| + sqrt(d^2 + g^2)), scaled so that |d| + |g| is near 1: the arguments of the two approximations are then
// in float's range, while t itself may be as small as it is.  (Not alpha + beta: what rounding leaves of the norm of a column that
// rotations have all but cancelled, as in a matrix of lower rank, may be zero or below.)
__host__ __device__ __forceinline__ f64x2_t svd_rotation(double alpha, double beta, double gamma, double tol2, double nil = 0.0,
                                                         double low = 0.0)
{
    f64x2_t r = {1.0, 0.0};
    if (svd_orthogonal(alpha, beta, gamma, tol2, nil, low)) return r;
    const double d1 = beta - alpha, g1 = 2.0 * gamma, most = fabs(d1) + fabs(g1);
    const double d = svd_scaled(d1, most), g = svd_scaled(g1, most);
    const double q = d * d + g * g, n = fabs(d) + q * svd_rsqrt(q), t = (d < 0.0 ? -g : g) * svd_rcp(n), c = svd_rsqrt(1.0 + t * t);
    r[0] = c;
    r[1] = c * t;
    return r;
}

} // namespace pf
