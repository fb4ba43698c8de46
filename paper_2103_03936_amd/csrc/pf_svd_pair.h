// The decisions of the Jacobi SVD (pf_svd.hip), for device and host.
#pragma once

#include "pf_common.h"

namespace pf {

constexpr int SVD_MAX_SWEEPS = 24;
typedef __attribute__((ext_vector_type(2))) double f64x2_t;

// Device-side state of a call
struct SvdCtrl {
    unsigned arrived[2]; // grid barriers of the two cooperative kernels
    unsigned failed;     // a barrier's wait ran out
    unsigned broken;     // a singular value is not finite: the matrix was not
    unsigned violations; // pairs of B that are not orthogonal after the preconditioner
    unsigned rot[2][SVD_MAX_SWEEPS + 1]; // block pairs rotated per sweep, of L and of B
    unsigned sweeps;     // sweeps over the pairs of B, the check included
    unsigned last;       // block pairs rotated in the last of them
};

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
// Written so that NaN and infinity say no: a matrix that holds any never counts as converged.
__host__ __device__ __forceinline__ bool svd_orthogonal(double alpha, double beta, double gamma, double tol2)
{
    const double g2 = gamma * gamma;
    return g2 <= tol2 * (alpha * beta) && g2 < __builtin_huge_val();
}

// The rotation that takes gamma out of [[alpha, gamma], [gamma, beta]].  The angle needs no more than float precision (what
// it leaves of gamma is 1e-7 of it); c is refined so that c^2 + s^2 = 1 to the last bit.
__host__ __device__ __forceinline__ f64x2_t svd_rotation(double alpha, double beta, double gamma, double tol2)
{
    f64x2_t r = {1.0, 0.0};
    if (svd_orthogonal(alpha, beta, gamma, tol2)) return r;
#if defined(__HIP_DEVICE_COMPILE__)
    const int e = -__builtin_amdgcn_frexp_exp(alpha + beta);
    const float d = (float)__builtin_amdgcn_ldexp(beta - alpha, e), g = (float)__builtin_amdgcn_ldexp(2.0 * gamma, e);
    const float z = d * __builtin_amdgcn_rcpf(g), az = fabsf(z);
    const float ta = az > 1e18f ? 0.5f * __builtin_amdgcn_rcpf(az) : __builtin_amdgcn_rcpf(az + __builtin_amdgcn_sqrtf(1.f + z * z));
    const double t = (double)copysignf(ta, z), w = 1.0 + t * t;
    double c = (double)__builtin_amdgcn_rsqf((float)w);
#else
    const double z = (beta - alpha) / (2.0 * gamma), t = (z >= 0.0 ? 1.0 : -1.0) / (fabs(z) + sqrt(1.0 + z * z)), w = 1.0 + t * t;
    double c = 1.0 / sqrt(w);
#endif
    c = c * (1.5 - 0.5 * w * c * c); // Newton: 23 -> 45 bits
    c = c * (1.5 - 0.5 * w * c * c);
    r[0] = c;
    r[1] = c * t;
    return r;
}

} // namespace pf
