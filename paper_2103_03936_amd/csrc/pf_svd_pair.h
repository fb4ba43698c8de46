// The decisions of the Jacobi SVD (pf_svd.hip), for device and host.
#pragma once

#include "pf_common.h"

namespace pf {

constexpr int SVD_MAX_SWEEPS = 24;

// Device-side state of a call
struct SvdCtrl {
    unsigned arrived[2]; // grid barriers of the two cooperative kernels
    unsigned failed;     // a barrier's wait ran out
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
    return nc > 1 ? SvdOutcome{(int)c.sweeps, (int)c.last, false} : SvdOutcome{0, 0, false};
}

} // namespace pf
