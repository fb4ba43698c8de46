// Eigenvectors of a symmetric matrix in double precision (pf_svd_eigen.hip): the SVD's fast preconditioner.
#pragma once

#include "pf_common.h"
#include "pf_svd_pair.h"

namespace pf {

constexpr int SVD_NT = 512; // threads of the cooperative kernels

// Columns that the tridiagonal route takes.  Up to 16 the two blocks of columns of the Jacobi iteration are one workgroup's and need
// few barriers (16 columns of 16 rows: 232 us a call on it, 222 on this one; 20 columns: 359 and 243; 64: 791 and 250; 512: 11750
// and 1340); above 2048 a column of the matrix exceeds what a wavefront keeps of it.
constexpr int SVD_EIGEN_MIN = 17, SVD_EIGEN_MAX = 2048;

// The columns that the reduction leaves to one workgroup; and the workgroups that have the others, of four or eight columns each,
// which wait for one another.  A device that cannot hold them all at once (one per compute unit) does without them.
constexpr int SVD_TAIL = 128;
__host__ __device__ constexpr int svd_eigen_columns(int n) { return n <= 512 ? 4 : 8; }
inline int svd_eigen_workgroups(int n) { return n <= SVD_TAIL ? 0 : (n + svd_eigen_columns(n) - 1) / svd_eigen_columns(n); }
inline bool svd_takes_eigenvectors(int n, int cus)
{
    return n >= SVD_EIGEN_MIN && n <= SVD_EIGEN_MAX && svd_eigen_workgroups(n) <= cus;
}

// A launch whose workgroups are all resident (they wait for one another)
template <class... ARGS>
static int launch_cooperative(hipStream_t s, const char *name, void (*kernel)(ARGS...), int blocks, int threads, ARGS... args)
{
    TimingScope ts(name, s);
    void *list[] = {(void *)&args...};
    const hipError_t e = hipLaunchCooperativeKernel((const void *)kernel, dim3(blocks), dim3(threads), list, 0, s);
    return e == hipSuccess ? PF_OK : set_hip_error(e);
}

// X (n columns, leading dimension ld) = unit eigenvectors of the symmetric G, as orthogonal as the gaps between the eigenvalues
// allow, in ascending order of the eigenvalues.  place[j]: -1, or 0 where row j of G is zero off the diagonal; such rows are given
// eigenvalues below all of G's, and place comes back with the column of X that is the j-th unit vector, one of the first ctrl->isolated.
// G (overwritten), L (n columns of ld), tau (n) and X (2 n columns of ld) are scratch.
int launch_svd_eigenvectors(hipStream_t s, double *G, double *L, double *tau, double *X, int *place, SvdCtrl *ctrl, int n, int ld);

} // namespace pf
