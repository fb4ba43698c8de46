// The decisions of the Jacobi SVD on the host (test infrastructure, CPU only).  Built by tests/test_host_svd.py; nothing in
// the product loads it.
#include "pf_svd_eigen.h"

using namespace pf;

extern "C" {
int emu_orthogonal(double alpha, double beta, double gamma, double tol) { return svd_orthogonal(alpha, beta, gamma, tol * tol); }
int emu_orthogonal_short(double alpha, double beta, double gamma, double tol, double longest, int hold)
{
    const SvdShort few = svd_short(longest);
    return svd_orthogonal(alpha, beta, gamma, tol * tol, few.nil, hold ? few.low : 0.0);
}
void emu_rotation(double alpha, double beta, double gamma, double *cs)
{
    const f64x2_t r = svd_rotation(alpha, beta, gamma, 0.0);
    cs[0] = r[0], cs[1] = r[1];
}
int emu_before(double a, int i, double b, int j) { return svd_before(a, i, b, j); }
int emu_takes_eigenvectors(int n, int cus) { return svd_takes_eigenvectors(n, cus); }
void emu_outcome(unsigned failed, unsigned broken, unsigned sweeps, unsigned last, int nc, int *out)
{
    SvdCtrl c = {};
    c.failed = failed, c.broken = broken, c.sweeps = sweeps, c.last = last;
    const SvdOutcome o = svd_outcome(c, nc);
    out[0] = o.sweeps, out[1] = o.last, out[2] = o.lost;
}
}
