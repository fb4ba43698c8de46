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
// Polls of a workgroup that waits while others take `rounds` rounds of `each` polls: all of them, or those after which it gave up
long long emu_polls(int rounds, int each)
{
    SvdPatience p;
    long long n = 0;
    for (; n < (long long)rounds * each; ++n)
        if (!p.goes_on([&] { return (unsigned)(n / each); })) break;
    return n;
}
// ... of one that waits while others take `rounds` rounds and then none
long long emu_polls_then_stuck(int rounds, int each, long long most)
{
    SvdPatience p;
    long long n = 0;
    for (; n < most; ++n)
        if (!p.goes_on([&] { return (unsigned)(n / each < rounds ? n / each : rounds); })) break;
    return n;
}
int emu_crew(int stage, int nc, int sweepers) { return svd_crew(stage, nc, sweepers); }
void emu_outcome(unsigned failed, unsigned broken, unsigned sweeps, unsigned last, int nc, int *out)
{
    SvdCtrl c = {};
    c.failed = failed, c.broken = broken, c.sweeps = sweeps, c.last = last;
    const SvdOutcome o = svd_outcome(c, nc);
    out[0] = o.sweeps, out[1] = o.last, out[2] = o.lost;
}
}
