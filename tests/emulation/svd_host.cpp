// The decisions of the Jacobi SVD on the host (test infrastructure, CPU only).  Built by tests/test_host_svd.py; nothing in
// the product loads it.
#include "pf_svd_pair.h"

using namespace pf;

extern "C" {
void emu_outcome(unsigned failed, unsigned sweeps, unsigned last, int nc, int *out)
{
    SvdCtrl c = {};
    c.failed = failed, c.sweeps = sweeps, c.last = last;
    const SvdOutcome o = svd_outcome(c, nc);
    out[0] = o.sweeps, out[1] = o.last, out[2] = o.lost;
}
}
