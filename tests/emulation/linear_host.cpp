// Host side of the bf16 linear kernels (test infrastructure, CPU only): which shapes the factor gradients take.
#include "pf_linear_grad.h"

extern "C" int emu_grad_takes(long long M, long long in, long long out, long long r) { return pf::linear_grad_supported(M, in, out, r); }
extern "C" int emu_grad_splits(long long M, long long in, long long out, long long r) { return pf::plan_linear_grad(M, in, out, r).splits; }
