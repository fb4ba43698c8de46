// Eigenvectors of a symmetric matrix in double precision: Householder tridiagonalisation in one cooperative launch, eigenvalues
// by multisection, eigenvectors of the tridiagonal matrix by twisted factorisations, reflectors applied to them.
//
// The SVD (pf_svd.hip) uses the result as a preconditioner only: it is made orthonormal there, rejected where it is not nearly so
// already (clusters of eigenvalues), and what it leaves of the columns' inner products is checked and taken out.  One-sided Jacobi,
// which does the same for any matrix, needs eight sweeps of n / 8 - 1 rounds with a grid barrier each.  At n = 512: 9.8 ms there;
// here 0.80 ms for the reduction, 0.15 for the eigenvectors of T, 0.09 for the reflectors.
#include "pf_svd_eigen.h"

#include <type_traits>

namespace pf {

typedef unsigned long long u64;

// ------------------------------------------------------------------ sums over a wavefront
// x + (x of the lane that the data-parallel-primitive control word names)
template <int CTRL>
__device__ __forceinline__ double dpp_plus(double x)
{
    const u64 b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return x + __longlong_as_double((u64)hi << 32 | lo);
}
__device__ __forceinline__ double lane_value(double x, int lane)
{
    const u64 b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, lane), hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __longlong_as_double((u64)hi << 32 | lo);
}
// x + y after the upper half of x and the lower half of y, or x's odd rows of 16 and y's even ones, have changed places: half of
// the lanes have a sum over two halves (rows) of x, the others of y
__device__ __forceinline__ double halves_plus(double x, double y)
{
    const u64 a = __double_as_longlong(x), b = __double_as_longlong(y);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double((u64)hi[0] << 32 | lo[0]) + __longlong_as_double((u64)hi[1] << 32 | lo[1]);
}
__device__ __forceinline__ double rows_plus(double x, double y)
{
    const u64 a = __double_as_longlong(x), b = __double_as_longlong(y);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double((u64)hi[0] << 32 | lo[0]) + __longlong_as_double((u64)hi[1] << 32 | lo[1]);
}
// the sum over a row of 16 lanes, in all of them: neighbours, pairs, the mirrored halves of eight and sixteen
__device__ __forceinline__ double row_sum(double x)
{
    x = dpp_plus<0xB1>(x);
    x = dpp_plus<0x4E>(x);
    x = dpp_plus<0x141>(x);
    return dpp_plus<0x140>(x);
}
// the sum over the 64 lanes, in all of them (the four rows by readlane and scalar operands: the tail below 138 us, 134 so)
__device__ __forceinline__ double wave_sum(double x)
{
    x = row_sum(x);
    x = rows_plus(x, x);
    return halves_plus(x, x);
}
// four sums at once, with seven additions for 24: row q of the lanes has that of x[fold4_at(q)]
__device__ __forceinline__ double fold4(double x0, double x1, double x2, double x3)
{
    return row_sum(rows_plus(halves_plus(x0, x1), halves_plus(x2, x3)));
}
__device__ __forceinline__ int fold4_at(int q) { return (q & 1) << 1 | q >> 1; }

// 1 / q and 1 / sqrt(q) of any normal double: the hardware's approximation (at least 2^-23) and two Newton steps
__device__ __forceinline__ double rcp_any(double q)
{
    double y = __builtin_amdgcn_rcp(q);
    y = fma(y, fma(-q, y, 1.0), y);
    return fma(y, fma(-q, y, 1.0), y);
}
__device__ __forceinline__ double rsqrt_any(double q)
{
    double y = __builtin_amdgcn_rsq(q);
    y = fma(0.5 * y, fma(-q * y, y, 1.0), y);
    return fma(0.5 * y, fma(-q * y, y, 1.0), y);
}

// what the lanes of a wavefront wrote to LDS is there for its other lanes
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------ exchange between workgroups
// A value goes to a slot of its own that holds a bit pattern no computation leaves (all ones: arithmetic NaNs have a clear
// payload, and a NaN that came in as a float has clear low bits), past the writer's L2; readers poll the slot itself, so an
// exchange is one store and one load, with no flag and no barrier.
constexpr u64 SLOT_EMPTY = ~0ull;

// A row of G that is zero off the diagonal (a zero column of the matrix, or one orthogonal to all others) has a unit vector for
// its eigenvector, and several such rows may well have one eigenvalue: a filter bank with pruned filters has a zero for each.  Left
// as they are, their vectors would come out alike, and the whole matrix would go to the Jacobi iteration as well.  So their diagonal
// entries, which nothing else depends on, become distinct and lie below all other eigenvalues, at the scale of the rest of the
// matrix.  A call with a quarter of the columns zero, us, before -> now (Jacobi's preconditioner alone): 1024 x 512 10540 -> 1340
// (11390), 2304 x 256 4260 -> 720 (3910), 576 x 64 995 -> 290 (840); where no row is so, 576 x 64 248 -> 249.
template <int CHUNKS>
__device__ __forceinline__ void svd_isolate(double *G, int *place, SvdCtrl *ctrl, int n, int ld)
{
    __shared__ int count[4 * CHUNKS];
    __shared__ double most[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    u64 alone[CHUNKS];
    double scale = 0.0;
#pragma unroll
    for (int m = 0; m < CHUNKS; ++m) {
        const int j = min(tid + 256 * m, n - 1), flag = place[j];
        if (flag < 0) scale = fmax(scale, G[(i64)j * ld + j]);
        alone[m] = __ballot(tid + 256 * m < n && flag == 0);
        if (lane == 0) count[4 * m + wave] = __popcll(alone[m]);
    }
    for (int s = 32; s > 0; s >>= 1) scale = fmax(scale, __shfl_xor(scale, s, 64));
    if (lane == 0) most[wave] = scale;
    __syncthreads();
    int all = 0;
    for (int i = 0; i < 4 * CHUNKS; ++i) all += count[i];
    scale = fmax(fmax(most[0], most[1]), fmax(most[2], most[3]));
    if (!(scale > 0.0)) scale = 1.0;
#pragma unroll
    for (int m = 0; m < CHUNKS; ++m) {
        const int j = tid + 256 * m;
        int at = __popcll(alone[m] & ((1ull << lane) - 1));
        for (int i = 0; i < 4 * m + wave; ++i) at += count[i];
        if (alone[m] >> lane & 1) {
            place[j] = at;
            G[(i64)j * ld + j] = -scale * (double)(all - at) / (double)all;
        }
    }
    if (tid == 0) ctrl->isolated = (unsigned)all;
    __syncthreads();
}

// (the last workgroup has svd_isolate)
template <int CHUNKS>
__global__ __launch_bounds__(256) void svd_slots_kernel(u64 *slots, i64 n, double *G, int *place, SvdCtrl *ctrl, int nc, int ld)
{
    if (blockIdx.x == gridDim.x - 1) {
        svd_isolate<CHUNKS>(G, place, ctrl, nc, ld);
        return;
    }
    for (i64 i = (i64)blockIdx.x * 256 + threadIdx.x; i < n; i += (i64)(gridDim.x - 1) * 256) slots[i] = SLOT_EMPTY;
}
__device__ __forceinline__ void slot_put(u64 *slot, double x)
{
    __hip_atomic_store(slot, (u64)__double_as_longlong(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 slot_get(const u64 *slot) { return __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

template <int I, int END, int STEP, class F>
__device__ __forceinline__ void static_for(F f)
{
    if constexpr (I < END) {
        f(std::integral_constant<int, I>{});
        static_for<I + STEP, END, STEP>(f);
    }
}

// Sum over the workgroup: over the wavefront, and over the NT / 64 wavefronts through LDS (nothing to do with one)
template <int NT>
__device__ __forceinline__ double group_sum(double x, double *red)
{
    x = wave_sum(x);
    if constexpr (NT > 64) {
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
        __syncthreads();
        x = red[0];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) x += red[w];
    }
    return x;
}

// G = Q T Q^T, T tridiagonal.  The matrix stays in registers: a wavefront has CPW columns of both halves (dealt out cyclically, so
// that all keep work to the end), a lane every 64th row.  A step of the reduction
//   v from column k, p = G v, w = tau p - (tau^2 v.p / 2) v, G -= v w^T + w v^T
// needs p and column k + 1 from the other workgroups and nothing else: from them everyone forms w, the next column and the next
// v for itself, with the same arithmetic.  So a step is one exchange; column k + 1 as it was before the step goes out ahead of
// the products, and those are G x, x the column below row k + 1: v = e + x / (alpha - beta) and G e is column k + 1, so what is
// sent need not wait for the norm (829 -> 752 us); the products of a wavefront's four columns are summed together (-> 674).
// v goes to column k of L (below row k + 1, where it is 1), T's diagonal and subdiagonal to L[k][k] and L[k][k + 1], tau to tau[k].
// The chain of an exchange, two sums and a square root per step is what it takes, so a workgroup is one wavefront where the
// matrix allows it: everything but its columns' own elements of the vectors (LDS) stays in the lanes that need it, and nothing
// waits for a barrier (n = 512 to the last column, us: 1070; two wavefronts 1280, four 1290, eight 1615; two columns a wavefront 1180, eight 1390).
// NT > 64: the vectors are formed row tid + NT m per thread and handed to the wavefronts through LDS.
// The last SVD_TAIL columns are left to svd_tridiag_tail_kernel: what they are by then goes back to G.
// A wait is bounded; when it runs out, everyone leaves and ctrl->failed says so.
template <int RPT, int CPW, int NT>
__global__ __launch_bounds__(NT) void svd_tridiag_kernel(double *G, double *L, double *tau_out, u64 *slots, SvdCtrl *ctrl, int n, int ld)
{
    constexpr int ROWS = 64 * RPT, NW = NT / 64, RV = (ROWS + NT - 1) / NT;
    __shared__ double xs[ROWS], ws[ROWS], red1[NW], red2[NW];
    __shared__ int gave_up;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = blockIdx.x, nwg = gridDim.x;
    u64 *P = slots, *C = slots + (i64)(n - SVD_TAIL) * ld;
    const auto column = [&](int j) { return (j * NW + wave) * nwg + g; };
    double a[CPW][RPT], vr[RPT], vc[CPW]; // the columns; v at this lane's rows and at this wavefront's columns
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
        vc[j] = 0.0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int c = column(j), r = lane + 64 * i;
            a[j][i] = G[(i64)min(c, n - 1) * ld + min(r, n - 1)];
        }
    }
    __builtin_amdgcn_sched_barrier(0); // (a select on each load would become a branch around it, and every load a wait of its own)
#pragma unroll
    for (int j = 0; j < CPW; ++j)
#pragma unroll
        for (int i = 0; i < RPT; ++i) a[j][i] = column(j) < n && lane + 64 * i < n ? a[j][i] : 0.0;
#pragma unroll
    for (int i = 0; i < RPT; ++i) vr[i] = 0.0;
    double x[RV], w[RV], v[RV];
    double sq = 0.0;
#pragma unroll
    for (int m = 0; m < RV; ++m) {
        const int t = tid + NT * m;
        x[m] = t < n ? G[t] : 0.0;
        w[m] = 0.0;
        if (t < ROWS) xs[t] = x[m], ws[t] = 0.0;
        if (t > 1) sq += x[m] * x[m];
    }
    if (tid == 0) gave_up = 0;
    bool left = false;
    // steps [k0, k1), in which no row below 64 I0 and no vector element below NT M0 is looked at any more
    const auto run = [&](auto i0, int k0, int k1) {
        constexpr int I0 = decltype(i0)::value, M0 = 64 * I0 / NT;
        for (int k = k0; k < k1; ++k) {
            double rest;
            if constexpr (NT > 64)
                rest = group_sum<NT>(sq, red2); // (also: what the last step left in LDS is there)
            else
                wave_sync();
            const double alpha = xs[k + 1];
            double xc[CPW], wc[CPW];
#pragma unroll
            for (int j = 0; j < CPW; ++j) xc[j] = xs[column(j)], wc[j] = ws[column(j)];
            double xr[RPT], wr[RPT];
            if constexpr (NT > 64) {
#pragma unroll
                for (int i = I0; i < RPT; ++i) xr[i] = xs[lane + 64 * i], wr[i] = ws[lane + 64 * i];
            } else {
#pragma unroll
                for (int i = I0; i < RPT; ++i) xr[i] = x[i], wr[i] = w[i];
            }
            // the previous step's update
#pragma unroll
            for (int j = 0; j < CPW; ++j)
#pragma unroll
                for (int i = I0; i < RPT; ++i) a[j][i] = fma(-wr[i], vc[j], fma(-vr[i], wc[j], a[j][i]));
#pragma unroll
            for (int j = 0; j < CPW; ++j) {
                if (column(j) == k + 1) {
#pragma unroll
                    for (int i = I0; i < RPT; ++i) {
                        const int r = lane + 64 * i;
                        if (r > k && r < n) slot_put(C + (i64)k * ld + r, a[j][i]);
                    }
                }
            }
            // the products with x below row k + 1
            double dot[CPW];
#pragma unroll
            for (int i = I0; i < RPT; ++i) xr[i] = lane + 64 * i > k + 1 ? xr[i] : 0.0;
#pragma unroll
            for (int j = 0; j < CPW; ++j) {
                dot[j] = 0.0;
#pragma unroll
                for (int i = I0; i < RPT; ++i) dot[j] = fma(a[j][i], xr[i], dot[j]);
            }
            if constexpr (CPW == 4) {
                const double sum = fold4(dot[0], dot[1], dot[2], dot[3]);
                const int c = column(fold4_at(lane >> 4));
                if ((lane & 15) == 0 && c > k && c < n) slot_put(P + (i64)k * ld + c, sum);
            } else {
#pragma unroll
                for (int j = 0; j < CPW; ++j) dot[j] = wave_sum(dot[j]);
#pragma unroll
                for (int j = 0; j < CPW; ++j) {
                    const int c = column(j);
                    if (lane == j && c > k && c < n) slot_put(P + (i64)k * ld + c, dot[j]);
                }
            }
            asm volatile("" ::: "memory"); // (everything is on its way before anyone waits)
            // this step's v
            if constexpr (NT == 64) rest = wave_sum(sq);
            double tau = 0.0, beta = alpha, inv = 0.0;
            if (!(rest == 0.0)) {
                const double q = fma(alpha, alpha, rest), y = rsqrt_any(q), len = q * y;
                beta = alpha < 0.0 ? len : -len;
                tau = fma(fabs(alpha), y, 1.0);
                inv = rcp_any(alpha - beta);
            }
#pragma unroll
            for (int i = I0; i < RPT; ++i) {
                const int r = lane + 64 * i;
                vr[i] = r == k + 1 ? 1.0 : xr[i] * inv;
            }
#pragma unroll
            for (int j = 0; j < CPW; ++j) {
                const int c = column(j);
                vc[j] = c > k + 1 ? xc[j] * inv : c == k + 1 ? 1.0 : 0.0;
            }
#pragma unroll
            for (int m = M0; m < RV; ++m) {
                const int t = tid + NT * m;
                if constexpr (NT > 64)
                    v[m] = t > k + 1 ? x[m] * inv : t == k + 1 ? 1.0 : 0.0;
                else
                    v[m] = vr[m];
                if (g == k % nwg && t >= k && t < n) L[(i64)k * ld + t] = t > k + 1 ? v[m] : t == k + 1 ? beta : x[m];
            }
            if (g == k % nwg && tid == 0) tau_out[k] = tau;
            // the products and the next column; row k + 1 of both for everyone
            u64 bp[RV], bc[RV], b1, c1;
            for (int spin = 0;; ++spin) {
                bool wait = false;
                b1 = slot_get(P + (i64)k * ld + k + 1);
                c1 = slot_get(C + (i64)k * ld + k + 1);
#pragma unroll
                for (int m = M0; m < RV; ++m) {
                    const int t = min(max(tid + NT * m, k + 1), n - 1); // (rows that nobody needs read a neighbour's slot)
                    bp[m] = slot_get(P + (i64)k * ld + t);
                    bc[m] = slot_get(C + (i64)k * ld + t);
                }
#pragma unroll
                for (int m = M0; m < RV; ++m) wait |= bp[m] == SLOT_EMPTY || bc[m] == SLOT_EMPTY;
                if (!__any(wait || b1 == SLOT_EMPTY || c1 == SLOT_EMPTY)) break;
                if (spin > 2000000 || ((spin & 255) == 255 && __hip_atomic_load(&ctrl->failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                    __hip_atomic_store(&ctrl->failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    gave_up = 1;
                    left = true;
                    break;
                }
            }
            double s = 0.0, p[RV]; // G v: with v = e + x inv, column k + 1 and the product
#pragma unroll
            for (int m = M0; m < RV; ++m) {
                p[m] = fma(inv, __longlong_as_double(bp[m]), __longlong_as_double(bc[m]));
                s = fma(p[m], v[m], s);
            }
            s = group_sum<NT>(s, red1);
            if constexpr (NT > 64) left = gave_up != 0;
            if (left) return;
            const double h = 0.5 * tau * tau * s, w1 = fma(tau, fma(inv, __longlong_as_double(b1), __longlong_as_double(c1)), -h);
            sq = 0.0;
#pragma unroll
            for (int m = M0; m < RV; ++m) {
                const int t = tid + NT * m;
                w[m] = t > k && t < n ? fma(tau, p[m], -h * v[m]) : 0.0;
                x[m] = t > k && t < n ? fma(-v[m], w1, __longlong_as_double(bc[m])) - w[m] : 0.0;
                if (t < ROWS) ws[t] = w[m], xs[t] = x[m];
                if (t > k + 2) sq = fma(x[m], x[m], sq);
            }
        }
    };
    constexpr int STEP = RPT <= 8 ? 1 : RPT / 2;
    const int end = n - SVD_TAIL;
    static_for<0, RPT, STEP>([&](auto i0) {
        constexpr int I0 = decltype(i0)::value;
        if (!left) run(i0, 64 * I0, min(64 * (I0 + STEP), end));
    });
    __syncthreads();
    if (left || gave_up) return;
    // the last step's update and what is left (nobody reads G any more but its owner)
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
        const int c = column(j);
        if (c >= end && c < n) {
            const double wc = ws[c];
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                const int r = lane + 64 * i;
                if (r >= end && r < n) G[(i64)c * ld + r] = fma(-ws[r], vc[j], fma(-vr[i], wc, a[j][i]));
            }
        }
    }
}

// The same reduction of a matrix of at most SVD_TAIL columns, the last of G's, by one workgroup of four wavefronts, one per SIMD:
// nothing leaves the compute unit, a step has one barrier.  Row 32 q + 4 (lane / 8) + wavefront of the matrix, which stands at the
// end of 128 x 128, is held by eight lanes, 16 columns each; so a product's sum is one over eight lanes, an operand read from LDS
// serves four rows, and what is done falls away in quarters.  The vectors (elements lane and lane + 64) every wavefront forms for
// itself, with the same arithmetic.
// A step takes 0.95 us where it takes 2.1 between compute units, 1.75 at the end: n = 512 1072 -> 829 + 121 us (the rest 674 by now), n = 128 224 -> 121 (eight
// wavefronts 134; each q by itself, its sums in a row: 130).
// The chain of a step: x to LDS and back into the lanes' columns, update and product, their sums to LDS, the barrier, v.p, the
// next x.  The product is with x, not v = (e + x / (alpha - beta)), so the norm, a square root and a reciprocal run beside it; row and
// column k + 1, where v is 1, are used for the last time in step k and not updated.
template <int Q0>
__device__ __forceinline__ void tridiag_tail_steps(double (&a)[4][16], double (&x)[2], double &sq, double *X, double *W, double (*P)[SVD_TAIL],
                                                   double (*R)[SVD_TAIL], double *L, double *tau_out, int k0, int k1, int base, int n, int ld)
{
    constexpr int J0 = 2 * Q0; // columns from 16 J0 on
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ri = lane >> 3, cb = lane & 7;
    const auto columns = [&](const double *from, double (&to)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = J0; j < 8; ++j) {
            const double2 t = *(const double2 *)(from + 16 * j + 2 * cb);
            to[2 * j] = t.x, to[2 * j + 1] = t.y;
        }
    };
    double xc[16], xi[4]; // x below row k + 1, zeros above, at this lane's columns and rows
    columns(X, xc);
#pragma unroll
    for (int q = Q0; q < 4; ++q) xi[q] = X[32 * q + 4 * ri + wave];
    for (int k = k0; k < k1; ++k) {
        double *p = P[k & 1], *row = R[k & 1];
        double dot[4] = {};
#pragma unroll
        for (int j = 2 * J0; j < 16; ++j)
#pragma unroll
            for (int q = Q0; q < 4; ++q) dot[q] = fma(a[q][j], xc[j], dot[q]);
#pragma unroll
        for (int q = Q0; q < 4; ++q) dot[q] = dpp_plus<0xB1>(dot[q]);
#pragma unroll
        for (int q = Q0; q < 4; ++q) dot[q] = dpp_plus<0x4E>(dot[q]);
#pragma unroll
        for (int q = Q0; q < 4; ++q) dot[q] = dpp_plus<0x141>(dot[q]);
        const double rest = wave_sum(sq), alpha = lane_value(k + 1 < 64 ? x[0] : x[1], (k + 1) & 63);
        double tau = 0.0, beta = alpha, inv = 0.0;
        if (!(rest == 0.0)) {
            const double q = fma(alpha, alpha, rest), y = rsqrt_any(q), len = q * y;
            beta = alpha < 0.0 ? len : -len;
            tau = fma(fabs(alpha), y, 1.0);
            inv = rcp_any(alpha - beta);
        }
        if (cb == 0) {
#pragma unroll
            for (int q = Q0; q < 4; ++q) p[32 * q + 4 * ri + wave] = dot[q];
        }
        if (32 * Q0 + 4 * ri + wave == k + 1) { // (row k + 1: steps k of this Q0 have it among the first 32 that are left)
#pragma unroll
            for (int j = J0; j < 8; ++j) *(double2 *)(row + 16 * j + 2 * cb) = make_double2(a[Q0][2 * j], a[Q0][2 * j + 1]);
        }
        double v[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int t = lane + 64 * m;
            v[m] = t > k + 1 ? x[m] * inv : t == k + 1 ? 1.0 : 0.0;
            if (wave == 0 && t >= k) L[(i64)(base + k) * ld + base + t] = t > k + 1 ? v[m] : t == k + 1 ? beta : x[m];
        }
        if (threadIdx.x == 0) tau_out[base + k] = tau;
        __syncthreads(); // (the next step writes the other of P and R)
        double pv[2], sum = 0.0;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int t = lane + 64 * m;
            x[m] = t > k ? row[t] : 0.0;
            pv[m] = t > k ? fma(inv, p[t], x[m]) : 0.0;
            sum = fma(pv[m], v[m], sum);
        }
        const double b1 = lane_value(k + 1 < 64 ? pv[0] : pv[1], (k + 1) & 63);
        sum = wave_sum(sum);
        const double h = 0.5 * tau * tau * sum, w1 = fma(tau, b1, -h);
        sq = 0.0;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int t = lane + 64 * m;
            const double w = t > k ? fma(tau, pv[m], -h * v[m]) : 0.0;
            x[m] = t > k ? fma(-v[m], w1, x[m]) - w : 0.0;
            W[t] = w;
            X[t] = t > k + 2 ? x[m] : 0.0;
            if (t > k + 2) sq = fma(x[m], x[m], sq);
        }
        wave_sync();
        double wc[16];
        columns(W, wc);
#pragma unroll
        for (int q = Q0; q < 4; ++q) {
            const int i = 32 * q + 4 * ri + wave;
            const double wv = -W[i] * inv, xv = -xi[q] * inv;
#pragma unroll
            for (int j = 2 * J0; j < 16; ++j) a[q][j] = fma(wv, xc[j], fma(xv, wc[j], a[q][j]));
            xi[q] = X[i];
        }
        columns(X, xc);
        wave_sync(); // (they have been read)
    }
}
__global__ __launch_bounds__(256) void svd_tridiag_tail_kernel(double *G, double *L, double *tau_out, int *place, SvdCtrl *ctrl, int n, int ld)
{
    __shared__ __attribute__((aligned(16))) double X[4][SVD_TAIL], W[4][SVD_TAIL], P[2][SVD_TAIL], R[2][SVD_TAIL];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ri = lane >> 3, cb = lane & 7;
    const int base = n - SVD_TAIL, first = max(-base, 0); // place t of the 128 is row (and column) base + t of G, first .. 127 exist
    double a[4][16], x[2], sq = 0.0;
    const auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int r = 32 * q + 4 * ri + wave, c = 16 * (j >> 1) + 2 * cb + (j & 1); // (the matrix is symmetric: lanes read along it)
                a[q][j] = G[(i64)(base + max(r, first)) * ld + base + max(c, first)];
            }
        __builtin_amdgcn_sched_barrier(0); // (a select on each load would become a branch around it, and every load a wait of its own)
    };
    const int flag0 = place[min(lane, n - 1)], flag1 = place[min(lane + 64, n - 1)];
    fetch();
    if (base <= 0 && __any(flag0 == 0 || flag1 == 0)) { // (every wavefront comes to the same answer)
        svd_isolate<1>(G, place, ctrl, n, ld);
        fetch();
    }
    if (first > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int r = 32 * q + 4 * ri + wave, c = 16 * (j >> 1) + 2 * cb + (j & 1);
                a[q][j] = r >= first && c >= first ? a[q][j] : 0.0;
            }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int t = lane + 64 * m;
        const double y = G[(i64)(base + first) * ld + base + max(t, first)];
        x[m] = t >= first ? y : 0.0;
        X[wave][t] = t > first + 1 ? y : 0.0;
        if (t > first + 1) sq = fma(y, y, sq);
    }
    wave_sync();
    static_for<0, 4, 1>([&](auto q0) {
        constexpr int Q0 = decltype(q0)::value;
        tridiag_tail_steps<Q0>(a, x, sq, X[wave], W[wave], P, R, L, tau_out, max(first, 32 * Q0 - 1), min(32 * Q0 + 31, SVD_TAIL - 1), base, n, ld);
    });
    if (threadIdx.x == 63) L[(i64)(n - 1) * ld + n - 1] = x[1];
}

// The reflectors made whole (zeros above, the 1 at row k + 1), T's diagonal and subdiagonal to T[0 .. n) and T[n .. 2 n): the
// kernels that follow read both without a select (the one that applies reflectors spent a fifth of its instructions on them).
__global__ __launch_bounds__(256) void svd_unpack_kernel(double *L, double *T, int n, int ld)
{
    const int k = blockIdx.x;
    double *a = L + (i64)k * ld;
    if (threadIdx.x == 0) {
        T[k] = a[k];
        T[n + k] = k + 1 < n ? a[k + 1] : 0.0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < min(k + 2, n); i += 256) a[i] = i == k + 1 ? 1.0 : 0.0;
}

// ------------------------------------------------------------------ eigenvectors of T
// One wavefront per eigenvalue.  Nine multisections (64 points at a time; the sign changes in the determinants of T - x's leading
// minors say how many eigenvalues lie below x) leave an interval of 2^-54 of the whole.  The eigenvector: pivots of T - lambda
// from the top (lane 0) and from the bottom (lane 1); where the two meet with the smallest defect the vector is 1, outward it
// follows from the pivots.
// All of it are chains of n steps.  The determinants follow a three-term recurrence, one dependent FMA per step, where a chain of
// pivots has a reciprocal (512, four wavefronts a workgroup: 427 us with those, 170 so); T is scaled to norm 1/2 .. 1, and the
// last two determinants are scaled back together every eight steps, in which they grow by 3^8 at most.  A pivot is the quotient of
// two neighbours.
// Eigenvalues that are one to rounding (those of the null space of a matrix of lower rank, to begin with) would give vectors that are
// one as well.  So where more than one lie in an interval of 65^-7, 2^-42, of the whole, their vectors are those of T with a diagonal
// that grows by SVD_APART from row to row: distinct eigenvalues, far enough apart (2^-33) for vectors orthogonal to 1e-5, which the
// Newton steps make so to rounding.  All wavefronts whose eigenvalue lies in the interval come to the same answer, and the others'
// vectors need not change: they are orthogonal to these to n SVD_APART over the gap.  576 x 64 of rank 8, a call: 1.87 ms where the Jacobi
// preconditioner came after such vectors, 1.22 now.
constexpr int SVD_CHUNK = 8, SVD_ALIKE = 7;
constexpr double SVD_APART = 1.0 / (1ll << 33);
__device__ __forceinline__ void rescale(double &p0, double &p1)
{
    const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
    p0 = __builtin_amdgcn_ldexp(p0, e);
    p1 = __builtin_amdgcn_ldexp(p1, e);
}
__global__ void svd_tridiag_vectors_kernel(const double *D, double *X, int n, int ld)
{
    // T, (diagonal, squared subdiagonal above it) from the top, padded with rows that change no sign; then, per wavefront, the
    // T of eigenvalues that are one, or what the two directions have, element by element from their ends on, padded to whole chunks
    extern __shared__ f64x2_t lds2[];
    const int np = (n + SVD_CHUNK - 1) / SVD_CHUNK * SVD_CHUNK;
    f64x2_t *T = lds2;
    const double *E = D + n; // E[i]: between i and i + 1
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    double *top = (double *)(lds2 + (np + 2 * SVD_CHUNK) * (1 + wave)), *bottom = top + np + SVD_CHUNK;
    // all eigenvalues lie within the row sums
    double lo = __builtin_huge_val(), hi = -lo;
    for (int i = lane; i < n; i += 64) {
        const double di = D[i], r = fabs(E[i]) + (i > 0 ? fabs(E[i - 1]) : 0.0);
        lo = fmin(lo, di - r);
        hi = fmax(hi, di + r);
    }
    for (int s = 32; s > 0; s >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, s, 64));
        hi = fmax(hi, __shfl_xor(hi, s, 64));
    }
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(lo), fabs(hi)));
    lo = __builtin_amdgcn_ldexp(lo, ex) - 1e-15;
    hi = __builtin_amdgcn_ldexp(hi, ex) + 1e-15;
    for (int i = tid; i < np + 2 * SVD_CHUNK; i += blockDim.x) {
        f64x2_t t = {4.0, 0.0};
        if (i < n) {
            const double b = i > 0 ? __builtin_amdgcn_ldexp(E[i - 1], ex) : 0.0;
            t[0] = __builtin_amdgcn_ldexp(D[i], ex);
            t[1] = b * b;
        }
        T[i] = t;
    }
    __syncthreads();
    const int j = blockIdx.x * waves + wave;
    if (j >= n) return;
    const f64x2_t *S = T;
    int fewer = 0, most = n; // eigenvalues below lo, and below hi
    bool alike = false;
    for (int round = 0; round < 9; ++round) {
        if (round == SVD_ALIKE && most - fewer > 1 && !alike) {
            f64x2_t *own = (f64x2_t *)top;
            for (int i = lane; i < np + 2 * SVD_CHUNK; i += 64) {
                f64x2_t t = T[i];
                t[0] = fma(SVD_APART, (double)i, t[0]);
                own[i] = t;
            }
            wave_sync();
            S = own;
            alike = true;
            hi += n * SVD_APART; // (the eigenvalues move up by less)
            round = 4;
        }
        const double x = lo + (hi - lo) * ((lane + 1) * (1.0 / 65.0));
        double p0 = 0.0, p1 = 1.0; // the last two determinants
        int below = 0;
        f64x2_t a[SVD_CHUNK], b[SVD_CHUNK]; // two chunks in turn: one is on its way from LDS while the other is worked on
        const auto fetch = [&](f64x2_t (&t)[SVD_CHUNK], int i) {
#pragma unroll
            for (int u = 0; u < SVD_CHUNK; ++u) t[u] = S[i + u];
            __builtin_amdgcn_sched_barrier(0);
        };
        const auto steps = [&](const f64x2_t (&t)[SVD_CHUNK]) {
#pragma unroll
            for (int u = 0; u < SVD_CHUNK; ++u) {
                const double p = fma(t[u][0] - x, p1, -(t[u][1] * p0));
                below += (unsigned)(__double2hiint(p) ^ __double2hiint(p1)) >> 31;
                p0 = p1;
                p1 = p;
            }
            rescale(p0, p1);
            __builtin_amdgcn_sched_barrier(0);
        };
        fetch(a, 0);
        for (int i = 0; i < np; i += 2 * SVD_CHUNK) {
            fetch(b, i + SVD_CHUNK);
            steps(a);
            fetch(a, i + 2 * SVD_CHUNK < np ? i + 2 * SVD_CHUNK : 0);
            steps(b); // (past the end: padding)
        }
        const u64 above = __ballot(below > j);
        const int f = above ? __ffsll(above) - 1 : 64; // the first point with the eigenvalue below it
        const double nlo = f > 0 ? lo + (hi - lo) * (f * (1.0 / 65.0)) : lo, nhi = f < 64 ? lo + (hi - lo) * ((f + 1) * (1.0 / 65.0)) : hi;
        if (f > 0) fewer = __builtin_amdgcn_readlane(below, f - 1);
        if (f < 64) most = __builtin_amdgcn_readlane(below, f);
        lo = nlo;
        hi = nhi;
    }
    wave_sync();
    const double lambda = 0.5 * (lo + hi);
    // determinants from the top (lane 0) and from the bottom (lane 1), and the pivots that they are quotients of
    double *mine = lane & 1 ? bottom : top;
    if (lane < 2) {
        double p0 = 0.0, p1 = 1.0;
        for (int s = 0; s < np; s += SVD_CHUNK) {
            double di[SVD_CHUNK], e2[SVD_CHUNK], q[SVD_CHUNK];
#pragma unroll
            for (int u = 0; u < SVD_CHUNK; ++u) {
                const int i = lane ? max(n - 1 - s - u, 0) : s + u;
                di[u] = T[i][0] - lambda;
                e2[u] = T[lane ? i + 1 : i][1];
            }
            if (alike) { // (S is no longer there)
#pragma unroll
                for (int u = 0; u < SVD_CHUNK; ++u) di[u] = fma(SVD_APART, (double)(lane ? n - 1 - s - u : s + u), di[u]);
            }
#pragma unroll
            for (int u = 0; u < SVD_CHUNK; ++u) {
                const double p = fma(di[u], p1, -(e2[u] * p0));
                q[u] = p * rcp_any(p1);
                p0 = p1;
                p1 = p;
            }
            rescale(p0, p1);
#pragma unroll
            for (int u = 0; u < SVD_CHUNK; ++u) mine[s + u] = q[u];
        }
    }
    wave_sync();
    double best = __builtin_huge_val();
    int k = 0;
    for (int i = lane; i < n; i += 64) {
        const double defect = fabs(top[i] + bottom[n - 1 - i] - (fma(alike ? SVD_APART : 0.0, (double)i, T[i][0]) - lambda));
        if (defect < best) best = defect, k = i;
    }
    for (int s = 32; s > 0; s >>= 1) {
        const double b = __shfl_xor(best, s, 64);
        const int kk = __shfl_xor(k, s, 64);
        if (b < best || (b == best && kk < k)) best = b, k = kk;
    }
    // pivots -> factors from an element to the next outward one
    for (int i = lane; i < n; i += 64) {
        if (i == k) continue;
        double *f = i < k ? top + i : bottom + (n - 1 - i);
        *f = -__builtin_amdgcn_ldexp(E[i < k ? i : i - 1], ex) * rcp_any(*f);
    }
    wave_sync();
    if (lane < 2) {
        double q = 1.0;
        const int first = lane ? n - 2 - k : k - 1, steps = max(k, n - 1 - k);
        for (int s = 0; s < steps; s += SVD_CHUNK) {
            double f[SVD_CHUNK];
            int at[SVD_CHUNK];
#pragma unroll
            for (int u = 0; u < SVD_CHUNK; ++u) {
                at[u] = first - s - u >= 0 ? first - s - u : np + u;
                f[u] = mine[at[u]];
            }
#pragma unroll
            for (int u = 0; u < SVD_CHUNK; ++u) f[u] = q *= f[u];
#pragma unroll
            for (int u = 0; u < SVD_CHUNK; ++u) mine[at[u]] = f[u];
        }
    }
    wave_sync();
    double sum = 0.0;
    for (int i = lane; i < n; i += 64) {
        const double z = i < k ? top[i] : i > k ? bottom[n - 1 - i] : 1.0;
        sum = fma(z, z, sum);
    }
    const double inv = rsqrt_any(wave_sum(sum));
    for (int i = lane; i < n; i += 64) X[(i64)j * ld + i] = (i < k ? top[i] : i > k ? bottom[n - 1 - i] : 1.0) * inv;
}

// ------------------------------------------------------------------ X = Q Z
// A wavefront applies all reflectors to one of Z's columns, kept in registers, two at a time:
//   H1 H2 z = z - tau2 d2 v2 - tau1 (d1 - tau2 d2 v1.v2) v1,  d = v.z
// so a pair costs the chain one sum over the wavefront.  The next DEPTH pairs are on their way meanwhile (one reflector at a time and
// one ahead: 298 us at 512; two, all rows read 121; without the rows where both are zero, in blocks of 64: 104; three sums in one: 91; two wavefronts a
// workgroup instead of four, which read the same reflectors together: 138).
template <int RPT, int DEPTH>
__global__ __launch_bounds__(256) void svd_reflect_kernel(const double *L, const double *tau, double *X, int n, int ld)
{
    const int lane = threadIdx.x & 63, j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= n) return;
    double z[RPT], v1[DEPTH][RPT], v2[DEPTH][RPT], t1[DEPTH], t2[DEPTH];
    // pair q: reflectors last - 2 q (first to be applied) and the one before it; where there is none, a factor of zero.  Rows past
    // the last are read from it, and z is zero there.
    const int last = n - 3, pairs = (n - 1) / 2;
    const auto fetch = [&](auto i0, int q, int d) {
        const int kb = max(last - 2 * q, 0), ka = max(kb - 1, 0);
        t1[d] = tau[ka];
        t2[d] = tau[kb];
#pragma unroll
        for (int i = decltype(i0)::value; i < RPT; ++i) {
            const int r = min(lane + 64 * i, n - 1);
            v1[d][i] = L[(i64)ka * ld + r];
            v2[d][i] = L[(i64)kb * ld + r];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < RPT; ++i) z[i] = X[(i64)j * ld + min(lane + 64 * i, n - 1)];
#pragma unroll
    for (int i = 0; i < RPT; ++i) z[i] = lane + 64 * i < n ? z[i] : 0.0;
    // pairs [q0, end), whose vectors are zero above row 64 I0: those rows are not read
    const auto apply = [&](auto i0, int q0, int end) {
        constexpr int I0 = decltype(i0)::value;
        if (q0 >= end) return;
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) fetch(i0, q0 + d, d);
        for (; q0 < end; q0 += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                const int kb = last - 2 * (q0 + d);
                double d1 = 0.0, d2 = 0.0, cross = 0.0;
#pragma unroll
                for (int i = I0; i < RPT; ++i) {
                    cross = fma(v1[d][i], lane + 64 * i < n ? v2[d][i] : 0.0, cross);
                    d1 = fma(v1[d][i], z[i], d1);
                    d2 = fma(v2[d][i], z[i], d2);
                }
                const bool in = q0 + d < end;
                const double tau1 = in && kb > 0 ? t1[d] : 0.0, tau2 = in && kb >= 0 ? t2[d] : 0.0;
                const double sums = fold4(cross, d1, d2, 0.0);
                d2 = -tau2 * lane_value(sums, 16);
                d1 = -tau1 * fma(d2, lane_value(sums, 0), lane_value(sums, 32));
#pragma unroll
                for (int i = I0; i < RPT; ++i) z[i] = lane + 64 * i < n ? fma(d1, v1[d][i], fma(d2, v2[d][i], z[i])) : 0.0;
                fetch(i0, q0 + DEPTH + d, d);
            }
        }
    };
    constexpr int STEP = RPT <= 8 ? 1 : RPT / 2;
    int q0 = 0;
    static_for<0, RPT, STEP>([&](auto i) {
        constexpr int I0 = RPT - STEP - decltype(i)::value;
        const int end = I0 == 0 ? pairs : last >= 64 * I0 ? (last - 64 * I0) / 2 + 1 : 0;
        apply(std::integral_constant<int, I0>{}, q0, end);
        q0 = max(q0, end);
    });
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = lane + 64 * i;
        if (r < n) X[(i64)j * ld + r] = z[i];
    }
}

template <int RPT, int CPW, int NT, int DEPTH>
static int eigenvectors(hipStream_t s, double *G, double *L, double *tau, double *X, int *place, SvdCtrl *ctrl, int n, int ld)
{
    int st = PF_OK;
    u64 *slots = (u64 *)X;
    double *T = G; // (free once it is tridiagonal; 2 n <= n ld)
    if constexpr (64 * RPT > SVD_TAIL) {
        const i64 words = 2 * (i64)(n - SVD_TAIL) * ld; // P's rows and C's, one per step
        const i64 blocks = (words + 1023) / 1024;
        PF_LAUNCH(st, "svd_slots", svd_slots_kernel<(64 * RPT + 255) / 256>, dim3((unsigned)(blocks < 1024 ? blocks : 1024) + 1), dim3(256), s, slots,
                  words, G, place, ctrl, n, ld);
        static_assert(NT / 64 * CPW == svd_eigen_columns(64 * RPT), "a workgroup's columns");
        if (st == PF_OK)
            st = launch_cooperative(s, "svd_tridiag", svd_tridiag_kernel<RPT, CPW, NT>, svd_eigen_workgroups(n), NT, G, L, tau, slots, ctrl, n, ld);
    }
    PF_LAUNCH(st, "svd_tridiag_tail", svd_tridiag_tail_kernel, dim3(1), dim3(256), s, G, L, tau, place, ctrl, n, ld);
    PF_LAUNCH(st, "svd_unpack", svd_unpack_kernel, dim3(n), dim3(256), s, L, T, n, ld);
    // two wavefronts per workgroup while those do not fill the chip (512: 171 -> 149 us), else what 64 KB of LDS hold, or one: with
    // more than 2032 columns that one takes 66048 bytes, of the 160 KB that a workgroup may have
    const int np = (n + SVD_CHUNK - 1) / SVD_CHUNK * SVD_CHUNK, waves = np <= 512 ? 2 : np <= 800 ? 4 : np <= 1000 ? 3 : np <= 1344 ? 2 : 1;
    PF_LAUNCH_LDS(st, "svd_tridiag_vectors", svd_tridiag_vectors_kernel, dim3((n + waves - 1) / waves), dim3(64 * waves),
                  (size_t)(1 + waves) * (np + 2 * SVD_CHUNK) * 16, s, (const double *)T, X, n, ld);
    PF_LAUNCH(st, "svd_reflect", (svd_reflect_kernel<RPT, DEPTH>), dim3((n + 3) / 4), dim3(256), s, (const double *)L,
              (const double *)tau, X, n, ld);
    return st;
}

int launch_svd_eigenvectors(hipStream_t s, double *G, double *L, double *tau, double *X, int *place, SvdCtrl *ctrl, int n, int ld)
{
    if (n > SVD_EIGEN_MAX) return PF_ERR_UNSUPPORTED;
    // what the registers hold without spilling: up to 512 rows one wavefront per workgroup, four columns each
    const auto run = n <= 64     ? eigenvectors<1, 4, 64, 4>
                     : n <= 128  ? eigenvectors<2, 4, 64, 4>
                     : n <= 256  ? eigenvectors<4, 4, 64, 4>
                     : n <= 512  ? eigenvectors<8, 4, 64, 4>
                     : n <= 1024 ? eigenvectors<16, 2, 256, 2>
                     : n <= 1536 ? eigenvectors<24, 2, 256, 1>
                                 : eigenvectors<32, 2, 256, 1>;
    return run(s, G, L, tau, X, place, ctrl, n, ld);
}

} // namespace pf
