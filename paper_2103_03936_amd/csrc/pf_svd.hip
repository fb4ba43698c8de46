// Truncated-SVD factor initialisation (Algorithm 1: W ~ U V^T with U = Ut_r S_r^(1/2), V = Vt_r S_r^(1/2)):
// preconditioned one-sided Jacobi in double precision.
//
// The matrix with fewer columns is taken (A = W or W^T, rows >= cols) and stored column-major.  One-sided Jacobi
// orthogonalises every pair of columns once per sweep; on A itself a sweep moves rows x cols numbers cols times and
// eight or more sweeps follow.  So an orthogonal V comes first that does most of it:
//   G = A^T A, V = its eigenvectors (pf_svd_eigen.hip), made orthonormal by two Newton steps V (3 I - V^T V) / 2, or, where
//   close eigenvalues leave vectors that cannot be made so (and for few columns, and very many):
//   G + shift I = L L^T, one-sided Jacobi on the cols x cols matrix L: L W = V S (no rotations accumulated: the normalised
//   columns themselves are the eigenvectors of G; the shift, the rounding level of G, keeps L defined for any matrix);
//   B = A V: columns orthogonal to about eps kappa^2.
// V is a preconditioner only.  All pairs of B's columns are checked against the threshold that the iteration on A would use.
// What is not orthogonal is taken out, V carried along: by B (I + K), K the first-order rotations from the Gram matrix, where
// they are so small that I + K is orthogonal to rounding, otherwise by rotations of the pairs of blocks that hold some.
// Unless a second check is content, sweeps of the Jacobi iteration follow until one finds nothing to rotate.
// So singular values far below the largest come out as exactly as without the preconditioner, down to 2^-92 of it or so (V carries
// 2^-52 of the long columns into the short ones, and what A V rounds of that stays).
// Singular values = column norms of B, sorted by counting; the r largest triplets are scaled and written out.
// 2048 x 512: 11.7 ms with Jacobi's preconditioner, 1.30 with the eigenvectors; 1024 x 512 with orthonormal columns 15.5 and 1.3
// (rounding to float tells the values apart); matrices of lower rank, whose noise takes sweeps either way, 576 x 64 of rank 8 1.67 and 1.19,
// 2304 x 256 of rank 32 15.0 and 10.4, 1024 x 512 with 16 columns twice 17.2 and 7.8.  A matrix whose eigenvalues lie close without being
// one (graded down to the rounding of G) pays for both: 300 x 60 with values down to 1e-9 1.29 / 1.43, 1024 x 256 8.9 / 9.2.  So does
// one in two blocks that share no row and no column, the first of lower rank and the other 1e-9 of it, whose columns the noise gets
// among: 1024 x 256 12.4 / 18.0 (1e-6 of it: 12.1 / 8.6).
//
// A pair of eight-column blocks is a workgroup's unit: Gram matrix of the 16 columns on the matrix unit, rotations of
// every column of one block against every column of the other (in a sweep's first round also within the blocks) found on
// that 16 x 16 matrix in LDS by one wavefront and applied to the rows, one row per thread.  Pairs of blocks are dealt into rounds by round-robin;
// the rounds of all sweeps run in ONE cooperative kernel with a grid barrier between them, because the number of sweeps is known on the device only:
// a launch per round has to be enqueued for the most sweeps that may be needed, at 2.8 us each (2048 x 512: 12264 launches, 84 ms).
// A barrier's wait is bounded: after about two seconds in which those it waits for have not got on a workgroup gives up; the call then
// reports no convergence and its outputs are NaN.
#include "pf_gemm.h"
#include "pf_svd_eigen.h"

namespace pf {

typedef __attribute__((ext_vector_type(4))) double f64x4_t;

// A pair counts as orthogonal when |a_p . a_q| <= tol |a_p| |a_q|.  The inner product of two columns of `rows` doubles carries
// rounding noise of about rows * 2^-53 relative to |a_p| |a_q|, so a tighter threshold never stops the sweeps.  A looser one
// leaves columns mixed whose singular values are close: by tol / (2 d) for values a relative d apart.
static double svd_tolerance(int rows)
{
    const double t = (double)rows * 2.220446049250313e-16;
    return t < 1e-15 ? 1e-15 : t;
}
// That of the preconditioner, whose columns become V: rounding level.
static double svd_tolerance_v(int rows) { return (double)(rows < 64 ? 64 : rows) * 2.220446049250313e-16; }

__global__ __launch_bounds__(256) void svd_init_kernel(const float *W, double *At, SvdCtrl *ctrl, int *place, int n, int nr, int nc, int ld,
                                                        int transposed)
{
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < (int)(sizeof(SvdCtrl) / 4); i += 256) ((unsigned *)ctrl)[i] = 0u;
    const i64 idx = (i64)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (i64)nc * ld) return;
    const int j = (int)(idx / ld), i = (int)(idx % ld);
    if (i == 0) place[j] = 0;
    At[idx] = i >= nr ? 0.0 : (double)(transposed ? W[(i64)j * n + i] : W[(i64)i * n + j]);
}

// Lane l of a wavefront holds column c0 + l % 16 of a column-major matrix at rows r0 + 2 (l / 16) + {0, 1}: fragments of
// two 16x16x4 MFMAs, for the left and for the right operand alike.  Past the last column or row a neighbour is read, and
// svd_masked makes it zero when it is used: a select on the load itself becomes a branch around it, with a wait of its own.
__device__ __forceinline__ f64x2_t svd_frag(const double *M, int ld, int col, int nc, int row, int nr)
{
    return *(const f64x2_t *)(M + (i64)min(col, nc - 1) * ld + min(row, (nr - 1) & ~1));
}
__device__ __forceinline__ double svd_masked(double v, bool in) { return in ? v : 0.0; }

// Sum over the wavefronts of a workgroup of a 32 x 32 tile: each has it as 2 x 2 MFMA tiles over its share of the contraction.
// put(i, j, sum) for the elements of thread tid.
template <int WAVES, class PUT>
__device__ __forceinline__ void svd_tile_out(const f64x4_t (&acc)[2][2], double (&part)[4][32][33], PUT put)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4;
#pragma unroll
    for (int q = 0; q < WAVES / 4; ++q) { // four at a time
        if (wave / 4 == q) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        double &sum = part[wave & 3][16 * a + g + 4 * v][16 * b + c];
                        sum = q ? sum + acc[a][b][v] : acc[a][b][v];
                    }
        }
        __syncthreads();
    }
    for (int e = tid; e < 1024; e += 64 * WAVES) {
        const int i = e >> 5, j = e & 31;
        put(i, j, (part[0][i][j] + part[1][i][j]) + (part[2][i][j] + part[3][i][j]));
    }
}

constexpr int SVD_U = 4; // pieces of eight contraction indices that a wavefront has in flight

// C = M^T M (symmetric, both halves written), 32 x 32 tile ti, tj <= ti by a workgroup; the wavefronts split the rows, and SVD_U pieces are
// requested while the SVD_U before are multiplied: a piece takes about a microsecond to arrive, its MFMAs 64 clocks each (2048 x 512:
// 88 us with one at a time, 64 with SVD_U and a wait before they are multiplied, 36 so; the product of the two below 58 -> 38
// us; with eight wavefronts, or columns that start in other channels of the L2, the same).  place
// (nullable): -1 for columns that have an inner product other than zero with another.
template <int WAVES, int U>
__device__ __forceinline__ void svd_gram_tile(const double *M, double *C, int nr, int nc, int ld, int ldc, int ti, int tj, int *place,
                                              double (&part)[4][32][33])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4;
    f64x4_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[a][b][v] = 0.0;
    struct Pieces {
        f64x2_t x[U][2], y[U][2];
    };
    const auto fetch = [&](Pieces &p, int r) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                p.x[u][a] = svd_frag(M, ld, 32 * ti + 16 * a + c, nc, r + 8 * u + 2 * g, nr);
                p.y[u][a] = svd_frag(M, ld, 32 * tj + 16 * a + c, nc, r + 8 * u + 2 * g, nr);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    const auto multiply = [&](const Pieces &p, int r) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const bool in = r + 8 * u + 2 * g + e < nr; // (columns past the last give sums that nobody stores)
                double x[2], y[2];
#pragma unroll
                for (int a = 0; a < 2; ++a) x[a] = svd_masked(p.x[u][a][e], in), y[a] = svd_masked(p.y[u][a][e], in);
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[a], y[b], acc[a][b], 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int STEP = 8 * WAVES * U;
    Pieces p0, p1;
    fetch(p0, 8 * U * wave);
    for (int r = 8 * U * wave; r < nr; r += 2 * STEP) {
        fetch(p1, r + STEP);
        multiply(p0, r);
        fetch(p0, r + 2 * STEP);
        multiply(p1, r + STEP); // (past the last row: zeros.  A condition here cost a wait: 65536 x 16 1605 us a call, 1568 without)
    }
    __shared__ int met[2][32];
    if (tid < 64) met[tid >> 5][tid & 31] = 0;
    svd_tile_out<WAVES>(acc, part, [&](int i, int j, double s) {
        const int gi = 32 * ti + i, gj = 32 * tj + j;
        if (gi < nc && gj < nc && (ti != tj || i >= j)) {
            C[(i64)gj * ldc + gi] = s;
            C[(i64)gi * ldc + gj] = s;
            if (place && gi != gj && !(s == 0.0)) met[0][i] = met[1][j] = 1;
        }
    });
    if (!place) return;
    __syncthreads();
    if (tid < 64 && met[tid >> 5][tid & 31]) place[32 * (tid < 32 ? ti : tj) + (tid & 31)] = -1;
}
// instead (nullable): nothing is done where it is set
__global__ __launch_bounds__(256) void svd_gram_kernel(const double *M, double *C, int nr, int nc, int ld, int ldc, const unsigned *instead,
                                                        int *place)
{
    __shared__ double part[4][32][33];
    if ((instead && *instead) || blockIdx.y > blockIdx.x) return;
    svd_gram_tile<4, SVD_U>(M, C, nr, nc, ld, ldc, blockIdx.x, blockIdx.y, place, part);
}

// The first-order rotation that takes the inner product g_ij of two columns out (0 where they count as orthogonal): with
// K = (k_ij), k_ij = -k_ji, the columns of B (I + K) are orthogonal to second order.
__device__ __forceinline__ double svd_small_rotation(double g_ii, double g_jj, double g_ij, double tol2)
{
    return svd_orthogonal(g_ii, g_jj, g_ij, tol2) ? 0.0 : g_ij / (g_jj - g_ii);
}
// The largest row sum of |K| for which B (I + K) will do: I + K is orthogonal to its square, the rounding level.
constexpr double SVD_COARSE = 3e-8;

// Counts the pairs of columns whose Gram entry says that they are not orthogonal, and says whether K is too large.  Column j by a
// workgroup, 256 threads of it (red: 256 doubles of LDS).
__device__ __forceinline__ void svd_check_column(const double *G, unsigned *violations, unsigned *coarse, int j, int nc, int ld, double tol,
                                                 double *red)
{
    const int tid = threadIdx.x;
    const double gj = G[(i64)j * ld + j];
    int bad = 0;
    double sum = 0.0;
    for (int i = tid; tid < 256 && i < nc; i += 256) {
        if (i == j) continue;
        const double gi = G[(i64)i * ld + i], g = G[(i64)j * ld + i];
        if (svd_orthogonal(gi, gj, g, tol * tol)) continue;
        bad += i > j ? 1 : 0;
        sum += fabs(g / (gj - gi));
    }
    __shared__ unsigned count;
    if (tid == 0) count = 0u;
    if (tid < 256) red[tid] = sum;
    __syncthreads();
    if (bad) atomicAdd(&count, (unsigned)bad);
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    if (tid == 0) {
        if (count) atomicAdd(violations, count);
        if (!(red[0] <= SVD_COARSE)) __hip_atomic_store(coarse, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
}
__global__ __launch_bounds__(256) void svd_check_kernel(const double *G, SvdCtrl *ctrl, int nc, int ld, double tol)
{
    __shared__ double red[256];
    if (ctrl->mixed) return;
    svd_check_column(G, &ctrl->violations[0], &ctrl->coarse[0], blockIdx.x, nc, ld, tol, red);
}

// How far the columns behind the Gram matrix S may be from orthonormal for one more Newton step to make them so: the norm of
// S - I is at most nc times its largest element, a step leaves 3/4 of its square (2e-13 here, at the very most).
constexpr double SVD_MIXED = 5e-7; // over nc
__global__ __launch_bounds__(256) void svd_mixed_kernel(const double *S, unsigned *mixed, int nc, int ld)
{
    const int j = blockIdx.x;
    bool bad = false;
    for (int i = threadIdx.x; i < nc; i += 256) bad |= !(fabs(S[(i64)j * ld + i] - (i == j ? 1.0 : 0.0)) <= SVD_MIXED / nc);
    if (bad) *mixed = 1u;
}

// out[:, j] = sum_k left[:, k] right[k, j], all column-major: one tile of 32 columns x 32 rows per workgroup, the wavefronts split k.
//   SVD_TIMES    right as it is (B = A V)
//   SVD_NEWTON   right = 3/2 I - S / 2, S the Gram matrix of left's columns: the Newton step towards orthonormal columns; what
//                rounding left in unit vectors (place) and in their rows goes
//   SVD_CORRECT  right = I + K from the Gram matrix of left's columns; rows from split on go to out2
enum { SVD_TIMES, SVD_NEWTON, SVD_CORRECT };
template <int MODE, int WAVES, int U>
__device__ __forceinline__ void svd_product_tile(const double *left, const double *right, double *out, double *out2, int nr, int nc, int ld,
                                                 int ldr, int ldo, int ldo2, int split, double tol, int units, const int *place, int ti, int tj,
                                                 double (&part)[4][32][33])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4;
    const int j0 = tj * 32, i0 = ti * 32;
    f64x4_t acc[2][2];
    double gj[2] = {1.0, 1.0};
    const int unit = MODE == SVD_NEWTON ? place[min(i0 + (tid & 31), nc - 1)] : -1;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int j = j0 + 16 * a + c;
        if (MODE == SVD_CORRECT && j < nc) gj[a] = right[(i64)j * ldr + j];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[a][b][v] = 0.0;
    }
    struct Pieces {
        f64x2_t x[U][2], y[U][2], gk[U];
    };
    const auto fetch = [&](Pieces &p, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kk = k + 8 * u + 2 * g;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int row = min(i0 + 16 * a + c, nr - 1);
                p.x[u][a] = svd_frag(right, ldr, j0 + 16 * a + c, nc, kk, nc);
#pragma unroll
                for (int e = 0; e < 2; ++e) p.y[u][a][e] = left[(i64)min(kk + e, nc - 1) * ld + row];
            }
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (MODE == SVD_CORRECT) p.gk[u][e] = right[(i64)min(kk + e, nc - 1) * (ldr + 1)];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    const auto multiply = [&](const Pieces &p, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int kk = k + 8 * u + 2 * g + e;
                const bool in = kk < nc; // (columns and rows past the last give sums that nobody stores)
                double w[2], y[2];
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const int j = j0 + 16 * a + c;
                    w[a] = p.x[u][a][e];
                    if (MODE == SVD_NEWTON) w[a] = (j == kk ? 1.5 : 0.0) - 0.5 * w[a];
                    if (MODE == SVD_CORRECT) w[a] = j == kk ? 0.0 : svd_small_rotation(p.gk[u][e], gj[a], w[a], tol * tol);
                    w[a] = svd_masked(w[a], in);
                    y[a] = svd_masked(p.y[u][a][e], in);
                }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[a], y[b], acc[a][b], 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int STEP = 8 * WAVES * U;
    Pieces p0, p1;
    fetch(p0, 8 * U * wave);
    for (int k = 8 * U * wave; k < nc; k += 2 * STEP) {
        fetch(p1, k + STEP);
        multiply(p0, k);
        fetch(p0, k + 2 * STEP);
        if (k + STEP < nc) multiply(p1, k + STEP);
    }
    svd_tile_out<WAVES>(acc, part, [&](int jj, int ii, double s) {
        const int j = j0 + jj, i = i0 + ii;
        if (j >= nc || i >= nr) return;
        if (MODE == SVD_NEWTON && (unit >= 0 || j < units)) s = unit == j ? 1.0 : 0.0; // (ii is tid & 31)
        if (MODE == SVD_CORRECT) s += left[(i64)j * ld + i];
        if (MODE == SVD_CORRECT && i >= split)
            out2[(i64)j * ldo2 + i - split] = s;
        else
            out[(i64)j * ldo + i] = s;
    });
}

template <int MODE>
__global__ __launch_bounds__(256) void svd_product_kernel(const double *left, const double *right, double *out, int nr, int nc, int ld, int ldr,
                                                                 int ldo, const SvdCtrl *ctrl, const int *place)
{
    __shared__ double part[4][32][33];
    if (MODE == SVD_TIMES && ctrl->mixed) return;
    svd_product_tile<MODE, 4, SVD_U>(left, right, out, nullptr, nr, nc, ld, ldr, ldo, 0, 0, 0.0, MODE == SVD_NEWTON ? (int)ctrl->isolated : 0, place,
                                  blockIdx.x, blockIdx.y, part);
}

// L[:, j] /= |L[:, j]|, also into the V part of BV (rows v0 ..), by NT threads
template <int NT>
__device__ __forceinline__ void svd_normalise(double *L, double *BV, int j, int nc, int ldl, int ldb, int v0, double *red)
{
    const int tid = threadIdx.x;
    double *a = L + (i64)j * ldl, *b = BV + (i64)j * ldb;
    double acc = 0.0;
    for (int i = tid; tid < 256 && i < nc; i += 256) acc += a[i] * a[i];
    if (tid < 256) red[tid] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    const double n = sqrt(red[0]), inv = n > 0.0 ? 1.0 / n : 0.0;
    for (int i = tid; i < nc; i += NT) {
        a[i] *= inv;
        b[v0 + i] = a[i];
    }
    // (the padding row between the two parts, and the one below)
    if (tid == 0) {
        for (int i = v0 + nc; i < ldb; ++i) b[i] = 0.0;
    }
    __syncthreads();
}
__global__ __launch_bounds__(256) void svd_normalise_kernel(double *L, double *BV, int nc, int ldl, int ldb, int v0)
{
    __shared__ double red[256];
    svd_normalise<256>(L, BV, blockIdx.x, nc, ldl, ldb, v0, red);
}

// ------------------------------------------------------------------ grid barrier
// Every workgroup of a cooperative launch is resident, so all of them arrive.  The wait is bounded all the same (SvdPatience);
// false: some workgroup gave up, and everyone leaves.  sweeping (nullable): the others are sweeping, this counter is that of their barrier,
// and polls are 10 us apart (of 124 waiting workgroups, at two a microsecond beside 132 sweeping ones, the barriers of these took a quarter longer).
// shared: what others read was stored for them (agent scope), and has only to be complete.
__device__ __forceinline__ bool svd_grid_barrier(unsigned *arrived, unsigned *failed, unsigned &generation, unsigned nwg, const unsigned *sweeping = nullptr,
                                                 bool shared = false)
{
    __shared__ int ok;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
    __syncthreads();
    if (threadIdx.x == 0) {
        if (!shared) __threadfence(); // what this workgroup wrote is visible before it arrives
        generation += nwg;
        __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        SvdPatience patience;
        bool good, others = true;
        do {
            good = (int)(__hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - generation) >= 0;
            if (good) break;
            if (sweeping) {
#pragma unroll
                for (int i = 0; i < 3; ++i) __builtin_amdgcn_s_sleep(127);
            } else {
                __builtin_amdgcn_s_sleep(1);
            }
        } while (patience.goes_on([&] {
                     others = __hip_atomic_load(failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
                     return sweeping ? __hip_atomic_load(sweeping, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
                 }) &&
                 others);
        if (!good) __hip_atomic_store(failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence(); // and what the others wrote before they arrived is read afresh
        ok = good;
    }
    __syncthreads();
    return ok != 0;
}

// ------------------------------------------------------------------ one pair of blocks
// Rounds of eight disjoint pairs of the 16 columns.  Rounds 0 .. 7 pair every column of the first block with one of the
// second; rounds 8 .. 14 the columns within the blocks, four pairs in each (round-robin of eight).
__host__ __device__ constexpr int svd_in_block(int t, int q, bool second)
{
    return second ? (q == 0 ? 7 : (t + q) % 7) : (q == 0 ? t % 7 : (t - q + 7) % 7);
}
__host__ __device__ constexpr int svd_inner_lo(int t, int q)
{
    if (t < 8) return q;
    const int a = svd_in_block(t - 8, q & 3, false), b = svd_in_block(t - 8, q & 3, true);
    return (q >> 2) * 8 + (a < b ? a : b);
}
__host__ __device__ constexpr int svd_inner_hi(int t, int q)
{
    if (t < 8) return 8 + ((q + t) & 7);
    const int a = svd_in_block(t - 8, q & 3, false), b = svd_in_block(t - 8, q & 3, true);
    return (q >> 2) * 8 + (a < b ? b : a);
}

struct SvdShared {
    double part[SVD_NT / 64][16][17];
    double g[16][17];
    f64x2_t cs[120];
    int any[4];
};

template <int T, int END>
__device__ __forceinline__ void svd_rotate_row(const f64x2_t *cs, double (&x)[16])
{
    if constexpr (T < END) {
        asm volatile("" ::: "memory"); // (the rotations are read round by round, not all kept in registers)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            constexpr int t = T;
            const int lo = svd_inner_lo(t, q), hi = svd_inner_hi(t, q);
            const f64x2_t r = cs[8 * t + q];
            const double u = x[lo], v = x[hi];
            x[lo] = r[0] * u - r[1] * v;
            x[hi] = r[1] * u + r[0] * v;
        }
        svd_rotate_row<T + 1, END>(cs, x);
    }
}

// Blocks p and q of M (columns 8 p .., 8 q ..): every column of one against every column of the other, with `within` also
// the pairs inside the blocks.  Inner products over rows [0, nr), rotations applied to rows [0, rows).  Thread 0 returns how many
// pairs were rotated; large_pair: some pair was farther from orthogonal than SVD_SMALL.  known (nullable): the Gram matrix of all
// columns as it was before this sweep; where it says that every pair is orthogonal nothing is read.
constexpr double SVD_SMALL = 3e-8; // rotations this small leave their square: orthogonal to rounding level
__device__ __forceinline__ int svd_block_pair(double *M, int ld, int nc, int nr, int rows, int p, int q, bool within, double tol, SvdShort few,
                                              SvdShared &sh, bool &large_pair, bool &held_pair, const double *known, int ldk)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4;
    constexpr int NW = SVD_NT / 64;
    const auto column = [&](int k) { return (k < SVD_B ? SVD_B * p : SVD_B * q - SVD_B) + k; };
    const auto candidate = [&](int i, int j) { return i > j && (within || (i >= 8 && j < 8)); };
    if (known) {
        const int i = tid >> 4 & 15, j = tid & 15, ci = column(i), cj = column(j);
        const bool some = candidate(i, j) && ci < nc && cj < nc &&
                          !svd_orthogonal(known[(i64)ci * ldk + ci], known[(i64)cj * ldk + cj], known[(i64)cj * ldk + ci], tol * tol, few.nil, few.low);
        if (!__syncthreads_or(some)) return 0;
    }
    // Gram matrix, rows dealt to the wavefronts eight at a time, eight pieces in flight; the rows that this thread will
    // rotate come along
    double x[16];
    const auto fetch = [&](int row) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int cc = column(k);
            x[k] = cc < nc && row < rows ? M[(i64)cc * ld + row] : 0.0;
        }
    };
    f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
    const int col = column(c);
    for (int r = 8 * wave; r < nr; r += 8 * NW * 8) {
        f64x2_t y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) y[u] = svd_frag(M, ld, col, nc, r + 8 * NW * u + 2 * g, nr);
        __builtin_amdgcn_sched_barrier(0);
        if (r < 8 * NW) fetch(tid);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const double v = svd_masked(y[u][e], col < nc && r + 8 * NW * u + 2 * g + e < nr);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, acc, 0, 0, 0);
            }
        }
    }
    if (8 * wave >= nr) fetch(tid); // (fewer rows than wavefronts)
#pragma unroll
    for (int v = 0; v < 4; ++v) sh.part[wave][g + 4 * v][c] = acc[v];
    __syncthreads();
    const double tol2 = tol * tol;
    if (tid < 256) { // entry (i, j), and whether the pair needs a rotation
        const int i = tid >> 4, j = tid & 15;
        double y = 0.0, a = 0.0, b = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            y += sh.part[w][i][j];
            a += sh.part[w][i][i];
            b += sh.part[w][j][j];
        }
        sh.g[i][j] = y;
        const bool some = candidate(i, j) && !svd_orthogonal(a, b, y, tol2, few.nil, few.low), large = some && y * y > SVD_SMALL * SVD_SMALL * (a * b);
        const bool held = few.low > 0.0 && candidate(i, j) && !some && !svd_orthogonal(a, b, y, tol2, few.nil);
        const bool anyone = __any(some), anylarge = __any(large), anyheld = __any(held);
        if (lane == 0) sh.any[wave] = (anyone ? 1 : 0) | (anylarge ? 2 : 0) | (anyheld ? 4 : 0);
    }
    __syncthreads();
    const int any = sh.any[0] | sh.any[1] | sh.any[2] | sh.any[3];
    large_pair = any & 2;
    held_pair = any & 4;
    if (!(any & 1)) return 0;
    int rotations = 0;
    if (wave == 0) {
        // lane (a, b) owns the four entries where row pair a meets column pair b
        const int a = lane >> 3, b = lane & 7, rounds = within ? 15 : 8;
        for (int t = 0; t < rounds; ++t) {
            const int i0 = svd_inner_lo(t, a), i1 = svd_inner_hi(t, a), j0 = svd_inner_lo(t, b), j1 = svd_inner_hi(t, b);
            const double g00 = sh.g[i0][j0], g01 = sh.g[i0][j1], g10 = sh.g[i1][j0], g11 = sh.g[i1][j1];
            const f64x2_t rb = svd_rotation(sh.g[j0][j0], sh.g[j1][j1], sh.g[j0][j1], tol2, few.nil, few.low);
            f64x2_t ra; // that of row pair a: lane (0, a) has it
            ra[0] = __shfl(rb[0], a, 64);
            ra[1] = __shfl(rb[1], a, 64);
            if (a == 0) sh.cs[8 * t + b] = rb;
            rotations += __popcll(__ballot(a == 0 && !(rb[1] == 0.0)));
            const double h00 = ra[0] * g00 - ra[1] * g10, h10 = ra[1] * g00 + ra[0] * g10;
            const double h01 = ra[0] * g01 - ra[1] * g11, h11 = ra[1] * g01 + ra[0] * g11;
            __builtin_amdgcn_wave_barrier(); // (all lanes have read before any writes)
            sh.g[i0][j0] = rb[0] * h00 - rb[1] * h01;
            sh.g[i0][j1] = rb[1] * h00 + rb[0] * h01;
            sh.g[i1][j0] = rb[0] * h10 - rb[1] * h11;
            sh.g[i1][j1] = rb[1] * h10 + rb[0] * h11;
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    for (int row = tid; row < rows; row += SVD_NT) {
        if (row != tid) fetch(row);
        svd_rotate_row<0, 8>(sh.cs, x);
        if (within) svd_rotate_row<8, 15>(sh.cs, x);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int cc = column(k);
            if (cc < nc) __hip_atomic_store(&M[(i64)cc * ld + row], x[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    return rotations;
}

// At most `most` sweeps, until one rotates nothing -- or, with `quick`, nothing but small angles.  Returns false when a barrier
// gave up.
__device__ __forceinline__ bool svd_sweeps(double *M, int ld, int nc, int nr, int rows, double tol, SvdShort few, int most, unsigned *arrived,
                                           unsigned &generation, unsigned *rot, bool quick, SvdCtrl *ctrl, SvdShared &sh,
                                           int *ran, unsigned nwg, const double *known = nullptr, int ldk = 0)
{
    const int nbl = ((nc + SVD_B - 1) / SVD_B + 1) / 2 * 2, m1 = nbl - 1;
    int sweep = 0;
    for (; sweep < most; ++sweep) {
        for (int round = 0; round < m1; ++round) {
            for (int k = blockIdx.x; k < nbl / 2; k += nwg) {
                int p = k == 0 ? m1 : (round + k) % m1, q = k == 0 ? round % m1 : (round - k + m1) % m1;
                if (p > q) {
                    const int t = p;
                    p = q;
                    q = t;
                }
                bool large = false, held = false;
                const int did = svd_block_pair(M, ld, nc, nr, rows, p, q, round == 0, tol, few, sh, large, held, sweep == 0 ? known : nullptr, ldk);
                if (held && threadIdx.x == 0) __hip_atomic_store(&ctrl->held[sweep], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (did > 0 && (large || !quick) && threadIdx.x == 0)
                    __hip_atomic_fetch_add(&rot[sweep], (unsigned)did, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __syncthreads(); // (the LDS tables are used again)
            }
            if (!svd_grid_barrier(arrived, &ctrl->failed, generation, nwg, nullptr, true)) return false;
        }
        if (__hip_atomic_load(&rot[sweep], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) {
            if (few.low > 0.0 && __hip_atomic_load(&ctrl->held[sweep], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                few.low = 0.0; // the short columns' turn
                continue;
            }
            ++sweep;
            break;
        }
    }
    *ran = sweep;
    return true;
}

// G (overwritten) -> L with G + shift I = L L^T, sixteen columns at a time.
// By workgroups 0 .. nwg - 1; false: a barrier gave up.
__device__ __forceinline__ bool svd_factorize(double *G, double *L, SvdCtrl *ctrl, int nc, int ld, double rel, unsigned nwg, unsigned &generation, double *red)
{
    __shared__ double d[16][17];
    __shared__ double shift_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4;
    // the shift: rounding level of the largest diagonal entry (read by every workgroup before anyone changes G)
    {
        double m = 0.0;
        for (int i = tid; i < nc; i += SVD_NT) m = fmax(m, G[(i64)i * ld + i]);
        red[tid] = m;
        __syncthreads();
        if (tid == 0) {
            for (int i = 1; i < SVD_NT; ++i) m = fmax(m, red[i]);
            shift_s = m > 0.0 ? rel * m : 1.0;
        }
        __syncthreads();
    }
    const double shift = shift_s;
    if (!svd_grid_barrier(&ctrl->arrived[0], &ctrl->failed, generation, nwg)) return false;
    for (int p0 = 0; p0 < nc; p0 += 16) {
        const int w = min(16, nc - p0);
        // the diagonal block, by every workgroup
        if (tid < 256) {
            const int i = tid & 15, j = tid >> 4;
            d[i][j] = i < w && j < w ? G[(i64)(p0 + j) * ld + p0 + i] + (i == j ? shift : 0.0) : (i == j ? 1.0 : 0.0);
        }
        __syncthreads();
        for (int k = 0; k < 16; ++k) {
            const int i = tid & 15, j = tid >> 4;
            const double piv = d[k][k], s = piv > 0.0 ? 1.0 / sqrt(piv) : 0.0;
            double u = 0.0;
            if (tid < 256 && i >= j && j > k) u = d[i][j] - (d[i][k] * s) * (d[j][k] * s);
            double col = 0.0;
            if (tid < 256 && j == k && i >= k) col = d[i][k] * s;
            __syncthreads();
            if (tid < 256 && i >= j && j > k) d[i][j] = u;
            if (tid < 256 && j == k && i >= k) d[i][k] = col;
            __syncthreads();
        }
        // rows below: X = G[rows, block] d^-T, one row per thread over all workgroups
        for (i64 r = p0 + (i64)blockIdx.x * SVD_NT + tid; r < nc; r += (i64)nwg * SVD_NT) {
            double x[16];
            if (r < p0 + w) {
                for (int j = 0; j < w; ++j) L[(i64)(p0 + j) * ld + r] = r - p0 >= j ? d[r - p0][j] : 0.0;
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    asm volatile("" ::: "memory"); // (row j of d is read now, not all of d kept in registers)
                    double v = j < w ? G[(i64)(p0 + j) * ld + r] : 0.0;
#pragma unroll
                    for (int k = 0; k < j; ++k) v -= x[k] * d[j][k];
                    const double piv = d[j][j];
                    x[j] = piv > 0.0 ? v / piv : 0.0;
                    if (j < w) L[(i64)(p0 + j) * ld + r] = x[j];
                }
            }
        }
        for (i64 e = (i64)blockIdx.x * SVD_NT + tid; e < (i64)p0 * w; e += (i64)nwg * SVD_NT)
            L[(p0 + e / p0) * ld + e % p0] = 0.0; // above the diagonal block
        if (!svd_grid_barrier(&ctrl->arrived[0], &ctrl->failed, generation, nwg)) return false;
        // trailing blocks: G_ij -= X_i X_j^T, one 16 x 16 tile per wavefront
        const int n0 = p0 + 16, nt = n0 < nc ? (nc - n0 + 15) / 16 : 0;
        for (i64 t = (i64)blockIdx.x * (SVD_NT / 64) + wave; t < (i64)nt * nt; t += (i64)nwg * (SVD_NT / 64)) {
            const int ti = (int)(t / nt), tj = (int)(t % nt);
            if (tj > ti) continue;
            const int gi = n0 + 16 * ti, gj = n0 + 16 * tj;
            f64x4_t acc;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = gi + g + 4 * v, j = gj + c;
                acc[v] = i < nc && j < nc ? G[(i64)j * ld + i] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int kc = p0 + 4 * k + g;
                const double a = kc < nc && gi + c < nc ? L[(i64)kc * ld + gi + c] : 0.0;
                const double b = kc < nc && gj + c < nc ? L[(i64)kc * ld + gj + c] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-a, b, acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = gi + g + 4 * v, j = gj + c;
                if (i < nc && j < nc) G[(i64)j * ld + i] = acc[v];
            }
        }
        if (!svd_grid_barrier(&ctrl->arrived[0], &ctrl->failed, generation, nwg)) return false;
    }
    return true;
}

// The preconditioner alone, for more columns than the eigenvectors take: in the kernel below its loops have fewer registers (2200 x 2100: 139 ms
// a call, 115 so; 1024 x 256 with values down to 1e-6 of the largest, whose eigenvectors do not do, 5.53 in it and 5.43 in launches of their own).
// And for few columns of many rows, whose products then have launches over the whole chip instead of eight workgroups.
__global__ __launch_bounds__(SVD_NT) void svd_jacobi_kernel(double *G, double *L, SvdCtrl *ctrl, int nc, int ld, double rel, double tol)
{
    __shared__ SvdShared sh;
    unsigned generation = 0;
    int ran = 0;
    if (svd_factorize(G, L, ctrl, nc, ld, rel, gridDim.x, generation, &sh.part[0][0][0]))
        (void)svd_sweeps(L, ld, nc, nc, nc, tol, SvdShort{0.0, 0.0}, SVD_MAX_SWEEPS, &ctrl->arrived[0], generation, ctrl->rot[0], true, ctrl, sh, &ran, gridDim.x);
}

// What an ordinary call does not need, in one launch: a cooperative one costs 22 us around it even if it has nothing to do, and a launch
// that leaves at once 2 to 5.  (Three of the first and six of the second took their places before: 2048 x 512 1356 -> 1302 us a call, 576 x 64
// 266 -> 205, 320 x 240 604 -> 550.)  Jacobi as the preconditioner, where the eigenvectors do not do (ctrl->mixed) or were not formed, and B from it; the
// correction B (I + K) or, where K is too large, one sweep over the pairs of blocks that have pairs to rotate (a preconditioned basis usually
// leaves few, by rounding: 2048 x 512 13.2 -> 11.9 ms, where a sweep over everything and another that finds nothing followed); a second
// check, and sweeps over everything.  The sweeps' workgroups are one per pair of blocks, the first `sweepers`; products are dealt to all.
struct SvdRest {
    double *At, *G, *L, *BV;
    SvdCtrl *ctrl;
    int nr, nc, lda, ldn, ldb, sweepers, jacobi; // jacobi: there is no B yet, whatever ctrl->mixed says
    double tol, tol_v, rel;
};
__global__ __launch_bounds__(SVD_NT) void svd_rest_kernel(SvdRest a)
{
    SvdCtrl *ctrl = a.ctrl;
    const int nr = a.nr, nc = a.nc, tiles = (nc + 31) / 32, wg = blockIdx.x, nwg = gridDim.x;
    const bool jacobi = a.jacobi || ctrl->mixed;
    unsigned found = ctrl->violations[0], coarse = ctrl->coarse[0], later = 0u;
    bool ok = ctrl->failed == 0u;
    int ran = 0, before = 1; // sweeps; before them
    SvdShort few = {0.0, 0.0};
    if (ok && (jacobi || found)) {
        __shared__ SvdShared sh;
        __shared__ double part[4][32][33];
        double *red = &part[0][0][0];
        constexpr int W = SVD_NT / 64;
        unsigned everyone = 0;
        const auto meet = [&](const unsigned *sweeping = nullptr) { return svd_grid_barrier(&ctrl->everyone, &ctrl->failed, everyone, nwg, sweeping); };
        const auto gram = [&](const double *M, int ld) {
            for (int t = wg; t < tiles * tiles; t += nwg) {
                if (t % tiles > t / tiles) continue;
                svd_gram_tile<W, 1>(M, a.G, nr, nc, ld, a.ldn, t / tiles, t % tiles, (int *)nullptr, part);
                __syncthreads(); // (the sums' LDS is used again)
            }
        };
        const auto counted = [&](const unsigned *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        // Sweeps of L, of B where the first check found pairs, of B where the second did
#pragma unroll 1
        for (int stage = jacobi ? 0 : 1; ok && stage < 3; ++stage) {
            const bool first = stage == 0;
            if (first) {
                gram(a.At, a.lda);
                ok = meet();
            }
            const unsigned now = first ? 1u : stage == 1 ? found : later;
            if (!ok || now == 0u) break;
            // (half of all pairs or more: another check would only say that there are some left)
            const bool many = stage == 1 && coarse && found > (unsigned)nc * (nc - 1) / 4u;
            if (many) later = found, stage = 2;
            const int crew = svd_crew(stage, nc, a.sweepers);
            const bool swept = stage != 1 || coarse;
            if (swept) {
                few = SvdShort{0.0, 0.0};
                if (!first) {
                    double longest = 0.0;
                    for (int j = threadIdx.x; j < nc; j += SVD_NT) longest = fmax(longest, a.G[(i64)j * a.ldn + j]);
                    for (int s = 32; s > 0; s >>= 1) longest = fmax(longest, __shfl_xor(longest, s, 64));
                    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = longest;
                    __syncthreads();
#pragma unroll
                    for (int w = 0; w < W; ++w) longest = fmax(longest, red[w]);
                    __syncthreads();
                    few = svd_short(longest);
                }
                unsigned generation = 0;
                if (wg < crew && first) // (a call of its own: what it has no use for goes)
                    ok = svd_factorize(a.G, a.L, ctrl, nc, a.ldn, a.rel, a.sweepers, generation, red) &&
                         svd_sweeps(a.L, a.ldn, nc, nc, nc, a.tol_v, SvdShort{0.0, 0.0}, SVD_MAX_SWEEPS, &ctrl->arrived[0], generation, ctrl->rot[0], true, ctrl,
                                    sh, &ran, a.sweepers);
                else if (wg < crew)
                    ok = svd_sweeps(a.BV, a.ldb, nc, nr, a.ldb, a.tol, few, stage == 1 ? 1 : SVD_MAX_SWEEPS - 1 + many, &ctrl->arrived[stage], generation,
                                    ctrl->rot[stage], false, ctrl, sh, &ran, crew, stage == 1 || many ? a.G : nullptr, a.ldn);
                before = many ? 0 : 1;
                if (stage == 2) break;
            } else { // (into At and L, and back)
                const int down = (a.ldb + 31) / 32;
                for (int t = wg; t < down * tiles; t += nwg) {
                    svd_product_tile<SVD_CORRECT, W, 1>(a.BV, a.G, a.At, a.L, a.ldb, nc, a.ldb, a.ldn, a.lda, a.ldn, a.lda, a.tol, 0, nullptr, t % down,
                                                     t / down, part);
                    __syncthreads();
                }
                ok = meet();
                for (int j = wg; ok && j < nc; j += nwg)
                    for (int i = threadIdx.x; i < a.ldb; i += SVD_NT)
                        a.BV[(i64)j * a.ldb + i] = i < a.lda ? a.At[(i64)j * a.lda + i] : a.L[(i64)j * a.ldn + i - a.lda];
            }
            ok = ok && meet(swept && wg >= crew ? &ctrl->arrived[stage] : nullptr);
            if (first) {
                for (int j = wg; ok && j < nc; j += nwg) svd_normalise<SVD_NT>(a.L, a.BV, j, nc, a.ldn, a.ldb, a.lda, red);
                ok = ok && meet();
                const int down = (a.lda + 31) / 32;
                for (int t = wg; ok && t < down * tiles; t += nwg) {
                    svd_product_tile<SVD_TIMES, W, 1>(a.At, a.BV + a.lda, a.BV, nullptr, a.lda, nc, a.lda, a.ldb, a.ldb, 0, 0, 0.0, 0, nullptr, t % down,
                                                   t / down, part);
                    __syncthreads();
                }
                ok = ok && meet();
            }
            if (ok) gram(a.BV, a.ldb);
            ok = ok && meet();
            for (int j = wg; ok && j < nc; j += nwg)
                svd_check_column(a.G, &ctrl->violations[stage], &ctrl->coarse[stage], j, nc, a.ldn, a.tol, red);
            ok = ok && meet();
            if (first) found = counted(&ctrl->violations[0]), coarse = counted(&ctrl->coarse[0]);
            else later = counted(&ctrl->violations[1]);
            if (!first) few = SvdShort{0.0, 0.0};
        }
    }
    if (wg == 0 && threadIdx.x == 0) {
        // (a check that found nothing counts as one clean sweep)
        ctrl->sweeps = !ok ? SVD_MAX_SWEEPS : found == 0u ? 1 : later == 0u ? 2 : before + ran;
        ctrl->last = !ok ? 1u : later == 0u ? 0u : ctrl->rot[2][ran - 1];
        ctrl->nil = few.nil;
    }
}

__global__ __launch_bounds__(256) void svd_sigma_kernel(const double *At, double *sig, SvdCtrl *ctrl, int nr, int ld)
{
    const double *a = At + (i64)blockIdx.x * ld;
    double acc = 0.0;
    for (int i = threadIdx.x; i < nr; i += 256) acc += a[i] * a[i];
    __shared__ double red[256];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sig[blockIdx.x] = red[0] < ctrl->nil ? 0.0 : sqrt(red[0]);
        if (!(red[0] < __builtin_huge_val())) ctrl->broken = 1u; // (also a matrix of one column, which has no pairs)
    }
}

// position of column j in descending order of singular value (ties: lower index first; NaN before all others)
__global__ __launch_bounds__(256) void svd_rank_kernel(const double *sig, int *rank, int nc)
{
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63; // a wavefront per column (a thread: 63 us at 512)
    if (j >= nc) return;
    const double s = sig[j];
    int k = 0;
    for (int i = 0; i < nc; i += 64) k += __popcll(__ballot(i + lane < nc && svd_before(sig[min(i + lane, nc - 1)], i + lane, s, j)));
    if (lane == 0) rank[j] = k;
}

// column j of B (= sigma_j x left vector) and of V (right vector, from row v0 on) -> column rank[j] of the balanced factors
__global__ __launch_bounds__(256) void svd_emit_kernel(const double *BV, const double *sig, const int *rank, float *U, float *V,
                                                        float *sigma_out, int nr, int nc, int v0, int ld, int r,
                                                        int transposed, const SvdCtrl *ctrl, int *info)
{
    const SvdOutcome done = svd_outcome(*ctrl, nc);
    if (info && blockIdx.x == 0 && threadIdx.x == 0) {
        info[0] = done.sweeps;
        info[1] = done.last;
    }
    const int j = blockIdx.x, k = done.lost ? j : rank[j];
    const double s = done.lost ? __builtin_nan("") : sig[j];
    if (threadIdx.x == 0 && sigma_out) sigma_out[k] = (float)s;
    if (k >= r) return;
    const double rs = sqrt(s), inv = done.lost ? s : s > 0.0 ? rs / s : 0.0;
    float *left = transposed ? V : U, *right = transposed ? U : V;
    const double *a = BV + (i64)j * ld, *qv = a + v0;
    for (int i = threadIdx.x; i < nr; i += 256) left[(i64)i * r + k] = (float)(a[i] * inv);
    for (int i = threadIdx.x; i < nc; i += 256) right[(i64)i * r + k] = (float)(qv[i] * rs);
}

struct SvdPlan {
    int nr, nc, transposed, lda, ldn, ldb; // leading dimensions are even: columns are read two rows at a time
    size_t n_At, n_G, n_BV, bytes;
};
static int plan_svd(const pf_svd_desc *d, SvdPlan *p)
{
    if (!d) return PF_ERR_NULL;
    if (d->m <= 0 || d->n <= 0 || d->r <= 0) return PF_ERR_SHAPE;
    const i64 mn = d->m < d->n ? d->m : d->n, mx = d->m < d->n ? d->n : d->m;
    if (d->r > mn) return PF_ERR_SHAPE;
    if (mn > 8192 || mx > (1 << 24) || mn * mx > (1LL << 31)) return PF_ERR_UNSUPPORTED;
    p->transposed = d->m < d->n;
    p->nr = (int)mx;
    p->nc = (int)mn;
    p->lda = (p->nr + 1) / 2 * 2;
    p->ldn = (p->nc + 1) / 2 * 2;
    p->ldb = p->lda + p->ldn;
    p->n_At = (size_t)p->nc * p->lda;
    p->n_G = (size_t)p->nc * p->ldn;
    p->n_BV = (size_t)p->nc * p->ldb;
    p->bytes = align_up(p->n_At * 8) + 2 * align_up(p->n_G * 8) + align_up(p->n_BV * 8) + align_up((size_t)mn * 8) +
               align_up((size_t)mn * 4) + align_up(sizeof(SvdCtrl));
    return PF_OK;
}

} // namespace pf

using namespace pf;

extern "C" {

size_t pf_svd_split_workspace_bytes(const pf_svd_desc *d)
{
    SvdPlan p;
    return plan_svd(d, &p) == PF_OK ? p.bytes : 0;
}

int pf_svd_split(const pf_svd_desc *d, const void *W, void *U, void *V_out, void *sigma, void *info, void *workspace,
                 size_t workspace_bytes, void *stream)
{
    SvdPlan p;
    int st = plan_svd(d, &p);
    if (st != PF_OK) return st;
    if (!W || !U || !V_out) return PF_ERR_NULL;
    if (any_misaligned({W, U, V_out, sigma, info}, 4)) return PF_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < p.bytes) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    Workspace ws(workspace, workspace_bytes);
    hipStream_t s = (hipStream_t)stream;
    double *At = ws.take<double>(p.n_At), *G = ws.take<double>(p.n_G), *L = ws.take<double>(p.n_G);
    double *BV = ws.take<double>(p.n_BV), *sig = ws.take<double>(p.nc);
    int *rank = ws.take<int>(p.nc);
    SvdCtrl *ctrl = ws.take<SvdCtrl>(1);
    const int nc = p.nc, nr = p.nr;
    const i64 cells = (i64)nc * p.lda;
    PF_LAUNCH(st, "svd_init", svd_init_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), s, (const float *)W, At, ctrl, rank,
              (int)d->n, nr, nc, p.lda, p.transposed);
    const dim3 gram((nc + 31) / 32, (nc + 31) / 32);
    double *V = BV + p.lda; // (leading dimension ldb, as B's)
    const dim3 square((nc + 31) / 32, (nc + 31) / 32);
    const unsigned *none = nullptr;
    // V: eigenvectors of G made orthonormal; where they cannot be (ctrl->mixed), and for few or very many columns, by Jacobi
    const int cus = cooperative_cus();
    const bool eigen = svd_takes_eigenvectors(nc, cus);
    if (eigen) {
        int *const place = rank; // (before the ranks are there)
        PF_LAUNCH(st, "svd_gram", svd_gram_kernel, gram, dim3(256), s, (const double *)At, G, nr, nc, p.lda, p.ldn, none, place);
        if (st == PF_OK) st = launch_svd_eigenvectors(s, G, L, sig, BV, place, ctrl, nc, p.ldn);
        PF_LAUNCH(st, "svd_gram", svd_gram_kernel, gram, dim3(256), s, (const double *)BV, G, nc, nc, p.ldn, p.ldn, none, (int *)nullptr);
        PF_LAUNCH(st, "svd_newton", svd_product_kernel<SVD_NEWTON>, square, dim3(256), s, (const double *)BV, (const double *)G, L, nc, nc, p.ldn,
                  p.ldn, p.ldn, (const SvdCtrl *)ctrl, (const int *)place);
        PF_LAUNCH(st, "svd_gram", svd_gram_kernel, gram, dim3(256), s, (const double *)L, G, nc, nc, p.ldn, p.ldn, none, (int *)nullptr);
        PF_LAUNCH(st, "svd_mixed", svd_mixed_kernel, dim3(nc), dim3(256), s, (const double *)G, &ctrl->mixed, nc, p.ldn);
        PF_LAUNCH(st, "svd_newton", svd_product_kernel<SVD_NEWTON>, square, dim3(256), s, (const double *)L, (const double *)G, V, nc, nc, p.ldn,
                  p.ldn, p.ldb, (const SvdCtrl *)ctrl, (const int *)place);
    }
    // sweeps: one workgroup per pair of blocks (at least eight for the factorization); products: one per tile; all of them resident
    const int pairs = ((nc + SVD_B - 1) / SVD_B + 1) / 2, sweepers = pairs < 8 ? 8 : pairs > 256 ? 256 : pairs;
    const i64 tiles = (i64)((p.lda + 31) / 32) * ((nc + 31) / 32);
    const int most = cus > 256 ? 256 : cus, wide = tiles < most ? (int)tiles : most;
    const double rel = 16.0 * 2.220446049250313e-16 * (nc + 16);
    // Few columns, us a call, Jacobi and products in the kernel below / in launches of their own: 1024 x 16 185 / 193, 2048 x 16 204 / 205, 4608 x 16 283 /
    // 272, 16384 x 16 597 / 517, 65536 x 16 1920 / 1568, 1048576 x 16 29.2 / 23.2 ms.
    const bool jacobi = !eigen && (nc > SVD_EIGEN_MAX || nr > 2048);
    if (jacobi) {
        PF_LAUNCH(st, "svd_gram", svd_gram_kernel, gram, dim3(256), s, (const double *)At, G, nr, nc, p.lda, p.ldn, none, (int *)nullptr);
        if (st == PF_OK)
            st = launch_cooperative(s, "svd_jacobi", svd_jacobi_kernel, sweepers, SVD_NT, G, L, ctrl, nc, p.ldn, rel, svd_tolerance_v(nc));
        PF_LAUNCH(st, "svd_normalise", svd_normalise_kernel, dim3(nc), dim3(256), s, L, BV, nc, p.ldn, p.ldb, p.lda);
    }
    if (eigen || jacobi) {
        PF_LAUNCH(st, "svd_apply", svd_product_kernel<SVD_TIMES>, dim3((p.lda + 31) / 32, (nc + 31) / 32), dim3(256), s, (const double *)At,
                  (const double *)V, BV, p.lda, nc, p.lda, p.ldb, p.ldb, (const SvdCtrl *)ctrl, (const int *)nullptr);
        PF_LAUNCH(st, "svd_gram", svd_gram_kernel, gram, dim3(256), s, (const double *)BV, G, nr, nc, p.ldb, p.ldn, (const unsigned *)&ctrl->mixed,
                  (int *)nullptr);
        PF_LAUNCH(st, "svd_check", svd_check_kernel, dim3(nc), dim3(256), s, (const double *)G, ctrl, nc, p.ldn, svd_tolerance(nr));
    }
    const SvdRest rest = {At, G, L, BV, ctrl, nr, nc, p.lda, p.ldn, p.ldb, sweepers, !eigen && !jacobi, svd_tolerance(nr), svd_tolerance_v(nc), rel};
    if (st == PF_OK) st = launch_cooperative(s, "svd_rest", svd_rest_kernel, (eigen || jacobi) && wide > sweepers ? wide : sweepers, SVD_NT, rest);
    PF_LAUNCH(st, "svd_sigma", svd_sigma_kernel, dim3(nc), dim3(256), s, (const double *)BV, sig, ctrl, nr, p.ldb);
    PF_LAUNCH(st, "svd_rank", svd_rank_kernel, dim3((nc + 3) / 4), dim3(256), s, (const double *)sig, rank, nc);
    PF_LAUNCH(st, "svd_emit", svd_emit_kernel, dim3(nc), dim3(256), s, (const double *)BV, (const double *)sig,
              (const int *)rank, (float *)U, (float *)V_out, (float *)sigma, nr, nc, p.lda, p.ldb, (int)d->r, p.transposed,
              (const SvdCtrl *)ctrl, (int *)info);
    return st;
}

} // extern "C"
