// Factorized linear layer in fp32 for a small batch (M <= 128 rows; the fully connected layers of a CNN head,
// Section 2.1): two launches per direction.
//
// At these sizes one product has too little work for the chip unless the long contraction (in or out, hundreds)
// is cut into slices, and every slice needs its own compute unit: the fp32 matrix instruction gives one compute
// unit 0.6 TFLOP/s.  So
//   launch 1 (ls_slices_kernel):   P[s] = X[:, slice s] V[slice s, :]   (32 x 32 tiles x S slices of the contraction)
//   launch 2 (ls_tiles_kernel):    every tile of every product that reads T = sum_s P[s]:  Y = T U^T + b forward;
//                                  dX = dT V^T, dU = dY^T T, dV = X^T dT, db backward (dT from its slices)
// and the slice sum is taken where an operand is staged in LDS, not by a launch of its own.  The rank-r intermediate
// crosses launches as S slices of M x r floats that stay in the last-level cache.
#include "pf_linear_small.h"

namespace pf {

constexpr int LS_PITCH = 33; // floats between the k rows of a staged operand tile (32 values + 1 against conflicts)
// Eight wavefronts per workgroup: a slice of 128 contraction indices is then two pieces per wavefront, and four slices do where four
// wavefronts needed eight, which every workgroup of the second launch reads (64 x 512 -> 128 -> 512, forward 3.4 + 8.4 us).
constexpr int LS_W = 8, LS_NT = 64 * LS_W;

__device__ __forceinline__ float ls_sum(const float (&red)[LS_W][32 * LS_PITCH], int at)
{
    return ((red[0][at] + red[1][at]) + (red[2][at] + red[3][at])) + ((red[4][at] + red[5][at]) + (red[6][at] + red[7][at]));
}

// ----------------------------------------------------------------- launch 1
// P[s][m][n] = sum over k in slice s of A[m][k] W[k][n]; grid (N / 32, row blocks, S).  The eight wavefronts are dealt the slice
// eight contraction indices at a time and add their tiles in LDS.
__global__ __launch_bounds__(LS_NT) void ls_slices_kernel(LsSliceArgs a0, LsSliceArgs a1)
{
    const LsSliceArgs a = blockIdx.z >= (unsigned)a0.S ? a1 : a0;
    const int s = blockIdx.z >= (unsigned)a0.S ? blockIdx.z - a0.S : blockIdx.z;
    const int ct = blockIdx.x, rb = blockIdx.y;
    if (ct * 32 >= a.N) return; // (the two problems may differ in width)
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, half = lane >> 5, col = lane & 31;
    const int KS = a.K / a.S;
    const int row = rb * 32 + col;
    const float *Ar = a.A + (i64)(row < a.M ? row : a.M - 1) * a.lda + s * KS + 4 * half;
    const float *Wc = a.W + (i64)(s * KS + 4 * half) * a.ldw + ct * 32 + col;
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    for (int kb = 8 * w; kb < KS; kb += 16 * LS_W) { // lane half h holds k = kb + 4 h + 0..3; two pieces in flight
        const int kc = min(kb + 8 * LS_W, KS - 8);
        f32x4_t av[2];
        float bv[2][4];
        av[0] = *(const f32x4_t *)(Ar + kb);
        av[1] = *(const f32x4_t *)(Ar + kc);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bv[0][j] = Wc[(i64)(kb + j) * a.ldw];
            bv[1][j] = Wc[(i64)(kc + j) * a.ldw];
        }
        if (kb + 8 * LS_W >= KS) { // (a piece past the end is someone else's; both factors are zeroed, for either may be infinite)
#pragma unroll
            for (int j = 0; j < 4; ++j) av[1][j] = bv[1][j] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(row < a.M ? av[u][j] : 0.f, bv[u][j], acc, 0, 0, 0);
    }
    __shared__ float red[LS_W][32 * LS_PITCH];
#pragma unroll
    for (int v = 0; v < 16; ++v) red[w][(8 * (v >> 2) + 4 * half + (v & 3)) * LS_PITCH + col] = acc[v];
    __syncthreads();
    float *P = a.P + (i64)s * a.M * a.N;
#pragma unroll
    for (int i = 0; i < 1024 / LS_NT; ++i) {
        const int e = tid + LS_NT * i, m = e >> 5, n = e & 31;
        if (rb * 32 + m < a.M) P[(i64)(rb * 32 + m) * a.N + ct * 32 + n] = ls_sum(red, m * LS_PITCH + n);
    }
}

// ----------------------------------------------------------------- launch 2
// One 32 x 32 output tile per workgroup: C[m][n] = sum_k A(m, k) B(k, n), k < K <= LS_MAX_K.  Both operands are
// staged in LDS k-major (element (k, i) at k * 33 + i), read from memory along their fast index:
//   LS_MK: element (i, k) at p[i * ld + k]   (a row-major activation, or U / V read as the right operand)
//   LS_KM: element (i, k) at p[k * ld + i]   (dY or X as the left operand of a factor gradient; T as the right one)
// and either may be the sum of `slices` slices `sstride` floats apart.
// A thread has two 16-byte pieces of either operand; all their slices are requested before the first is looked at (a slice past the
// end re-reads the first and counts zero times; slices are added in order).
template <bool SL>
struct LsPieces {
    static constexpr int NP = 32 * LS_MAX_K / 4 / LS_NT, NS = SL ? LS_MAX_SLICES : 1;
    f32x4_t v[NP][NS];
    bool mk, live[NP];
    int k[NP], i[NP], slices;

    __device__ __forceinline__ void load(const LsOperand &o, int i0, int ni, int K, int tid)
    {
        mk = o.layout == LS_MK;
        slices = o.slices;
        const int k4n = K >> 2, total = 8 * K; // (K and ni are multiples of 4 where it matters)
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int e = min(tid + LS_NT * q, total - 1);
            const int r = mk ? e / k4n : e >> 3;
            i[q] = mk ? r : 4 * (e & 7);      // consecutive threads along k (piece = 4 k of row i) ..
            k[q] = mk ? 4 * (e - r * k4n) : r; // .. or along i (piece = 4 i of row k)
            live[q] = i0 + i[q] < ni;
            const int ii = live[q] ? i0 + i[q] : i0;
            const float *p = o.p + (mk ? (i64)ii * o.ld + k[q] : (i64)k[q] * o.ld + ii);
#pragma unroll
            for (int s = 0; s < NS; ++s) v[q][s] = *(const f32x4_t *)(p + (i64)(s < slices ? s : 0) * o.sstride);
        }
    }
    __device__ __forceinline__ void stage(float *dst)
    {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            f32x4_t t = v[q][0];
#pragma unroll
            for (int s = 1; s < NS; ++s) {
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] += s < slices ? v[q][s][j] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) dst[mk ? (k[q] + j) * LS_PITCH + i[q] : k[q] * LS_PITCH + i[q] + j] = live[q] ? t[j] : 0.f;
        }
    }
};

template <bool SA, bool SB>
__device__ __forceinline__ void ls_stage(const LsTileProb &pr, int m0, int n0, float *As, float *Bs, int tid)
{
    LsPieces<SA> a;
    LsPieces<SB> b;
    a.load(pr.A, m0, pr.M, pr.K, tid);
    b.load(pr.B, n0, pr.N, pr.K, tid);
    a.stage(As);
    b.stage(Bs);
}

__global__ __launch_bounds__(LS_NT) void ls_tiles_kernel(LsTileArgs a)
{
    // which problem does this workgroup belong to?
    int q = 0;
#pragma unroll
    for (int i = 1; i < LS_MAX_PROB; ++i)
        if (i < a.nprob && (int)blockIdx.x >= a.p[i].wg0) q = i;
    const LsTileProb &pr = a.p[q];
    const int t = blockIdx.x - pr.wg0, nt = (pr.N + 31) / 32;
    const int m0 = 32 * (t / nt), n0 = 32 * (t % nt);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, half = lane >> 5, col = lane & 31;
    __shared__ float As[LS_MAX_K * LS_PITCH], Bs[LS_MAX_K * LS_PITCH];
    __shared__ float red[LS_W][32 * LS_PITCH];
    const int K = pr.K;
    if (pr.A.slices > 1) // (uniform; no product has both operands in slices)
        ls_stage<true, false>(pr, m0, n0, As, Bs, tid);
    else if (pr.B.slices > 1)
        ls_stage<false, true>(pr, m0, n0, As, Bs, tid);
    else
        ls_stage<false, false>(pr, m0, n0, As, Bs, tid);
    __syncthreads();
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    // wavefront w takes k = 2 (8 j + w) + half: the k pairs are dealt round the eight wavefronts, four in flight
    for (int kp = w; 2 * kp < K; kp += 4 * LS_W) {
        float av[4], bv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = 2 * (kp + LS_W * u) + half;
            av[u] = k < K ? As[k * LS_PITCH + col] : 0.f;
            bv[u] = k < K ? Bs[k * LS_PITCH + col] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[u], bv[u], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) red[w][(8 * (v >> 2) + 4 * half + (v & 3)) * LS_PITCH + col] = acc[v];
    if (pr.A_copy && n0 == 0) { // the summed left operand leaves once (T for the backward pass): [M][K]
        for (int e = tid; e < 32 * K; e += LS_NT) {
            const int i = e / K, k = e - i * K;
            if (m0 + i < pr.M) pr.A_copy[(i64)(m0 + i) * K + k] = As[k * LS_PITCH + i];
        }
    }
    if (pr.colsum && n0 == 0 && tid < 32 && m0 + tid < pr.M) { // sum of the left operand over k (a bias gradient)
        float part[4] = {0.f, 0.f, 0.f, 0.f}; // four running sums: the LDS reads do not wait for one another
        for (int k = 0; k < K; k += 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) part[j] += k + j < K ? As[(k + j) * LS_PITCH + tid] : 0.f;
        }
        const float sum = (part[0] + part[1]) + (part[2] + part[3]);
        pr.colsum[m0 + tid] = pr.accumulate ? pr.colsum[m0 + tid] + sum : sum;
    }
    __syncthreads();
    if (!pr.C) return;
#pragma unroll
    for (int i = 0; i < 1024 / LS_NT; ++i) {
        const int e = tid + LS_NT * i, m = e >> 5, n = e & 31;
        if (m0 + m < pr.M && n0 + n < pr.N) {
            float v = ls_sum(red, m * LS_PITCH + n);
            if (pr.bias) v += pr.bias[n0 + n];
            float *c = pr.C + (i64)(m0 + m) * pr.ldc + n0 + n;
            *c = pr.accumulate ? *c + v : v;
        }
    }
}

bool linear_small_supported(i64 M, i64 n_in, i64 n_out, i64 r)
{
    return M > 0 && M <= LS_MAX_K && r <= LS_MAX_K && n_in % 32 == 0 && n_out % 32 == 0 && r % 32 == 0 && n_in >= 32 &&
           n_out >= 32 && r >= 32 && n_in <= (1 << 20) && n_out <= (1 << 20);
}

int linear_small_slices(i64 K)
{
    for (int s = LS_MAX_SLICES; s > 1; s >>= 1)
        if (K % (32 * s) == 0) return s;
    return 1;
}

int launch_ls_slices(hipStream_t s, const char *name, const LsSliceArgs &a0, const LsSliceArgs &a1)
{
    int st = PF_OK;
    const int n = a0.N > a1.N ? a0.N : a1.N, m = a0.M > a1.M ? a0.M : a1.M;
    if (n <= 0 || m <= 0) return st;
    const dim3 grid((unsigned)(n / 32), (unsigned)((m + 31) / 32), (unsigned)(a0.S + a1.S));
    PF_LAUNCH(st, name, ls_slices_kernel, grid, dim3(LS_NT), s, a0, a1);
    return st;
}

void ls_add(LsTileArgs &a, const LsOperand &A, const LsOperand &B, int M, int N, int K, float *C, i64 ldc, const float *bias,
            int accumulate, float *A_copy, float *colsum)
{
    LsTileProb &p = a.p[a.nprob++];
    p.A = A;
    p.B = B;
    p.M = M;
    p.N = N;
    p.K = K;
    p.C = C;
    p.ldc = ldc;
    p.bias = bias;
    p.accumulate = accumulate;
    p.A_copy = A_copy;
    p.colsum = colsum;
    p.wg0 = a.nwg;
    a.nwg += ((M + 31) / 32) * ((N + 31) / 32);
}

int launch_ls_tiles(hipStream_t s, const char *name, const LsTileArgs &a)
{
    int st = PF_OK;
    if (a.nwg <= 0) return st;
    PF_LAUNCH(st, name, ls_tiles_kernel, dim3((unsigned)a.nwg), dim3(LS_NT), s, a);
    return st;
}

} // namespace pf
