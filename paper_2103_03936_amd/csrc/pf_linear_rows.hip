// Fused fully connected low-rank layer for few rows (bf16, rank 128): see launch_linear_rows in pf_linear_chain.h.
//
// A decoding step has 32 to a few hundred rows: with one workgroup of four wavefronts per 32 rows (linear_chain2_kernel) most of
// the chip is idle and each wavefront waits out every load of its chain.  Here 32 rows and 128 outputs are a workgroup of sixteen
// wavefronts, so four workgroups share the outputs of a 512-wide layer; each forms the whole rank-r intermediate for itself (all of
// W1, 128 KB, comes from L2).
//   stage 1: wavefront (rank block, quarter of the contraction): W1 passes through LDS as it lies in memory, in whole rows (as the
//            32 columns of one wavefront, half a cache line a row, 64 KB take 1.4 us), and comes back by transposing reads; what is
//            needed first is requested before anything is waited for
//   stage 2: wavefront (output block, quarter of the rank); its W2 fragments are in registers since the start
// The four quarters of either contraction meet in LDS in a fixed order.
// 64 rows, 512 -> 128 -> 512: 6.2 us a call, 7.0 before; 256 -> 1024: 5.0, 8.9; 512 -> 2048: 6.1, 9.5.  Bound by W1's way into one
// compute unit, 1.2 us per 64 KB, and by launch, first load and two sums over LDS, 3.7 us.
#include "pf_linear_chain.h"

namespace pf {

typedef unsigned int u32x4_r __attribute__((ext_vector_type(4), may_alias));
typedef unsigned int u32x2_r __attribute__((ext_vector_type(2), may_alias));

constexpr int LR_R = 128, LR_NT = 1024, LR_OUT = 128; // rank, threads, outputs per workgroup
constexpr int LR_VP = LR_R + 16;                      // LDS pitch (elements) of a chunk of W1, 64 rows of every quarter
constexpr int LR_TP = LR_R + 8, LR_RP = 36;           // of the intermediate; of a partial sum [32][32] (floats)

__device__ __forceinline__ bf16x8_t lr_frag(u32x4_r v) { return __builtin_bit_cast(bf16x8_t, v); }

// C1 = 256 NCH
template <int NCH>
__global__ __launch_bounds__(LR_NT, 4) void linear_rows_kernel(LinChainArgs a)
{
    constexpr int C1 = 256 * NCH, XP = C1 + 8;
    constexpr int chunk = 256 * LR_VP * 2, part = 16 * 32 * LR_RP * 4;
    __shared__ __attribute__((aligned(16))) uint16_t Xs[32 * XP];
    __shared__ __attribute__((aligned(16))) uint16_t Ts[32 * LR_TP];
    __shared__ __attribute__((aligned(16))) unsigned char raw[chunk > part ? chunk : part];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, half = lane >> 5, col = lane & 31;
    const int block = w & 3, quarter = w >> 2;
    const i64 row0 = (i64)blockIdx.x * 32;
    const int o0 = blockIdx.y * LR_OUT, group = blockIdx.z;
    const uint16_t *in = a.in + group * a.gs_in, *W1 = a.W1 + group * a.gs_W1, *W2 = a.W2 + group * a.gs_W2;

    u32x4_r xr[NCH], vr[2][4], ur[2];
#pragma unroll
    for (int i = 0; i < NCH; ++i) { // the rows, C1 / 8 pieces each
        const int e = tid + LR_NT * i, r = e / (C1 / 8), c = e - r * (C1 / 8);
        const i64 row = row0 + r < a.rows ? row0 + r : a.rows - 1; // (rows past the end: the last one, never stored)
        xr[i] = *(const u32x4_r *)(in + row * C1 + 8 * c);
    }
    const uint16_t *v = W1 + (i64)(quarter * (C1 / 4) + 16 * block + (lane >> 4)) * LR_R + 8 * (lane & 15);
    const auto fetch = [&](int c, int set) {
#pragma unroll
        for (int i = 0; i < 4; ++i) vr[set][i] = *(const u32x4_r *)(v + (i64)(64 * c + 4 * i) * LR_R);
    };
    fetch(0, 0);
    if (NCH > 1) fetch(1, 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) ur[j] = *(const u32x4_r *)(W2 + (i64)(o0 + 32 * block + col) * LR_R + 32 * quarter + 16 * j + 8 * half);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int e = tid + LR_NT * i, r = e / (C1 / 8), c = e - r * (C1 / 8);
        *(u32x4_r *)&Xs[r * XP + 8 * c] = xr[i];
    }
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    uint16_t *Vs = (uint16_t *)raw;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if (c > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) *(u32x4_r *)&Vs[(16 * w + 4 * i + (lane >> 4)) * LR_VP + 8 * (lane & 15)] = vr[c & 1][i];
        if (c + 2 < NCH) fetch(c + 2, c & 1);
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const u32x4_r x = *(const u32x4_r *)&Xs[col * XP + quarter * (C1 / 4) + 64 * c + 16 * ks + 8 * half];
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag_tr(Vs, LR_VP, 64 * quarter + 16 * ks, 32 * block, lane), lr_frag(x), acc, 0, 0, 0);
        }
    }
    // a wavefront's tile: lane holds row `col`, columns 8 q + 4 half + 0..3
    float *red = (float *)raw;
    const auto put = [&]() {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *(f32x4_t *)&red[(w * 32 + col) * LR_RP + 8 * q + 4 * half] = f32x4_t{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    };
    // thread: row r, columns 4 g .. 4 g + 3 of the 128; sum of the four quarters
    const int r = tid >> 5, g = tid & 31;
    const auto sum = [&]() {
        const float *p = &red[((g >> 3) * 32 + r) * LR_RP + 4 * (g & 7)];
        constexpr int Q = 4 * 32 * LR_RP;
        return (*(const f32x4_t *)p + *(const f32x4_t *)(p + Q)) + (*(const f32x4_t *)(p + 2 * Q) + *(const f32x4_t *)(p + 3 * Q));
    };
    __syncthreads(); // (the partial sums lie where W1 was)
    put();
    __syncthreads();
    {
        const f32x4_t t = sum();
        const u32x2_r pk = {pack_bf16x2(t[0], t[1]), pack_bf16x2(t[2], t[3])};
        *(u32x2_r *)&Ts[r * LR_TP + 4 * g] = pk;
        if (a.mid_save && blockIdx.y == 0 && row0 + r < a.rows) *(u32x2_r *)(a.mid_save + group * a.gs_mid + (row0 + r) * LR_R + 4 * g) = pk;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const u32x4_r t = *(const u32x4_r *)&Ts[col * LR_TP + 32 * quarter + 16 * j + 8 * half];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lr_frag(ur[j]), lr_frag(t), acc, 0, 0, 0);
    }
    put();
    __syncthreads();
    if (row0 + r >= a.rows) return;
    f32x4_t y = sum();
    const i64 at = (row0 + r) * a.C2 + o0 + 4 * g;
    const auto plus = [&](const uint16_t *p) {
        const u32x2_r b = *(const u32x2_r *)p;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] += bf16_bits_to_float((uint16_t)(b[e >> 1] >> (16 * (e & 1))));
    };
    if (a.bias) plus(a.bias + group * a.gs_bias + o0 + 4 * g);
    if (a.ep_add) plus(a.ep_add + at);
    if (a.ep_relu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = fmaxf(y[e], 0.f);
    }
    *(u32x2_r *)(a.out + group * a.gs_out + at) = u32x2_r{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
}

bool linear_rows_supported(i64 n_in, i64 n_out, i64 r)
{
    return linear_chain2_supported(n_in, n_out, r) && n_in <= 1024 && n_out <= (1 << 16);
}

int launch_linear_rows(hipStream_t s, const char *name, const LinChainArgs &a)
{
    int st = PF_OK;
    if (a.rows <= 0) return st;
    const int groups = a.groups > 1 ? a.groups : 1;
    const i64 tiles = (a.rows + 31) / 32;
    if (!linear_rows_supported(a.C1, a.C2, LR_R) || a.ep_mask || a.colsum || groups > LC_MAX_GROUPS || tiles > (1 << 20)) return PF_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)tiles, a.C2 / LR_OUT, groups), block(LR_NT);
    switch (a.C1 / 256) {
    case 1: PF_LAUNCH(st, name, linear_rows_kernel<1>, grid, block, s, a); break;
    case 2: PF_LAUNCH(st, name, linear_rows_kernel<2>, grid, block, s, a); break;
    case 3: PF_LAUNCH(st, name, linear_rows_kernel<3>, grid, block, s, a); break;
    default: PF_LAUNCH(st, name, linear_rows_kernel<4>, grid, block, s, a); break;
    }
    return st;
}

} // namespace pf
