// Factorized LSTM cell (paper Section 2.3, eq. (2)): one time step forward and one step of
// back-propagation through time.  Host-side validation, workspace planning and dispatch;
// the any-shape path composes the guarded tile GEMM with two pointwise kernels.
#include "pf_gemm.h"
#include "pf_skinny.h"
#include "pf_tile_plans.h"

namespace pf {

__device__ __forceinline__ float sigmoidf_acc(float z) { return 1.0f / (1.0f + expf(-z)); }

// z[B x 4h] pre-activations (i|f|g|o) -> gates, c, h
__global__ __launch_bounds__(256) void lstm_pointwise_fwd_kernel(const float *z, const float *bias, const float *c_prev,
                                                                  float *h_out, float *c_out, float *gates, int B, int h)
{
    const i64 idx = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (i64)B * h) return;
    const int b = (int)(idx / h), j = (int)(idx % h);
    const i64 base = (i64)b * 4 * h + j;
    const float b0 = bias ? bias[j] : 0.f, b1 = bias ? bias[j + h] : 0.f, b2 = bias ? bias[j + 2 * (i64)h] : 0.f,
                b3 = bias ? bias[j + 3 * (i64)h] : 0.f;
    const float ig = sigmoidf_acc(z[base] + b0), fg = sigmoidf_acc(z[base + h] + b1);
    const float gg = tanhf(z[base + 2 * (i64)h] + b2), og = sigmoidf_acc(z[base + 3 * (i64)h] + b3);
    const float c = fg * c_prev[idx] + ig * gg;
    gates[base] = ig;
    gates[base + h] = fg;
    gates[base + 2 * (i64)h] = gg;
    gates[base + 3 * (i64)h] = og;
    c_out[idx] = c;
    h_out[idx] = og * tanhf(c);
}

// dh, dc_next -> dz[B x 4h] (gradient at the pre-activations), dc_prev
__global__ __launch_bounds__(256) void lstm_pointwise_bwd_kernel(const float *gates, const float *c_prev,
                                                                  const float *c_out, const float *dh,
                                                                  const float *dc_next, float *dz, float *dc_prev, int B,
                                                                  int h)
{
    const i64 idx = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (i64)B * h) return;
    const int b = (int)(idx / h), j = (int)(idx % h);
    const i64 base = (i64)b * 4 * h + j;
    const float ig = gates[base], fg = gates[base + h], gg = gates[base + 2 * (i64)h], og = gates[base + 3 * (i64)h];
    const float tc = tanhf(c_out[idx]);
    const float dhv = dh[idx];
    const float dc = (dc_next ? dc_next[idx] : 0.f) + dhv * og * (1.f - tc * tc);
    dc_prev[idx] = dc * fg;
    dz[base] = dc * gg * ig * (1.f - ig);
    dz[base + h] = dc * c_prev[idx] * fg * (1.f - fg);
    dz[base + 2 * (i64)h] = dc * ig * (1.f - gg * gg);
    dz[base + 3 * (i64)h] = dhv * tc * og * (1.f - og);
}

// A(m, k, gate): [Tx | Th] of the gate's group, k in [0, 2r)
struct OpA_LstmT {
    const float *Tx, *Th;
    int r, gr, goff; // goff = r for groups == 4, 0 for groups == 1
    __device__ __forceinline__ float operator()(int m, int k, int gate) const
    {
        const i64 base = (i64)m * gr + (i64)gate * goff;
        return k < r ? Tx[base + k] : Th[base + k - r];
    }
};
// B(k, n, gate): [Ux | Uh] row gate * h + n
struct OpB_LstmU {
    const float *Ux, *Uh;
    int r, h;
    __device__ __forceinline__ float operator()(int k, int n, int gate) const
    {
        const i64 row = (i64)gate * h + n;
        return k < r ? Ux[row * r + k] : Uh[row * r + k - r];
    }
};

static int check_lstm_desc(const pf_lstm_desc *d)
{
    if (!d) return PF_ERR_NULL;
    if (d->dtype != PF_F32) return PF_ERR_UNSUPPORTED;
    if (d->groups != 1 && d->groups != 4) return PF_ERR_UNSUPPORTED;
    if (d->B < 0 || d->d_in <= 0 || d->h <= 0 || d->r <= 0) return PF_ERR_SHAPE;
    const i64 lim = 0x7fffffffLL;
    if (d->B > lim || d->d_in > lim || d->h * 4 > lim || d->r * 4 > lim) return PF_ERR_SHAPE;
    if (d->B * d->h * 4 > lim || d->B * d->d_in > lim) return PF_ERR_SHAPE;
    return PF_OK;
}

struct LstmPlan {
    size_t n_z, n_dT, fwd_bytes, bwd_bytes, n_part;
    // k-splits of the skinny products (the batch is a handful of rows, so the contraction is spread over the chip)
    int ks_Tx, ks_Th, ks_z, ks_dT, ks_dx, ks_dh;
};
static LstmPlan plan_lstm(const pf_lstm_desc *d)
{
    LstmPlan p;
    p.n_z = (size_t)(d->B * 4 * d->h);
    p.n_dT = (size_t)(d->B * d->groups * d->r);
    const i64 gr = (i64)d->groups * d->r, Kz = d->groups == 4 ? d->h : 4 * d->h, nb = d->groups == 4 ? 4 : 1;
    p.ks_Tx = choose_ksplit(d->B, gr, d->d_in);
    p.ks_Th = choose_ksplit(d->B, gr, d->h);
    p.ks_z = choose_ksplit(d->B, d->h, 2 * d->r, 4);
    p.ks_dT = choose_ksplit(d->B, d->r, Kz, (int)nb);
    p.ks_dx = choose_ksplit(d->B, d->d_in, gr);
    p.ks_dh = choose_ksplit(d->B, d->h, gr);
    size_t part = (size_t)colsum_chunks(d->B) * 4 * d->h;
    auto upd = [&](size_t n) {
        if (n > part) part = n;
    };
    upd((size_t)p.ks_Tx * d->B * gr);
    upd((size_t)p.ks_Th * d->B * gr);
    upd((size_t)p.ks_z * d->B * 4 * d->h);
    upd((size_t)p.ks_dT * d->B * gr);
    upd((size_t)p.ks_dx * d->B * d->d_in);
    upd((size_t)p.ks_dh * d->B * d->h);
    p.n_part = part;
    p.fwd_bytes = align_up(p.n_z * sizeof(float)) + align_up(p.n_part * sizeof(float));
    p.bwd_bytes = align_up(p.n_z * sizeof(float)) + 2 * align_up(p.n_dT * sizeof(float)) + align_up(p.n_part * sizeof(float));
    return p;
}

static int lstm_fwd_generic(const pf_lstm_desc *d, const float *x, const float *h_prev, const float *c_prev,
                            const float *Vx, const float *Ux, const float *Vh, const float *Uh, const float *bias,
                            float *h_out, float *c_out, float *gates, float *Tx, float *Th, Workspace &ws,
                            hipStream_t s)
{
    const int B = (int)d->B, din = (int)d->d_in, h = (int)d->h, r = (int)d->r, gr = d->groups * r;
    const LstmPlan p = plan_lstm(d);
    float *z = ws.take<float>(p.n_z);
    float *part = ws.take<float>(p.n_part);
    int st = launch_gemm_generic<float, true, false>("lstm_Tx=x*Vx", s, GemmShape{B, gr, din, 1, p.ks_Tx},
                                                     OpA_RowMajor<float>{x, din, 0}, OpB_KN<float>{Vx, gr, 0, 0},
                                                     EpiPartial{part, gr, (i64)B * gr});
    if (st == PF_OK) st = launch_splitk_reduce(s, part, Tx, (i64)B * gr, p.ks_Tx, 0);
    if (st != PF_OK) return st;
    st = launch_gemm_generic<float, true, false>("lstm_Th=h*Vh", s, GemmShape{B, gr, h, 1, p.ks_Th},
                                                 OpA_RowMajor<float>{h_prev, h, 0}, OpB_KN<float>{Vh, gr, 0, 0},
                                                 EpiPartial{part, gr, (i64)B * gr});
    if (st == PF_OK) st = launch_splitk_reduce(s, part, Th, (i64)B * gr, p.ks_Th, 0);
    if (st != PF_OK) return st;
    st = launch_gemm_generic<float, true, true>("lstm_z=[Tx|Th]*[Ux|Uh]t", s, GemmShape{B, h, 2 * r, 4, p.ks_z},
                                                OpA_LstmT{Tx, Th, r, gr, d->groups == 4 ? r : 0},
                                                OpB_LstmU{Ux, Uh, r, h},
                                                EpiPartial{part, 4 * (i64)h, (i64)B * 4 * h, h});
    if (st == PF_OK) st = launch_splitk_reduce(s, part, z, (i64)B * 4 * h, p.ks_z, 0);
    if (st != PF_OK) return st;
    dim3 grid((unsigned)(((i64)B * h + 255) / 256));
    PF_LAUNCH(st, "lstm_pointwise_fwd", lstm_pointwise_fwd_kernel, grid, dim3(256), s, z, d->has_bias ? bias : nullptr,
              c_prev, h_out, c_out, gates, B, h);
    return st;
}

static int lstm_bwd_generic(const pf_lstm_desc *d, const float *x, const float *h_prev, const float *c_prev,
                            const float *c_out, const float *gates, const float *Tx, const float *Th, const float *Vx,
                            const float *Ux, const float *Vh, const float *Uh, const float *dh, const float *dc_next,
                            float *dx, float *dh_prev, float *dc_prev, float *dVx, float *dUx, float *dVh, float *dUh,
                            float *dbias, int accumulate, Workspace &ws, hipStream_t s)
{
    const int B = (int)d->B, din = (int)d->d_in, h = (int)d->h, r = (int)d->r, G = d->groups, gr = G * r;
    const LstmPlan p = plan_lstm(d);
    float *dz = ws.take<float>(p.n_z);
    float *dTx = ws.take<float>(p.n_dT);
    float *dTh = ws.take<float>(p.n_dT);
    float *part = ws.take<float>(p.n_part);
    int st = PF_OK;
    if (B == 0) {
        if (!accumulate) {
            st = launch_zero_f32(s, dVx, (i64)din * gr);
            if (st == PF_OK) st = launch_zero_f32(s, dVh, (i64)h * gr);
            if (st == PF_OK) st = launch_zero_f32(s, dUx, (i64)4 * h * r);
            if (st == PF_OK) st = launch_zero_f32(s, dUh, (i64)4 * h * r);
            if (st == PF_OK) st = launch_zero_f32(s, dbias, (i64)4 * h);
        }
        return st;
    }
    dim3 grid((unsigned)(((i64)B * h + 255) / 256));
    PF_LAUNCH(st, "lstm_pointwise_bwd", lstm_pointwise_bwd_kernel, grid, dim3(256), s, gates, c_prev, c_out, dh,
              dc_next, dz, dc_prev, B, h);
    if (st != PF_OK) return st;
    // dT = dz U: one product over all 4h rows (groups == 1) or one per gate block (groups == 4)
    const int nb = G == 4 ? 4 : 1, Kz = G == 4 ? h : 4 * h;
    for (int path = 0; path < 2; ++path) {
        const float *U = path ? Uh : Ux;
        float *dT = path ? dTh : dTx;
        st = launch_gemm_generic<float, true, false>(path ? "lstm_dTh=dz*Uh" : "lstm_dTx=dz*Ux", s,
                                                     GemmShape{B, r, Kz, nb, p.ks_dT}, OpA_RowMajor<float>{dz, 4 * (i64)h, h},
                                                     OpB_KN<float>{U, r, h, 0}, EpiPartial{part, gr, (i64)B * gr, r});
        if (st == PF_OK) st = launch_splitk_reduce(s, part, dT, (i64)B * gr, p.ks_dT, 0);
        if (st != PF_OK) return st;
    }
    if (dx) {
        st = launch_gemm_generic<float, true, true>("lstm_dx=dTx*Vxt", s, GemmShape{B, din, gr, 1, p.ks_dx},
                                                    OpA_RowMajor<float>{dTx, gr, 0}, OpB_NK<float>{Vx, gr, 0},
                                                    EpiPartial{part, din, (i64)B * din});
        if (st == PF_OK) st = launch_splitk_reduce(s, part, dx, (i64)B * din, p.ks_dx, 0);
        if (st != PF_OK) return st;
    }
    st = launch_gemm_generic<float, true, true>("lstm_dh=dTh*Vht", s, GemmShape{B, h, gr, 1, p.ks_dh},
                                                OpA_RowMajor<float>{dTh, gr, 0}, OpB_NK<float>{Vh, gr, 0},
                                                EpiPartial{part, h, (i64)B * h});
    if (st == PF_OK) st = launch_splitk_reduce(s, part, dh_prev, (i64)B * h, p.ks_dh, 0);
    if (st != PF_OK) return st;
    // dU[gate rows, :] (+)= dz[:, gate rows]^T T[:, gate's group]
    for (int path = 0; path < 2; ++path) {
        const float *T = path ? Th : Tx;
        float *dU = path ? dUh : dUx;
        if (!dU) continue;
        st = launch_gemm_generic<float, false, false>(path ? "lstm_dUh=dzt*Th" : "lstm_dUx=dzt*Tx", s,
                                                      GemmShape{h, r, B, 4, 1}, OpA_ColMajor<float>{dz, 4 * (i64)h, h},
                                                      OpB_KN<float>{T, gr, 0, G == 4 ? r : 0},
                                                      EpiGrad{dU, r, h, 0, accumulate});
        if (st != PF_OK) return st;
    }
    if (dVx) {
        st = launch_gemm_generic<float, false, false>("lstm_dVx=xt*dTx", s, GemmShape{din, gr, B, 1, 1},
                                                      OpA_ColMajor<float>{x, din, 0}, OpB_KN<float>{dTx, gr, 0, 0},
                                                      EpiGrad{dVx, gr, 0, 0, accumulate});
        if (st != PF_OK) return st;
    }
    if (dVh) {
        st = launch_gemm_generic<float, false, false>("lstm_dVh=ht*dTh", s, GemmShape{h, gr, B, 1, 1},
                                                      OpA_ColMajor<float>{h_prev, h, 0}, OpB_KN<float>{dTh, gr, 0, 0},
                                                      EpiGrad{dVh, gr, 0, 0, accumulate});
        if (st != PF_OK) return st;
    }
    if (dbias) st = launch_colsum<float>(s, dz, part, dbias, B, 4 * (i64)h, 4 * (i64)h, accumulate);
    return st;
}


// z = bias + sum of the pre-activation slices, then the gate arithmetic of eq. (2)
// (zadd, nullable: pre-activations computed elsewhere, [B x 4h] -- the hoisted input path of a sequence)
__global__ __launch_bounds__(256) void lstm_slices_pointwise_fwd_kernel(const float *P, int nslices, i64 pcount,
                                                                         const float *bias, const float *zadd,
                                                                         const float *c_prev,
                                                                         float *h_out, float *c_out, float *gates, int B,
                                                                         int h)
{
    const i64 idx = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (i64)B * h) return;
    const int b = (int)(idx / h), j = (int)(idx % h);
    const i64 base = (i64)b * 4 * h + j;
    float z[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) z[g] = slices_at(P, nslices, pcount, base + (i64)g * h);
    if (bias) {
#pragma unroll
        for (int g = 0; g < 4; ++g) z[g] += bias[j + (i64)g * h];
    }
    if (zadd) {
#pragma unroll
        for (int g = 0; g < 4; ++g) z[g] += zadd[base + (i64)g * h];
    }
    const float ig = sigmoidf_acc(z[0]), fg = sigmoidf_acc(z[1]);
    const float gg = tanhf(z[2]), og = sigmoidf_acc(z[3]);
    const float c = fg * c_prev[idx] + ig * gg;
    gates[base] = ig;
    gates[base + h] = fg;
    gates[base + 2 * (i64)h] = gg;
    gates[base + 3 * (i64)h] = og;
    c_out[idx] = c;
    h_out[idx] = og * tanhf(c);
}

// ------------------------------------------------------------------ any batch, every extent at least four floats
// The products of a step on the tiled kernels (pf_tile.h), both paths (and the four gate blocks) side by side: forward
// T; z as two slices; gates.  Backward gate derivatives; dT; dx and dh_prev; all parameter gradients, the last two in one launch where that
// pays.  Products too small for the chip split their contraction; slices of T and dT are added by the tiles that read them, others by
// one more launch.  Forward and backward, us, factors in the caches, nine launches with streaming kernels for up to 32 rows before / now: 10 rows, 128
// units 36.4 / 19.2, 512 units 38.7 / 25.5 (a pair per gate 38.7 / 28.2), 1500 units, backward streamed, 61.1 / 55.9; 64 rows, 512 units 34.7 / 27.2.
static bool lstm_tiles_ok(const pf_lstm_desc *d) { return d->B > 0 && d->d_in >= 4 && d->h >= 4 && d->r >= 4; }

LstmTilePlan make_lstm_tile_plan(const pf_lstm_desc *d)
{
    LstmTilePlan p;
    const i64 B = d->B, h = d->h, r = d->r, G = d->groups, gr = G * r, din = d->d_in, rows = (B + 31) / 32 * 32;
    const TileNeed z[2] = {{B, 4 * h, r, false}, {B, 4 * h, r, false}};
    p.z = plan_tile_group(PF_F32, z, 2);
    const TileNeed T[2] = {{B, gr, din, true}, {B, gr, h, true}};
    p.T = plan_mid_group(PF_F32, T, 2, p.z.shape, 8 * rows * r * ((4 * h + 31) / 32), 128 * r);
    const TileNeed last[6] = {{B, din, gr, false}, {B, h, gr, false}, {4 * h, r, B, false}, {4 * h, r, B, false}, {din, gr, B, false}, {h, gr, B, false}};
    p.dxh = plan_tile_group(PF_F32, last, 2);
    const TileNeed dxh[2] = {{B, din, gr, true}, {B, h, gr, true}};
    const TileGroup split = plan_tile_group(PF_F32, dxh, 2);
    if (split.cost < p.dxh.cost) p.dxh = split;
    p.grads = plan_tile_group(PF_F32, last + 2, 4);
    p.last = plan_tile_group(PF_F32, last, 6);
    const TileNeed dT[2] = {{B, gr, G == 4 ? h : 4 * h, true}, {B, gr, G == 4 ? h : 4 * h, true}};
    const auto mid = [&](bool one) {
        return plan_mid_group(PF_F32, dT, 2, one ? p.last.shape : p.dxh.shape, 4 * rows * gr * ((din + 31) / 32 + (h + 31) / 32) * (one ? 2 : 1),
                              128 * (one && B > gr ? B : gr));
    };
    const MidGroup dT1 = mid(true), dT2 = mid(false);
    // One launch or two, each with the dT that its readers can take.  The tiles of dx and dh_prev are few and contract over all ranks: beside
    // the gradients' they are the longer for it.  (A launch costs 2000 clocks more than the 3000 that its plan has.)
    // Backward, us, one / two, factors in the caches: a pair per gate, 64 rows, 1500 units 91.9 / 86.8, 87 rows, 576 -> 1280 units 51.0 / 47.0, 188
    // rows, 448 units, rank 168 34.5 / 32.3, 200 rows, 448 -> 384 units 22.2 / 25.6; one pair, 7 rows, 768 units 19.7 / 21.6, 23 rows, 640 units
    // 18.0 / 20.1.  Over 550 cells of 1 to 256 rows 0.2 % from the faster one (geometric mean), six more than a
    // twentieth slower, three of which the streaming kernels take; out of the caches alike.
    const double chain = tile_chain_cost(PF_F32, p.last.shape, last, 6, 2), all = p.last.cost > chain ? p.last.cost : chain;
    const double in_one = all + dT1.g.cost, in_two = p.dxh.cost + p.grads.cost + dT2.g.cost + 2000;
    p.one = in_one < in_two;
    p.bwd = p.one ? in_one : in_two;
    p.dT = p.one ? dT1 : dT2;
    p.n_T = (size_t)((p.T.g.ksplit[0] + p.T.g.ksplit[1]) * B * gr) + 64;
    p.n_dT = (size_t)((p.dT.g.ksplit[0] + p.dT.g.ksplit[1]) * B * gr) + 64;
    p.n_dxh = (size_t)(p.dxh.ksplit[0] * B * din + p.dxh.ksplit[1] * B * h) + 64;
    const size_t nz = (size_t)(B * 4 * h);
    p.fwd_bytes = align_up(p.n_T * 4) + align_up(2 * nz * 4);
    p.bwd_bytes = align_up(nz * 4) + 2 * align_up((size_t)(B * gr) * 4) + align_up(p.n_dT * 4) + align_up(p.n_dxh * 4);
    return p;
}
static const LstmTilePlan &plan_lstm_tiles(const pf_lstm_desc *d)
{
    static thread_local PlanCache<PlanKey<5>, LstmTilePlan> cache;
    return cache.get(PlanKey<5>{{d->B, d->d_in, d->h, d->r, d->groups}}, [&] { return make_lstm_tile_plan(d); });
}

// Adds a product whose result is needed in full: straight to `out`, or through partial sums taken from `part`; sliced: these are what its
// readers take.
struct MidAt {
    float *p;
    int slices; // > 1: partial sums at p
};
static MidAt add_split(TileArgs &a, SplitSumArgs &ss, const TileGroup &g, int i, TileProb q, float *out, i64 count, float *&part,
                       bool sliced = false)
{
    const int ks = g.ksplit[i];
    MidAt at = {out, 1};
    q.o.f32 = 1;
    q.o.C = out;
    if (ks > 1) {
        q.o.C = part;
        q.o.split_stride = count;
    }
    tile_add(a, g.shape, PF_F32, q, ks);
    if (ks > 1) {
        const int got = a.p[a.n - 1].ksplit;
        if (sliced && got > 1) at = MidAt{part, got};
        else split_sum_add(ss, SplitSum{part, out, count, count, got, 0, nullptr, 0, 0});
        part += (ks * count + 3) / 4 * 4;
    }
    return at;
}

static int lstm_fwd_tiles(const pf_lstm_desc *d, const float *x, const float *h_prev, const float *c_prev, const float *Vx,
                          const float *Ux, const float *Vh, const float *Uh, const float *bias, float *h_out, float *c_out,
                          float *gates, float *Tx, float *Th, Workspace &ws, hipStream_t s)
{
    const int B = (int)d->B, din = (int)d->d_in, h = (int)d->h, r = (int)d->r, G = d->groups, gr = G * r;
    const LstmTilePlan p = plan_lstm_tiles(d);
    float *part = ws.take<float>(p.n_T), *z = ws.take<float>((size_t)2 * B * 4 * h);
    TileArgs a = {};
    SplitSumArgs ss = {};
    const MidAt T[2] = {
        add_split(a, ss, p.T.g, 0, tile_prob(TILE_NN, B, gr, din, x, din, Vx, gr, nullptr, gr), Tx, (i64)B * gr, part, p.T.sliced),
        add_split(a, ss, p.T.g, 1, tile_prob(TILE_NN, B, gr, h, h_prev, h, Vh, gr, nullptr, gr), Th, (i64)B * gr, part, p.T.sliced)};
    int st = launch_tiles_linear(s, "lstm_T=[x*Vx|h*Vh]", PF_F32, p.T.g.shape, a);
    if (st == PF_OK) st = launch_split_sums(s, ss);
    if (st != PF_OK) return st;
    TileArgs b = {};
    for (int path = 0; path < 2; ++path) {
        TileProb q = tile_prob(TILE_NT, B, G == 4 ? h : 4 * h, r, T[path].p, gr, path ? Uh : Ux, r, z + (i64)path * B * 4 * h, 4 * (i64)h);
        q.o.f32 = 1;
        if (T[path].slices > 1) q.aslices = T[path].slices, q.sstride = (i64)B * gr, q.acopy = path ? Th : Tx;
        if (G == 4) {
            q.nb = 4;
            q.sa = r;
            q.sb = (i64)h * r;
            q.sc = h;
        }
        tile_add(b, p.z.shape, PF_F32, q, 1);
    }
    st = launch_tiles_linear(s, "lstm_z=[Tx|Th]*[Ux|Uh]t", PF_F32, p.z.shape, b);
    if (st != PF_OK) return st;
    PF_LAUNCH(st, "lstm_pointwise_fwd", lstm_slices_pointwise_fwd_kernel, dim3((unsigned)(((i64)B * h + 255) / 256)), dim3(256),
              s, z, 2, (i64)B * 4 * h, d->has_bias ? bias : nullptr, (const float *)nullptr, c_prev, h_out, c_out, gates, B, h);
    return st;
}

static int lstm_bwd_tiles(const pf_lstm_desc *d, const float *x, const float *h_prev, const float *c_prev,
                          const float *c_out, const float *gates, const float *Tx, const float *Th, const float *Vx,
                          const float *Ux, const float *Vh, const float *Uh, const float *dh, const float *dc_next,
                          float *dx, float *dh_prev, float *dc_prev, float *dVx, float *dUx, float *dVh, float *dUh,
                          float *dbias, int accumulate, Workspace &ws, hipStream_t s)
{
    const int B = (int)d->B, din = (int)d->d_in, h = (int)d->h, r = (int)d->r, G = d->groups, gr = G * r;
    const LstmTilePlan p = plan_lstm_tiles(d);
    float *dz = ws.take<float>((size_t)B * 4 * h);
    float *dTx = ws.take<float>((size_t)B * gr), *dTh = ws.take<float>((size_t)B * gr);
    float *part = ws.take<float>(p.n_dT), *part_dxh = ws.take<float>(p.n_dxh);
    const bool sliced = p.dT.sliced && (p.one || dx); // (else the launch of dx and dh_prev leaves the sums for the gradients')
    MidAt dT[2];
    int st = PF_OK;
    PF_LAUNCH(st, "lstm_pointwise_bwd", lstm_pointwise_bwd_kernel, dim3((unsigned)(((i64)B * h + 255) / 256)), dim3(256), s,
              gates, c_prev, c_out, dh, dc_next, dz, dc_prev, B, h);
    if (st != PF_OK) return st;
    TileArgs a = {};
    SplitSumArgs ss = {};
    for (int path = 0; path < 2; ++path) { // dT = dz U: over all 4h columns, or per gate block
        TileProb q = tile_prob(TILE_NN, B, r, G == 4 ? h : 4 * h, dz, 4 * (i64)h, path ? Uh : Ux, r, nullptr, gr);
        if (G == 4) {
            q.nb = 4;
            q.sa = h;
            q.sb = (i64)h * r;
            q.sc = r;
        }
        dT[path] = add_split(a, ss, p.dT.g, path, q, path ? dTh : dTx, (i64)B * gr, part, sliced);
    }
    st = launch_tiles_linear(s, "lstm_dT=dz*[Ux|Uh]", PF_F32, p.dT.g.shape, a);
    if (st == PF_OK) st = launch_split_sums(s, ss);
    if (st != PF_OK) return st;
    TileArgs b = {}, c = {};
    SplitSumArgs sb = {};
    const TileGroup unsplit = {p.last.shape, {1, 1, 1, 1, 1, 1}, 0};
    const auto input = [&](int path, const float *V, int n, float *out) {
        TileProb q = tile_prob(TILE_NT, B, n, gr, dT[path].p, gr, V, gr, nullptr, n);
        if (dT[path].slices > 1) q.aslices = dT[path].slices, q.sstride = (i64)B * gr, q.acopy = p.one ? nullptr : path ? dTh : dTx;
        add_split(p.one ? c : b, sb, p.one ? unsplit : p.dxh, path, q, out, (i64)B * n, part_dxh);
    };
    if (dx) input(0, Vx, din, dx);
    input(1, Vh, h, dh_prev);
    if (!p.one) {
        st = launch_tiles_linear(s, "lstm_dxh=[dTx*Vxt|dTh*Vht]", PF_F32, p.dxh.shape, b);
        if (st == PF_OK) st = launch_split_sums(s, sb);
        if (st != PF_OK) return st;
    }
    const TileShape shape = p.one ? p.last.shape : p.grads.shape;
    const auto grad = [&](const float *A, i64 lda, int m, const float *Bm, i64 ldb, int n, float *out, float *sums) {
        TileProb q = tile_prob(TILE_TN, m, n, B, A, lda, Bm, ldb, out, n);
        q.o.f32 = 1;
        q.o.accumulate = accumulate;
        q.o.sums = sums;
        return q;
    };
    for (int path = 0; path < 2; ++path) {
        TileProb q = grad(dz, 4 * (i64)h, G == 4 ? h : 4 * h, path ? Th : Tx, gr, r, path ? dUh : dUx, path ? nullptr : dbias);
        if (G == 4) {
            q.nb = 4;
            q.sa = h;
            q.sb = r;
            q.sc = (i64)h * r;
            q.ssums = h;
        }
        tile_add(c, shape, PF_F32, q, 1);
    }
    for (int path = 0; path < 2; ++path) {
        const int m = path ? h : din;
        TileProb q = grad(path ? h_prev : x, m, m, path ? dTh : dTx, gr, gr, path ? dVh : dVx, nullptr);
        if (p.one && dT[path].slices > 1) q.B = dT[path].p, q.bslices = dT[path].slices, q.sstride = (i64)B * gr;
        tile_add(c, shape, PF_F32, q, 1);
    }
    return launch_tiles_linear(s, p.one ? "lstm_dxh,grads" : "lstm_grads", PF_F32, shape, c);
}

// ------------------------------------------------------------------ backward, few rows
// Every product streams its factor once from all compute units (pf_skinny.h); slice sums of dx and dh_prev ride along with the gradient
// updates.

// Both ways in microseconds, fitted to 300 cells of 1 to 32 rows and 128 to 1500 units (3 and 4 % rms; the means of factors in the caches and out
// of them).  Backward, us, here / tiled products, in the caches and out of them: a pair per gate, 2 rows, 1024 units 25.3 / 32.7 and 28.9 / 36.3, 20 rows 30.7
// / 33.0 and 34.0 / 36.4, 4 rows, 1296 units 34.6 / 43.1 and 40.7 / 46.3, 22 rows, 960 units 31.3 / 26.6 and 34.0 / 30.7; one pair, 4 rows, 1024 units, rank
// 453 28.0 / 34.2 and 32.0 / 36.7, 24 rows, 1216 units 32.7 / 27.9 and 35.6 / 30.0.  300 other cells: 0.4 % behind the
// faster one (geometric mean), two of them a twentieth or more in the caches, five out of them, 7 % at most.  Smaller layers: 10 rows, 512 units
// 20.9 / 13.4.
// (Every extent of the sliced products holds one 16-byte load: see launch_skinny_gemm.)
bool lstm_skinny_pays(const pf_lstm_desc *d)
{
    if (!lstm_tiles_ok(d) || d->B > SK_MAX_ROWS) return false;
    const LstmTilePlan &p = plan_lstm_tiles(d);
    const double B = (double)d->B, m = 1e-6 * ((double)d->groups * d->r * (d->d_in + d->h) + 8.0 * d->h * d->r); // millions of weights
    const double here = 19.3 + 2.26 * m + B * (0.18 + 0.031 * m);
    const double tiles = 7 + p.bwd / 1617 - 0.33 * m + (d->r % 4 ? 0.67 : 0) - (p.one ? 2.8 : 0);
    return here < 0.98 * tiles;
}

// The two launches with sliced contractions.  Each builder fills the problem list, places the slice sums
// from `part` on (NULL when only the size is wanted) and returns the number of floats they take.
// dT = dz U per path (per gate block when groups == 4)
static size_t build_dT(const pf_lstm_desc *d, const float *dz, const float *Ux, const float *Uh, float *part,
                       SkinnyArgs &a)
{
    const int B = (int)d->B, h = (int)d->h, r = (int)d->r, G = d->groups, gr = G * r;
    a = SkinnyArgs{};
    const i64 pc = (i64)B * gr;
    for (int path = 0; path < 2; ++path) {
        const float *U = path ? Uh : Ux;
        if (G == 1) {
            a.p[a.nprob++] = skinny_prob(B, dz, 4 * (i64)h, U, r, 4 * h, r, gr, pc);
        } else {
            for (int g = 0; g < 4; ++g)
                a.p[a.nprob++] = skinny_prob(B, dz ? dz + (i64)g * h : nullptr, 4 * (i64)h, U ? U + (i64)g * h * r : nullptr,
                                             r, h, r, gr, pc);
        }
    }
    skinny_plan(a);
    const int per = a.nprob / 2, ks = a.p[0].ksplit;
    for (int q = 0; q < a.nprob; ++q) {
        const int path = q / per, g = q % per;
        a.p[q].P = part ? part + (i64)(path ? ks : 0) * pc + (G == 4 ? (i64)g * r : 0) : nullptr;
    }
    return (size_t)(2 * ks * pc);
}

// dx = dTx Vx^T (skipped when dx == NULL and want_dx is false), dh_prev = dTh Vh^T
static size_t build_dxh(const pf_lstm_desc *d, bool want_dx, const float *dTx, const float *dTh, const float *Vx,
                        const float *Vh, float *part, SkinnyArgs &a)
{
    const int B = (int)d->B, h = (int)d->h, gr = (int)(d->groups * d->r), din = (int)d->d_in;
    a = SkinnyArgs{};
    if (want_dx) a.p[a.nprob++] = skinny_prob(B, dTx, gr, Vx, gr, gr, din, din, (i64)B * din);
    a.p[a.nprob++] = skinny_prob(B, dTh, gr, Vh, gr, gr, h, h, (i64)B * h);
    skinny_plan(a);
    size_t used = 0;
    for (int q = 0; q < a.nprob; ++q) {
        a.p[q].P = part ? part + used : nullptr;
        used += (size_t)(a.p[q].ksplit * a.p[q].pcount);
    }
    return used;
}

struct SkinnyLstmPlan {
    size_t n_part_bwd, bwd_bytes;
};
static SkinnyLstmPlan plan_lstm_skinny(const pf_lstm_desc *d)
{
    SkinnyLstmPlan p;
    SkinnyArgs a;
    const size_t b1 = build_dT(d, nullptr, nullptr, nullptr, nullptr, a);
    const size_t b2 = build_dxh(d, true, nullptr, nullptr, nullptr, nullptr, nullptr, a);
    p.n_part_bwd = b1 > b2 ? b1 : b2;
    p.bwd_bytes = align_up((size_t)(d->B * 4 * d->h) * sizeof(float)) +
                  2 * align_up((size_t)(d->B * d->groups * d->r) * sizeof(float)) +
                  align_up(p.n_part_bwd * sizeof(float));
    return p;
}

static int lstm_bwd_skinny(const pf_lstm_desc *d, const float *x, const float *h_prev, const float *c_prev,
                           const float *c_out, const float *gates, const float *Tx, const float *Th, const float *Vx,
                           const float *Ux, const float *Vh, const float *Uh, const float *dh, const float *dc_next,
                           float *dx, float *dh_prev, float *dc_prev, float *dVx, float *dUx, float *dVh, float *dUh,
                           float *dbias, int accumulate, Workspace &ws, hipStream_t s)
{
    const int B = (int)d->B, din = (int)d->d_in, h = (int)d->h, r = (int)d->r, G = d->groups, gr = G * r;
    const SkinnyLstmPlan p = plan_lstm_skinny(d);
    float *dz = ws.take<float>((size_t)B * 4 * h);
    float *dTx = ws.take<float>((size_t)B * gr);
    float *dTh = ws.take<float>((size_t)B * gr);
    float *part = ws.take<float>(p.n_part_bwd);
    int st = PF_OK;
    dim3 grid((unsigned)(((i64)B * h + 255) / 256));
    PF_LAUNCH(st, "lstm_pointwise_bwd", lstm_pointwise_bwd_kernel, grid, dim3(256), s, gates, c_prev, c_out, dh,
              dc_next, dz, dc_prev, B, h);
    if (st != PF_OK) return st;
    SkinnyArgs a;
    build_dT(d, dz, Ux, Uh, part, a);
    st = launch_skinny_gemm(s, "lstm_dT=dz*[Ux|Uh]", a, false);
    if (st != PF_OK) return st;
    SliceSumArgs ss = {};
    ss.nseg = 2;
    ss.s[0] = slice_seg(a.p[0], dTx, gr, gr);
    ss.s[1] = slice_seg(a.p[a.nprob / 2], dTh, gr, gr);
    st = launch_slice_sum(s, ss);
    if (st != PF_OK) return st;
    build_dxh(d, dx != nullptr, dTx, dTh, Vx, Vh, part, a);
    st = launch_skinny_gemm(s, "lstm_dxh=[dTx*Vxt|dTh*Vht]", a, true);
    if (st != PF_OK) return st;
    ss = SliceSumArgs{};
    int q = 0;
    if (dx) ss.s[ss.nseg++] = slice_seg(a.p[q++], dx, din, din);
    ss.s[ss.nseg++] = slice_seg(a.p[q], dh_prev, h, h);
    // weight gradients: rank-B updates, with the slice sums of dx and dh_prev in the same launch
    RankArgs ra = {};
    ra.M = B;
    ra.accumulate = accumulate;
    for (int path = 0; path < 2; ++path) {
        const float *T = path ? Th : Tx;
        float *dU = path ? dUh : dUx;
        if (G == 1) {
            rank_add(ra, dz, 4 * (i64)h, T, gr, dU, r, 4 * h, r);
        } else {
            for (int g = 0; g < 4; ++g)
                rank_add(ra, dz + (i64)g * h, 4 * (i64)h, T + (i64)g * r, gr, dU + (i64)g * h * r, r, h, r);
        }
    }
    rank_add(ra, x, din, dTx, gr, dVx, gr, din, gr);
    rank_add(ra, h_prev, h, dTh, gr, dVh, gr, h, gr);
    if (dbias) rank_add(ra, dz, 4 * (i64)h, nullptr, 0, dbias, 1, 4 * h, 1);
    return launch_rank_update(s, "lstm_grads", ra, ss);
}


} // namespace pf

using namespace pf;

extern "C" {

size_t pf_lowrank_lstm_cell_fwd_workspace_bytes(const pf_lstm_desc *d)
{
    if (check_lstm_desc(d) != PF_OK) return 0;
    return lstm_tiles_ok(d) ? plan_lstm_tiles(d).fwd_bytes : plan_lstm(d).fwd_bytes;
}

size_t pf_lowrank_lstm_cell_bwd_workspace_bytes(const pf_lstm_desc *d)
{
    if (check_lstm_desc(d) != PF_OK) return 0;
    return lstm_skinny_pays(d) ? plan_lstm_skinny(d).bwd_bytes
           : lstm_tiles_ok(d)  ? plan_lstm_tiles(d).bwd_bytes
                               : plan_lstm(d).bwd_bytes;
}

int pf_lowrank_lstm_cell_fwd(const pf_lstm_desc *d, const void *x, const void *h_prev, const void *c_prev,
                             const void *Vx, const void *Ux, const void *Vh, const void *Uh, const void *bias,
                             void *h_out, void *c_out, void *gates_save, void *Tx_save, void *Th_save, void *workspace,
                             size_t workspace_bytes, void *stream)
{
    int st = check_lstm_desc(d);
    if (st != PF_OK) return st;
    if (!Vx || !Ux || !Vh || !Uh || (d->has_bias && !bias)) return PF_ERR_NULL;
    if (d->B > 0 && (!x || !h_prev || !c_prev || !h_out || !c_out || !gates_save || !Tx_save || !Th_save))
        return PF_ERR_NULL;
    if (any_misaligned({x, h_prev, c_prev, Vx, Ux, Vh, Uh, bias, h_out, c_out, gates_save, Tx_save, Th_save}, 16))
        return PF_ERR_UNSUPPORTED;
    if (d->B == 0) return PF_OK; // nothing to compute, nothing to check
    const size_t need = pf_lowrank_lstm_cell_fwd_workspace_bytes(d);
    if (need > 0 && (!workspace || workspace_bytes < need)) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    Workspace ws(workspace, workspace_bytes);
    if (lstm_tiles_ok(d))
        return lstm_fwd_tiles(d, (const float *)x, (const float *)h_prev, (const float *)c_prev, (const float *)Vx,
                              (const float *)Ux, (const float *)Vh, (const float *)Uh, (const float *)bias, (float *)h_out,
                              (float *)c_out, (float *)gates_save, (float *)Tx_save, (float *)Th_save, ws,
                              (hipStream_t)stream);
    return lstm_fwd_generic(d, (const float *)x, (const float *)h_prev, (const float *)c_prev, (const float *)Vx,
                            (const float *)Ux, (const float *)Vh, (const float *)Uh, (const float *)bias,
                            (float *)h_out, (float *)c_out, (float *)gates_save, (float *)Tx_save, (float *)Th_save, ws,
                            (hipStream_t)stream);
}

int pf_lowrank_lstm_cell_bwd(const pf_lstm_desc *d, const void *x, const void *h_prev, const void *c_prev,
                             const void *c_out, const void *gates_saved, const void *Tx_saved, const void *Th_saved,
                             const void *Vx, const void *Ux, const void *Vh, const void *Uh, const void *dh,
                             const void *dc_next, void *dx, void *dh_prev, void *dc_prev, void *dVx, void *dUx,
                             void *dVh, void *dUh, void *dbias, int accumulate, void *workspace,
                             size_t workspace_bytes, void *stream)
{
    int st = check_lstm_desc(d);
    if (st != PF_OK) return st;
    if (!Vx || !Ux || !Vh || !Uh || !dVx || !dUx || !dVh || !dUh) return PF_ERR_NULL;
    if (d->B > 0 && (!x || !h_prev || !c_prev || !c_out || !gates_saved || !Tx_saved || !Th_saved || !dh || !dh_prev ||
                     !dc_prev))
        return PF_ERR_NULL;
    if (any_misaligned({x, h_prev, c_prev, c_out, gates_saved, Tx_saved, Th_saved, Vx, Ux, Vh, Uh, dh, dc_next, dx,
                        dh_prev, dc_prev}, 16) ||
        any_misaligned({dVx, dUx, dVh, dUh, dbias}, 4))
        return PF_ERR_UNSUPPORTED;
    const size_t need = pf_lowrank_lstm_cell_bwd_workspace_bytes(d);
    if (need > 0 && (!workspace || workspace_bytes < need)) return PF_ERR_WORKSPACE;
    if (pf::any_misaligned({workspace}, 256)) return PF_ERR_UNSUPPORTED; // NULL passes: the size check has caught it
    Workspace ws(workspace, workspace_bytes);
    if (lstm_skinny_pays(d))
        return lstm_bwd_skinny(d, (const float *)x, (const float *)h_prev, (const float *)c_prev,
                               (const float *)c_out, (const float *)gates_saved, (const float *)Tx_saved,
                               (const float *)Th_saved, (const float *)Vx, (const float *)Ux, (const float *)Vh,
                               (const float *)Uh, (const float *)dh, (const float *)dc_next, (float *)dx,
                               (float *)dh_prev, (float *)dc_prev, (float *)dVx, (float *)dUx, (float *)dVh,
                               (float *)dUh, (float *)dbias, accumulate, ws, (hipStream_t)stream);
    if (lstm_tiles_ok(d))
        return lstm_bwd_tiles(d, (const float *)x, (const float *)h_prev, (const float *)c_prev, (const float *)c_out,
                              (const float *)gates_saved, (const float *)Tx_saved, (const float *)Th_saved,
                              (const float *)Vx, (const float *)Ux, (const float *)Vh, (const float *)Uh,
                              (const float *)dh, (const float *)dc_next, (float *)dx, (float *)dh_prev,
                              (float *)dc_prev, (float *)dVx, (float *)dUx, (float *)dVh, (float *)dUh, (float *)dbias,
                              accumulate, ws, (hipStream_t)stream);
    return lstm_bwd_generic(d, (const float *)x, (const float *)h_prev, (const float *)c_prev, (const float *)c_out,
                            (const float *)gates_saved, (const float *)Tx_saved, (const float *)Th_saved,
                            (const float *)Vx, (const float *)Ux, (const float *)Vh, (const float *)Uh,
                            (const float *)dh, (const float *)dc_next, (float *)dx, (float *)dh_prev, (float *)dc_prev,
                            (float *)dVx, (float *)dUx, (float *)dVh, (float *)dUh, (float *)dbias, accumulate, ws,
                            (hipStream_t)stream);
}

} // extern "C"
