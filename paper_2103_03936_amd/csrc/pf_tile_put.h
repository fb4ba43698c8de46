// What the tiled products' kernels share: finding a workgroup's tile, and storing it.  One launch runs a
// list of problems: a workgroup finds its problem, its tile and its share of the contraction from its index.
#pragma once

#include "pf_tile_host.h"

namespace pf {

// One 16-byte piece of the output: V neighbouring columns n .. n + V - 1 of row m (n a multiple of V).
template <typename CT, int V>
__device__ __forceinline__ void put_piece(const TileProb &p, int ks, int zb, int m, int n, float *v)
{
    typedef typename TileEl<CT>::elem elem;
    const TileOut &o = p.o;
    if (m >= p.M || n >= p.N) return;
    if (o.f32) {
        float *c = (float *)o.C + ks * o.split_stride + zb * p.sc + (i64)m * o.ld + n;
        const int nv = min(V, p.N - n);
        if (nv == V && !o.accumulate) {
#pragma unroll
            for (int e = 0; e < V; e += 4) stg16(c + e, floats_piece<float>(v + e));
        } else {
            for (int e = 0; e < V; ++e)
                if (e < nv) c[e] = o.accumulate ? c[e] + v[e] : v[e];
        }
        return;
    }
    i64 at;
    int nv;
    int pos = 0;
    if (o.HC > 0) {
        const int cn = n / V, img = cn / o.HC;
        pos = (cn - img * o.HC) * V;
        nv = min(V, o.HW - pos);
        if (img >= o.N) return;
        if (o.s > 1) {
            at = ((i64)img * o.CH + m) * ((i64)o.H * o.W);
        } else {
            at = ((i64)img * o.CH + m) * o.HW + pos;
        }
    } else {
        at = zb * p.sc + (i64)m * o.ld + n;
        nv = min(V, p.N - n);
    }
    elem *c = (elem *)o.C;
    const elem *add = (const elem *)o.add, *mask = (const elem *)o.mask, *bias = o.bias ? (const elem *)o.bias + zb * p.sbias : nullptr;
    const float sc = o.scale ? o.scale[m] : 1.f, sh = o.shift ? o.shift[m] : 0.f;
    if (o.scale || o.shift) {
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = v[e] * sc + sh;
    }
    if (nv == V && !(o.s > 1)) {
        float f[8];
        if (bias) {
            piece_floats<CT>(ldg16(bias + n), f);
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] += f[e];
        }
        if (add) {
            piece_floats<CT>(ldg16(add + at), f);
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] += f[e];
        }
        if (o.relu) {
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = fmaxf(v[e], 0.f);
        }
        if (mask) {
            piece_floats<CT>(ldg16(mask + at), f);
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = f[e] > 0.f ? v[e] : 0.f;
        }
        stg16(c + at, floats_piece<CT>(v));
        return;
    }
    int y = 0, x = 0;
    if (o.s > 1) y = pos / o.gW, x = pos - y * o.gW;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        if (e < nv) {
            i64 i = at + e;
            bool in = true;
            if (o.s > 1) {
                const int yy = y * o.s + o.ph, xx = x * o.s + o.pw;
                in = yy < o.H && xx < o.W;
                i = at + (i64)yy * o.W + xx;
                if (++x == o.gW) x = 0, ++y;
            }
            if (in) {
                union {
                    uint32_t w[4];
                    elem e[V];
                } u;
                float t = v[e];
                if (bias) t += sizeof(elem) == 4 ? ((const float *)bias)[n + e] : bf16_bits_to_float((uint16_t)bias[n + e]);
                if (add) t += sizeof(elem) == 4 ? ((const float *)add)[i] : bf16_bits_to_float((uint16_t)add[i]);
                if (o.relu) t = fmaxf(t, 0.f);
                if (mask)
                    t = (sizeof(elem) == 4 ? ((const float *)mask)[i] : bf16_bits_to_float((uint16_t)mask[i])) > 0.f ? t
                                                                                                                   : 0.f;
                if (sizeof(elem) == 4) u.w[0] = __float_as_uint(t);
                else u.w[0] = float_to_bf16_bits(t);
                c[i] = u.e[0];
            }
        }
    }
}

// Two tiles that are the even and the odd pixels of the same rows (a dX with stride 2, whose pixels x = 2 i and 2 i + 1 are reached by
// different taps): the first one's sums stay in registers while the second is multiplied, and whole pieces of neighbouring pixels
// leave.  Pixel by pixel, as elements 2 apart, the store and what is added and masks took 15 of the 24 us of a 64 x 64 tile.
template <typename CT, class CFG>
struct PairOut {
    static constexpr bool TAKEN = CFG::BM == 64 && CFG::BN == 64; // (the shape of these products' tiles)
    typedef typename TileEl<CT>::elem elem;
    static constexpr int V = TileEl<CT>::V, W2 = V / 2, CPR = CFG::BN / W2, P = CFG::BM * CPR / TILE_THREADS, PITCH = CFG::BN + 4;
    float c0[P][W2];

    // (wavefronts that share a block: their sums together)
    static __device__ __forceinline__ float at(const unsigned char *smem, int m, int n)
    {
        const float *Cs = (const float *)smem;
        float v = Cs[m * PITCH + n];
#pragma unroll
        for (int w = 1; w < CFG::WK; ++w) v += Cs[(w * CFG::BM + m) * PITCH + n];
        return v;
    }
    __device__ __forceinline__ void keep(const unsigned char *smem, int tid)
    {
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int q = tid + TILE_THREADS * j;
#pragma unroll
            for (int e = 0; e < W2; ++e) c0[j][e] = at(smem, q / CPR, q % CPR * W2 + e);
        }
    }
    __device__ __forceinline__ void put(const TileProb &p, int m0, int n0, const unsigned char *smem, int tid) const
    {
        const TileOut &o = p.o;
        const int n = n0 + tid % CPR * W2, cell = o.HC * V, img = n / cell, pos = n - img * cell, y = pos / o.gW, x = pos - y * o.gW;
        if (n >= p.N || img >= o.N || pos >= o.HW) return;
        elem *c = (elem *)o.C;
        const elem *add = (const elem *)o.add, *mask = (const elem *)o.mask;
        constexpr int per = 4; // pieces whose operands are in flight together
        static_assert(P % per == 0 && TILE_THREADS % CPR == 0, "a thread's pieces are whole rounds, in the same pixels of every row");
#pragma unroll
        for (int j0 = 0; j0 < P; j0 += per) {
            uint4 ra[per], rm[per];
            i64 to[per];
#pragma unroll
            for (int u = 0; u < per; ++u) {
                const int m = min(m0 + (tid + TILE_THREADS * (j0 + u)) / CPR, p.M - 1);
                to[u] = ((i64)img * o.CH + m) * ((i64)o.H * o.W) + (i64)(2 * y + o.ph) * o.W + 2 * x;
                if (add) ra[u] = ldg16(add + to[u]);
                if (mask) rm[u] = ldg16(mask + to[u]);
            }
#pragma unroll
            for (int u = 0; u < per; ++u) {
                const int j = j0 + u, row = (tid + TILE_THREADS * j) / CPR;
                if (m0 + row >= p.M) continue;
                float v[V], f[8];
#pragma unroll
                for (int e = 0; e < W2; ++e) {
                    v[2 * e] = c0[j][e];
                    v[2 * e + 1] = at(smem, row, tid % CPR * W2 + e);
                }
                if (add) {
                    piece_floats<CT>(ra[u], f);
#pragma unroll
                    for (int e = 0; e < V; ++e) v[e] += f[e];
                }
                if (mask) {
                    piece_floats<CT>(rm[u], f);
#pragma unroll
                    for (int e = 0; e < V; ++e) v[e] = f[e] > 0.f ? v[e] : 0.f;
                }
                stg16(c + to[u], floats_piece<CT>(v));
            }
        }
    }
};

// Stores a tile and, from the loader that added them up, row sums r0 .. of at most nr.
template <typename CT, class CFG, class L>
__device__ __forceinline__ void finish(const TileProb &p, int ks, int zb, int m0, int n0, L &l, int r0, int nr, bool sums,
                                       unsigned char *smem, int tid)
{
    constexpr int V = TileEl<CT>::V;
    tile_pieces<CT, CFG>(smem, tid, [&](int m, int n, float *v) { put_piece<CT, V>(p, ks, zb, m0 + m, n0 + n, v); });
    if (sums) {
        __syncthreads();
        float *out = p.o.sums + ks * p.o.sums_stride + zb * p.ssums;
        const bool acc = p.o.accumulate != 0;
        l.put_sums((float *)smem, tid, [&](int r, float v) {
            if (r0 + r < nr) out[r0 + r] = acc ? out[r0 + r] + v : v;
        });
    }
}

// The argument block where the launch put it.  (Indexed by problem and, for the taps, by lane, the by-value parameter
// would be copied to scratch memory by every thread.)
__device__ __forceinline__ const TileArgs &tile_args(const TileArgs &a)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const TileArgs *)(const __attribute__((address_space(4))) TileArgs *)__builtin_amdgcn_kernarg_segment_ptr();
#else
    return a;
#endif
}

struct TileAt {
    int prob, index, ks, zb, m0, n0;
    bool live; // (not one of the workgroups that fill up a problem)
};
template <class CFG>
__device__ __forceinline__ TileAt find_tile(const TileArgs &a)
{
    TileAt t;
    // Workgroups are dealt to the eight dies in turn: every die gets a run of a problem's consecutive tiles, which share
    // operands in its L2, and its share of every problem (a problem's workgroups are padded to a multiple of eight).
    const int b = blockIdx.x;
    t.prob = 0;
#pragma unroll
    for (int i = 1; i < TILE_MAX_PROBS; ++i)
        if (i < a.n && b >= a.p[i].block0) t.prob = i;
    const TileProb &p = a.p[t.prob];
    const int n = p.tm * p.tn * p.ksplit * p.nb, w = b - p.block0;
    t.index = (w & 7) * ((n + 7) >> 3) + (w >> 3);
    t.live = t.index < n;
    const int per = p.tm * p.tn, zk = t.index / per, q = t.index - zk * per, tm = q / p.tn;
    t.zb = zk / p.ksplit;
    t.ks = zk - t.zb * p.ksplit;
    t.m0 = tm * CFG::BM;
    t.n0 = (q - tm * p.tn) * CFG::BN;
    return t;
}

} // namespace pf
