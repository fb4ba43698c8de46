// What the tiled products' kernels share: finding a workgroup's tile, and storing it.  One launch runs a
// list of problems: a workgroup finds its problem, its tile and its share of the contraction from its index.
#pragma once

#include "pf_tile_host.h"

namespace pf {

template <typename CT>
__device__ __forceinline__ float tile_float(typename TileEl<CT>::elem x)
{
    if constexpr (sizeof(CT) == 4) return x;
    else return bf16_bits_to_float(x);
}
template <typename CT>
__device__ __forceinline__ typename TileEl<CT>::elem tile_elem(float x)
{
    if constexpr (sizeof(CT) == 4) return x;
    else return float_to_bf16_bits(x);
}

// One 16-byte piece of a row-major output: V neighbouring columns n .. n + V - 1 of row m (n a multiple of V).
template <typename CT, int V>
__device__ __forceinline__ void put_piece(const TileProb &p, int ks, int zb, int m, int n, float *v)
{
    typedef typename TileEl<CT>::elem elem;
    const TileOut &o = p.o;
    if (m >= p.M || n >= p.N) return;
    const int nv = min(V, p.N - n);
    if (o.f32) {
        float *c = (float *)o.C + ks * o.split_stride + zb * p.sc + (i64)m * o.ld + n;
        if (nv == V && !o.accumulate) {
#pragma unroll
            for (int e = 0; e < V; e += 4) stg16(c + e, floats_piece<float>(v + e));
        } else {
            for (int e = 0; e < V; ++e)
                if (e < nv) c[e] = o.accumulate ? c[e] + v[e] : v[e];
        }
        return;
    }
    const i64 at = zb * p.sc + (i64)m * o.ld + n;
    elem *c = (elem *)o.C;
    const elem *add = (const elem *)o.add, *mask = (const elem *)o.mask, *bias = o.bias ? (const elem *)o.bias + zb * p.sbias : nullptr;
    if (nv == V) {
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
#pragma unroll
    for (int e = 0; e < V; ++e) {
        if (e < nv) {
            float t = v[e];
            if (bias) t += tile_float<CT>(bias[n + e]);
            if (add) t += tile_float<CT>(add[at + e]);
            if (o.relu) t = fmaxf(t, 0.f);
            if (mask) t = tile_float<CT>(mask[at + e]) > 0.f ? t : 0.f;
            c[at + e] = tile_elem<CT>(t);
        }
    }
}

// A tile of planes with its epilogue (the sums over k of a split product: row-major).  A thread's pieces lie in the same columns of several rows.
// What is added to up to four of them, scales and masks them is requested before the first is used: piece by piece, and element by element in planes
// that are no whole pieces, it was a chain of up to 24 waits, 4 to 5 us of a launch of 12.  A piece that would end past the array is pulled back
// inside and shifted into place, as the operands' are.
template <typename CT, class CFG>
__device__ __forceinline__ void put_planes(const TileProb &p, int ks, int zb, int m0, int n0, const unsigned char *smem, int tid)
{
    typedef typename TileEl<CT>::elem elem;
    constexpr int V = TileEl<CT>::V, CPR = CFG::BN / V, NT = TILE_THREADS * CFG::DEEP, ALL = CFG::BM * CPR, P = (ALL + NT - 1) / NT;
    constexpr int PER = P < 4 ? P : 4;
    static_assert(NT % CPR == 0 && P % PER == 0, "a thread's pieces are whole rounds, in the same columns of every row");
    const TileOut &o = p.o;
    if (o.HC == 0) {
        tile_pieces<CT, CFG>(smem, tid, [&](int m, int n, float *v) { put_piece<CT, V>(p, ks, zb, m0 + m, n0 + n, v); });
        return;
    }
    const int n = n0 + tid % CPR * V, row0 = m0 + tid / CPR;
    if (n >= p.N || (ALL < NT && tid >= ALL)) return;
    elem *c = (elem *)o.C;
    const elem *add = (const elem *)o.add, *mask = (const elem *)o.mask;
    const int cn = n / V, img = cn / o.HC, pos = (cn - img * o.HC) * V, nv = min(V, o.HW - pos);
    if (img >= o.N) return;
    const i64 step = o.s > 1 ? (i64)o.H * o.W : o.HW, total = (i64)o.N * o.CH * step; // from row to row, and to the array's end
    const i64 at0 = (i64)img * o.CH * step + (o.s > 1 ? 0 : pos);
    const auto sums = [&](int j, float *v) __attribute__((always_inline)) {
        constexpr int PITCH = CFG::BN + 4;
        const float *Cs = (const float *)smem + (tid / CPR + NT / CPR * j) * PITCH + tid % CPR * V;
#pragma unroll
        for (int e = 0; e < V; e += 4) {
            f32x4_t t = *(const f32x4_t *)&Cs[e];
#pragma unroll
            for (int w = 1; w < CFG::WK; ++w) t += *(const f32x4_t *)&Cs[w * CFG::BM * PITCH + e];
#pragma unroll
            for (int x = 0; x < 4; ++x) v[e + x] = t[x];
        }
    };
    if (o.s > 1) { // every second pixel (no scale)
        int off[V]; // from the channel's first pixel; -1: none
        int y = pos / o.gW, x = pos - y * o.gW;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int yy = y * o.s + o.ph, xx = x * o.s + o.pw;
            off[e] = e < nv && yy < o.H && xx < o.W ? yy * o.W + xx : -1;
            if (++x == o.gW) x = 0, ++y;
        }
        for (int j = 0; j < P; ++j) {
            const int m = row0 + NT / CPR * j;
            if (m >= p.M) break;
            const i64 at = at0 + m * step;
            elem fa[V], fm[V];
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const i64 i = at + max(off[e], 0);
                if (add) fa[e] = add[i];
                if (mask) fm[e] = mask[i];
            }
            float v[V];
            sums(j, v);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                if (add) v[e] += tile_float<CT>(fa[e]);
                if (o.relu) v[e] = fmaxf(v[e], 0.f);
                if (mask) v[e] = tile_float<CT>(fm[e]) > 0.f ? v[e] : 0.f;
                if (off[e] >= 0) c[at + off[e]] = tile_elem<CT>(v[e]);
            }
        }
        return;
    }
#pragma unroll 1
    for (int j0 = 0; j0 < P; j0 += PER) {
        uint4 ra[PER], rm[PER];
        float sc[PER], sh[PER];
        i64 at[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int m = min(row0 + NT / CPR * (j0 + u), p.M - 1);
            at[u] = at0 + m * step;
            const i64 from = min(at[u], total - V);
            if (add) ra[u] = ldg16(add + from);
            if (mask) rm[u] = ldg16(mask + from);
            if (o.scale) sc[u] = o.scale[m];
            if (o.shift) sh[u] = o.shift[m];
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (row0 + NT / CPR * (j0 + u) >= p.M) break;
            const int back = (int)(at[u] - min(at[u], total - V));
            float v[V], f[8];
            sums(j0 + u, v);
            if (o.scale || o.shift) {
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] = v[e] * (o.scale ? sc[u] : 1.f) + (o.shift ? sh[u] : 0.f);
            }
            if (add) {
                piece_floats<CT>(back ? piece_shift<sizeof(elem)>(ra[u], back) : ra[u], f);
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] += f[e];
            }
            if (o.relu) {
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] = fmaxf(v[e], 0.f);
            }
            if (mask) {
                piece_floats<CT>(back ? piece_shift<sizeof(elem)>(rm[u], back) : rm[u], f);
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] = f[e] > 0.f ? v[e] : 0.f;
            }
            if (nv == V) {
                stg16(c + at[u], floats_piece<CT>(v));
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (e < nv) c[at[u] + e] = tile_elem<CT>(v[e]);
            }
        }
    }
}

// Two tiles that are the even and the odd pixels of the same rows (a dX with stride 2, whose pixels x = 2 i and 2 i + 1 are reached by
// different taps): the first one's sums stay in registers while the second is multiplied, and whole pieces of neighbouring pixels
// leave.  Pixel by pixel, as elements 2 apart, the store and what is added and masks took 15 of the 24 us of a 64 x 64 tile.  Pieces that hold
// the end of a row leave so all the same, both phases at once.
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
        if (n >= p.N || img >= o.N || pos >= o.HW || 2 * y + o.ph >= o.H) return;
        elem *c = (elem *)o.C;
        const elem *add = (const elem *)o.add, *mask = (const elem *)o.mask;
        if (x + W2 > o.gW || 2 * x + V > o.W) { // pixels of two rows, or past the last one of an odd width
            int off[V]; // from the first pixel of the channel; -1: none
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const int cy = (pos + e / 2) / o.gW, yy = 2 * cy + o.ph, xx = 2 * (pos + e / 2 - cy * o.gW) + (e & 1);
                off[e] = pos + e / 2 < o.HW && yy < o.H && xx < o.W ? yy * o.W + xx : -1;
            }
#pragma unroll 1
            for (int j = 0; j < P; ++j) {
                const int row = (tid + TILE_THREADS * j) / CPR;
                if (m0 + row >= p.M) break;
                const i64 ch = ((i64)img * o.CH + m0 + row) * ((i64)o.H * o.W);
                elem fa[V], fm[V];
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    if (add) fa[e] = add[ch + max(off[e], 0)];
                    if (mask) fm[e] = mask[ch + max(off[e], 0)];
                }
                float first[W2];
#pragma unroll
                for (int q = 0; q < P; ++q)
#pragma unroll
                    for (int e = 0; e < W2; ++e) first[e] = q == j ? c0[q][e] : q == 0 ? 0.f : first[e];
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    float v = e & 1 ? at(smem, row, tid % CPR * W2 + e / 2) : first[e / 2];
                    if (add) v += tile_float<CT>(fa[e]);
                    if (mask) v = tile_float<CT>(fm[e]) > 0.f ? v : 0.f;
                    if (off[e] >= 0) c[ch + off[e]] = tile_elem<CT>(v);
                }
            }
            return;
        }
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
    tile_pieces<CT, CFG>(smem, tid, [&](int m, int n, float *v) { put_piece<CT, TileEl<CT>::V>(p, ks, zb, m0 + m, n0 + n, v); });
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
