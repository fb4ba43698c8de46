// Device side of pf_conv_px.h that its kernels share.
#pragma once

#include "pf_conv_px.h"
#include "pf_tile.h"

namespace pf {

// Tiles of 32 PB pixels by workgroups of NT threads: rows of a panel (a row for what lies outside the tile included), groups of V
// pixels, blocks of V channels x V pixels per thread (128 bytes of loads in flight), and the channels of a chunk.
// SD: a strided convolution, whose tiles reach over more pixels.
template <typename T, int PB, int NT, bool SD = false>
struct PxRows {
    static constexpr int V = PxEl<T>::V, rows = PB == 4 || SD ? 256 : PB == 2 ? 192 : 160, groups = (PB == 1 && !SD ? 128 : 256) / V, BL = 8 / V,
                         pieces = NT * BL / groups, CH = V * pieces, panels = CH / PxEl<T>::PC, panel = rows * 128, bytes = panels * panel;
};

__device__ __forceinline__ uint4 px_zero() { return make_uint4(0, 0, 0, 0); }
template <typename T>
__device__ __forceinline__ uint4 px_load(const T *p, int i) { return ldg16((const char *)p + (uint32_t)sizeof(T) * (uint32_t)i); }
template <typename T>
__device__ __forceinline__ void px_save(T *p, int i, uint4 v) { stg16((char *)p + (uint32_t)sizeof(T) * (uint32_t)i, v); }

__device__ __forceinline__ float px_float(uint16_t x) { return bf16_bits_to_float(x); }
__device__ __forceinline__ float px_float(float x) { return x; }
template <typename T>
__device__ __forceinline__ T px_round(float x)
{
    if constexpr (sizeof(T) == 2) return float_to_bf16_bits(x);
    else return x;
}
template <typename T>
__device__ __forceinline__ void px_unpack(uint4 r, float *f) { piece_floats<typename std::conditional<sizeof(T) == 2, bf16_t, float>::type>(r, f); }
template <typename T>
__device__ __forceinline__ uint4 px_piece(const float *f) { return floats_piece<typename std::conditional<sizeof(T) == 2, bf16_t, float>::type>(f); }
__device__ __forceinline__ uint32_t px_word(const uint4 &r, int i) { return i == 0 ? r.x : i == 1 ? r.y : i == 2 ? r.z : r.w; }

// V channels (r[j]: pixels 0 .. V - 1 of channel j) -> pixel e: channels 0 .. V - 1, and back (the same exchange).
__device__ __forceinline__ uint4 px_turn(const uint4 (&r)[8], int e)
{
    const uint32_t sel = e & 1 ? 0x07060302u : 0x05040100u;
    const auto w = [&](int j) { return px_word(r[j], e >> 1); };
    return make_uint4(__builtin_amdgcn_perm(w(1), w(0), sel), __builtin_amdgcn_perm(w(3), w(2), sel),
                      __builtin_amdgcn_perm(w(5), w(4), sel), __builtin_amdgcn_perm(w(7), w(6), sel));
}
__device__ __forceinline__ uint4 px_turn(const uint4 (&r)[4], int e) // (float: a matter of names)
{
    return make_uint4(px_word(r[0], e), px_word(r[1], e), px_word(r[2], e), px_word(r[3], e));
}

// One step of 2 V channels: the products of a lane's pieces.
template <typename T>
__device__ __forceinline__ void px_mma(f32x16_t &acc, uint4 a, uint4 b)
{
    if constexpr (sizeof(T) == 2) {
        union {
            uint4 u;
            bf16x8_t v;
        } x, y;
        x.u = a, y.u = b;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.v, y.v, acc, 0, 0, 0);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(px_word(a, e)), __uint_as_float(px_word(b, e)), acc, 0, 0, 0);
    }
}
__device__ __forceinline__ void px_clear(f32x16_t &t)
{
#pragma unroll
    for (int v = 0; v < 16; ++v) t[v] = 0.f;
}
// Sums of N blocks.  Float sums runs of at most 32 terms on their own before it adds them to the total, and one block's runs, chunk by chunk,
// in one more stage: the rounding error then grows with the number of runs of a chunk and of chunks, as it does in the tiled products,
// which split long sums over workgroups (3 x 3 taps of 256 channels, rms: 1.47e-7 without that stage, 1.10e-7 there).
template <typename T, int N>
struct PxSum {
    static constexpr bool RUNS = sizeof(T) == 4, FOLD = RUNS && N == 1;
    f32x16_t acc[N], run[RUNS ? N : 1], all[1];
    static __device__ __forceinline__ void move(f32x16_t &to, f32x16_t &from)
    {
#pragma unroll
        for (int v = 0; v < 16; ++v) to[v] += from[v];
        px_clear(from);
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            px_clear(acc[i]);
            if (RUNS) px_clear(run[RUNS ? i : 0]);
        }
        if (FOLD) px_clear(all[0]);
    }
    __device__ __forceinline__ f32x16_t &at(int i) { return RUNS ? run[RUNS ? i : 0] : acc[i]; }
    __device__ __forceinline__ void flush() // the end of a run
    {
        if (RUNS) {
#pragma unroll
            for (int i = 0; i < N; ++i) move(acc[i], run[RUNS ? i : 0]);
        }
    }
    __device__ __forceinline__ void fold() // of a chunk
    {
        if (FOLD) move(all[0], acc[0]);
    }
    __device__ __forceinline__ void total()
    {
        if (FOLD) move(acc[0], all[0]);
    }
};

// One thread's block of a chunk: V channels from the piece `o` on, V pixels.  Panels lie `panel` bytes apart.
template <typename T>
struct PxBlock {
    static constexpr int V = PxEl<T>::V;
    int at[V];  // LDS byte of every pixel (the spare row for those outside the tile)
    int off;    // element of the first pixel in channel V o of its image
    bool live;  // the group exists
    __device__ __forceinline__ void init(const PxPlaneOf<T> &g, const PxTile &t, int st, int C, int gi, int o, int spare, int panel)
    {
        int n, q;
        live = px_group(g, t, gi, n, q);
        if (!live) n = 0, q = 0;
        off = (n * C + V * o) * g.HW + q;
        const int y = px_div(q, g.W, g.mW);
        if (g.h == 0 && st > 1) { // (rows that no output pixel sees)
            const int last = px_div(q + V - 1, g.W, g.mW);
            live = live && last - last % st >= y;
        }
        int x = q - y * g.W, s = (n * g.Hp + y + g.h) * g.Wp + x + g.h - t.base;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            at[e] = (o >> 3) * panel + px_at(live && s >= 0 && s < t.slots ? s : spare, o & 7);
            ++s;
            if (++x == g.W) x = 0, s += g.h;
        }
    }
    // channels c0 + V o .. of a tensor with C channels (whole pieces): zero past the last
    __device__ __forceinline__ void load(const T *p, const PxPlaneOf<T> &g, int C, int c0, int o, uint4 (&r)[V]) const
    {
        if (live && c0 + V * o < C) {
#pragma unroll
            for (int j = 0; j < V; ++j) r[j] = px_load(p, off + (c0 + j) * g.HW);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) r[j] = px_zero();
        }
    }
    __device__ __forceinline__ void store(unsigned char *panel, const uint4 (&r)[V]) const
    {
#pragma unroll
        for (int e = 0; e < V; ++e) *(uint4 *)(panel + at[e]) = px_turn(r, e);
    }
};
// ... and all of a thread's
template <typename T, int PB, int NT, bool SD = false>
struct PxBlocks {
    typedef PxRows<T, PB, NT, SD> R;
    PxBlock<T> b[R::BL];
    static __device__ __forceinline__ int piece(int u) { return ((int)threadIdx.x + NT * u) / R::groups; }
    __device__ __forceinline__ void init(const PxPlaneOf<T> &g, const PxTile &t, int st, int C)
    {
#pragma unroll
        for (int u = 0; u < R::BL; ++u) b[u].init(g, t, st, C, threadIdx.x % R::groups, piece(u), R::rows - 1, R::panel);
    }
    __device__ __forceinline__ void load(const T *p, const PxPlaneOf<T> &g, int C, int c0, uint4 (&r)[R::BL][R::V]) const
    {
#pragma unroll
        for (int u = 0; u < R::BL; ++u) b[u].load(p, g, C, c0, piece(u), r[u]);
    }
    __device__ __forceinline__ void store(unsigned char *panel, const uint4 (&r)[R::BL][R::V]) const
    {
#pragma unroll
        for (int u = 0; u < R::BL; ++u) b[u].store(panel, r[u]);
    }
};

constexpr int PX_PACK = 4; // 16-byte pieces per thread
template <typename T, int NT>
__device__ __forceinline__ void px_pack(const PxPack<T> &p, int block)
{
    constexpr int V = PxEl<T>::V;
    const int n = p.C * p.kk, Kp = p.r <= 32 ? 32 : p.r <= 64 ? 64 : 128;
#pragma unroll
    for (int u = 0; u < PX_PACK; ++u) {
        const int i = (block * PX_PACK + u) * NT + (int)threadIdx.x, ro = i / n, j = i - ro * n;
        if (ro * V >= Kp) return;
        union {
            T e[V];
            uint4 u;
        } w;
#pragma unroll
        for (int e = 0; e < V; ++e) w.e[e] = ro * V + e < p.r ? p.Uk[(ro * V + e) * n + j] : T(0);
        const int c = j / p.kk, tap = j - c * p.kk;
        *(uint4 *)(p.to + ((p.kk - 1 - tap) * p.C + c) * Kp + ro * V) = w.u;
    }
}
template <typename T>
inline int px_pack_blocks(const PxPack<T> &p, int NT)
{
    return p.to ? (int)((px_pack_elems(p.C, p.r, 1) * p.kk / PxEl<T>::V + PX_PACK * NT - 1) / (PX_PACK * NT)) : 0;
}

// Elements i .. i + V - 1 of an array of `total` >= V elements, the first nv of them (0 .. V), zero after that.
template <typename T>
__device__ __forceinline__ uint4 px_row_piece(const T *p, int i, int nv, int total)
{
    constexpr int V = PxEl<T>::V;
    if (nv <= 0) return px_zero();
    const int a = min(i, total - V);
    uint4 v = px_load(p, a);
    if (nv < V) {
        v = piece_shift<(int)sizeof(T)>(v, i - a);
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (V == 8) w[j] &= nv >= 2 * j + 2 ? 0xffffffffu : nv == 2 * j + 1 ? 0xffffu : 0u;
            else w[j] = j < nv ? w[j] : 0u;
        }
        v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    return v;
}

// Where V pixels of the tile go.
struct PxPieceOut {
    int n, q, col; // image, pixel, column in the tile
    bool live;
    template <int S>
    __device__ __forceinline__ void init(const PxPlane<S> &g, const PxTile &t, const PxOut &o, int gi)
    {
        live = px_out_group(g, o, gi, n, q);
        col = live ? n * g.HW + q - t.p0 : 0;
    }
};

// V neighbouring floats in LDS (aligned: to 16 bytes)
template <int V>
__device__ __forceinline__ void px_read(const float *p, bool aligned, float *v)
{
    if (aligned) {
#pragma unroll
        for (int e = 0; e < V; e += 4) {
            const f32x4_t a = *(const f32x4_t *)(p + e);
#pragma unroll
            for (int x = 0; x < 4; ++x) v[e + x] = a[x];
        }
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = p[e];
    }
}

// V values of channel c of [N][CH][HW], with the epilogue (`add`, `mask`: its pieces), from v
template <typename T>
__device__ __forceinline__ void px_put(const PxPlaneOf<T> &g, const PxPieceOut &w, int CH, int c, T *out, const PxEpilogue<T> &ep, float *v,
                                       uint4 add, uint4 mask)
{
    constexpr int V = PxEl<T>::V;
    float f[V];
    if (ep.add) {
        px_unpack<T>(add, f);
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] += f[e];
    }
    if (ep.relu) {
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = fmaxf(v[e], 0.f);
    }
    if (ep.mask) {
        px_unpack<T>(mask, f);
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = f[e] > 0.f ? v[e] : 0.f;
    }
    px_save(out, (w.n * CH + c) * g.HW + w.q, px_piece<T>(v));
}
// The pixels that are left over, rows [0, rows) of the tile's sums `cs` (pitch `cp`), which are the channels c0 .. of out: four at a
// time, so that what is added and masks them is in flight together.
template <typename T, int NT>
__device__ __forceinline__ void px_put_rest(const PxPlaneOf<T> &g, const PxTile &t, const PxOut &o, int rest, const float *cs, int cp, int rows,
                                            int CH, int c0, T *out, const PxEpilogue<T> &ep)
{
    const int total = min(rows, CH - c0) * rest;
    for (int q0 = threadIdx.x; q0 < total; q0 += 4 * NT) {
        int at[4], col[4], row[4];
        T add[4], mask[4];
        float sc[4], sh[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = min(q0 + u * NT, total - 1);
            int n, px;
            row[u] = q / rest;
            px_out_pixel(g, o, q - row[u] * rest, n, px);
            at[u] = (n * CH + c0 + row[u]) * g.HW + px;
            col[u] = n * g.HW + px - t.p0;
            if (ep.add) add[u] = ep.add[at[u]];
            if (ep.mask) mask[u] = ep.mask[at[u]];
            sc[u] = ep.scale ? ep.scale[c0 + row[u]] : 1.f;
            sh[u] = ep.shift ? ep.shift[c0 + row[u]] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float x = cs[row[u] * cp + col[u]] * sc[u] + sh[u];
            if (ep.add) x += px_float(add[u]);
            if (ep.relu) x = fmaxf(x, 0.f);
            if (ep.mask) x = px_float(mask[u]) > 0.f ? x : 0.f;
            if (q0 + u * NT < total) out[at[u]] = px_round<T>(x);
        }
    }
}
template <typename T>
__device__ __forceinline__ uint4 px_fetch(const PxPlaneOf<T> &g, const PxPieceOut &w, int CH, int c, const T *p)
{
    return p && w.live ? px_load(p, (w.n * CH + c) * g.HW + w.q) : px_zero();
}

} // namespace pf
