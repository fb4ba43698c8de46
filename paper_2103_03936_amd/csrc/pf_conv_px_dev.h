// Device side of pf_conv_px.h that its kernels share.
#pragma once

#include "pf_conv_px.h"
#include "pf_tile.h"

namespace pf {

// Tiles of 32 PB pixels by workgroups of NT threads: rows of a panel (a row for what lies outside the tile included), groups of eight
// pixels, and the channels of a chunk, of which every thread has an octet of one group.
template <int PB, int NT>
struct PxRows {
    static constexpr int rows = PB == 4 ? 256 : PB == 2 ? 192 : 160, groups = PB == 1 ? 16 : 32, octets = NT / groups, CH = 8 * octets,
                         panels = CH / 64, panel = rows * 128, bytes = panels * panel;
};

__device__ __forceinline__ uint4 px_zero() { return make_uint4(0, 0, 0, 0); }

// Eight channels (r[j]: pixels 0..7 of channel j) -> pixel e: channels 0..7, and back (the same exchange).
__device__ __forceinline__ uint4 px_turn(const uint4 (&r)[8], int e)
{
    const uint32_t sel = e & 1 ? 0x07060302u : 0x05040100u;
    const auto w = [&](int j) { return e < 2 ? r[j].x : e < 4 ? r[j].y : e < 6 ? r[j].z : r[j].w; };
    return make_uint4(__builtin_amdgcn_perm(w(1), w(0), sel), __builtin_amdgcn_perm(w(3), w(2), sel),
                      __builtin_amdgcn_perm(w(5), w(4), sel), __builtin_amdgcn_perm(w(7), w(6), sel));
}

// One thread's block of a chunk: channel octet `o`, eight pixels.  Panels of 64 channels lie `panel` bytes apart.  Eight loads of 16 bytes, eight LDS rows.
struct PxBlock {
    int at[8];  // LDS byte of every pixel (the spare row for those outside the tile)
    int off;    // element of the first pixel in channel 8 o of its image
    bool live;  // the group exists
    __device__ __forceinline__ void init(const PxPlane &g, const PxTile &t, int C, int gi, int o, int spare, int panel)
    {
        int n, q;
        live = px_group(g, t, gi, n, q);
        if (!live) n = 0, q = 0;
        off = (n * C + 8 * o) * g.HW + q;
        const int y = px_div(q, g.W, g.mW);
        int x = q - y * g.W, s = (n * g.Hp + y + g.h) * g.Wp + x + g.h - t.base;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            at[e] = (o >> 3) * panel + px_at(live && s >= 0 && s < t.slots ? s : spare, o & 7);
            ++s;
            if (++x == g.W) x = 0, s += g.h;
        }
    }
    // channels c0 + 8 o .. of a tensor with C channels (C a multiple of eight): zero past the last
    __device__ __forceinline__ void load(const uint16_t *p, const PxPlane &g, int C, int c0, int o, uint4 (&r)[8]) const
    {
        if (live && c0 + 8 * o < C) {
#pragma unroll
            for (int j = 0; j < 8; ++j) r[j] = ldg16((const char *)p + 2u * (uint32_t)(off + (c0 + j) * g.HW));
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) r[j] = px_zero();
        }
    }
    // any number of channels
    __device__ __forceinline__ void load_any(const uint16_t *p, const PxPlane &g, int C, int o, uint4 (&r)[8]) const
    {
        if (C % 8 == 0) {
            load(p, g, C, 0, o, r);
            return;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            r[j] = px_zero();
            if (live && 8 * o + j < C) r[j] = ldg16((const char *)p + 2u * (uint32_t)(off + j * g.HW));
        }
    }
    __device__ __forceinline__ void store(unsigned char *panel, const uint4 (&r)[8]) const
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) *(uint4 *)(panel + at[e]) = px_turn(r, e);
    }
};

constexpr int PX_PACK = 4; // 16-byte pieces per thread
template <int NT>
__device__ __forceinline__ void px_pack(const PxPack &p, int block)
{
    const int n = p.C * p.kk, Kp = p.r <= 32 ? 32 : p.r <= 64 ? 64 : 128;
#pragma unroll
    for (int u = 0; u < PX_PACK; ++u) {
        const int i = (block * PX_PACK + u) * NT + (int)threadIdx.x, ro = i / n, j = i - ro * n;
        if (ro * 8 >= Kp) return;
        uint32_t w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = ro * 8 + e < p.r ? p.Uk[(ro * 8 + e) * n + j] : 0u;
        const int c = j / p.kk, tap = j - c * p.kk;
        *(uint4 *)(p.to + ((p.kk - 1 - tap) * p.C + c) * Kp + ro * 8) = make_uint4(w[0] | w[1] << 16, w[2] | w[3] << 16, w[4] | w[5] << 16, w[6] | w[7] << 16);
    }
}
inline int px_pack_blocks(const PxPack &p, int NT)
{
    return p.to ? (int)((px_pack_elems(p.C, p.r, 1) * p.kk / 8 + PX_PACK * NT - 1) / (PX_PACK * NT)) : 0;
}

// Elements i .. i + 7 of an array of `total` >= 8 elements, the first nv of them (0..8), zero after that.
__device__ __forceinline__ uint4 px_row_piece(const uint16_t *p, int i, int nv, int total)
{
    if (nv <= 0) return px_zero();
    const int a = min(i, total - 8);
    uint4 v = ldg16((const char *)p + 2u * (uint32_t)a);
    if (nv < 8) {
        v = piece_shift<2>(v, i - a);
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] &= nv >= 2 * j + 2 ? 0xffffffffu : nv == 2 * j + 1 ? 0xffffu : 0u;
        v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    return v;
}

// Where eight pixels of the tile go.
struct PxPieceOut {
    int n, q, col; // image, pixel, column in the tile
    bool live;
    __device__ __forceinline__ void init(const PxPlane &g, const PxTile &t, const PxOut &o, int gi)
    {
        live = px_out_group(g, o, gi, n, q);
        col = live ? n * g.HW + q - t.p0 : 0;
    }
};

// eight neighbouring floats in LDS (aligned: 16 bytes)
__device__ __forceinline__ void px_read8(const float *p, bool aligned, float *v)
{
    if (aligned) {
        const f32x4_t a = *(const f32x4_t *)p, b = *(const f32x4_t *)(p + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = a[e], v[4 + e] = b[e];
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = p[e];
    }
}

// eight values of channel c of [N][CH][HW], with the epilogue (`add`, `mask`: its pieces), from v
__device__ __forceinline__ void px_put(const PxPlane &g, const PxPieceOut &w, int CH, int c, uint16_t *out, const PxEpilogue &ep, float *v,
                                       uint4 add, uint4 mask)
{
    float f[8];
    if (ep.add) {
        piece_floats<bf16_t>(add, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += f[e];
    }
    if (ep.relu) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f);
    }
    if (ep.mask) {
        piece_floats<bf16_t>(mask, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = f[e] > 0.f ? v[e] : 0.f;
    }
    stg16((char *)out + 2u * (uint32_t)((w.n * CH + c) * g.HW + w.q), floats_piece<bf16_t>(v));
}
// The pixels that are left over, rows [0, rows) of the tile's sums `cs` (pitch `cp`), which are the channels c0 .. of out: four at a
// time, so that what is added and masks them is in flight together.
template <int NT>
__device__ __forceinline__ void px_put_rest(const PxPlane &g, const PxTile &t, const PxOut &o, int rest, const float *cs, int cp, int rows,
                                            int CH, int c0, uint16_t *out, const PxEpilogue &ep)
{
    const int total = min(rows, CH - c0) * rest;
    for (int q0 = threadIdx.x; q0 < total; q0 += 4 * NT) {
        int at[4], col[4], row[4];
        uint16_t add[4], mask[4];
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
            if (ep.add) x += bf16_bits_to_float(add[u]);
            if (ep.relu) x = fmaxf(x, 0.f);
            if (ep.mask) x = bf16_bits_to_float(mask[u]) > 0.f ? x : 0.f;
            if (q0 + u * NT < total) out[at[u]] = float_to_bf16_bits(x);
        }
    }
}
__device__ __forceinline__ uint4 px_fetch(const PxPlane &g, const PxPieceOut &w, int CH, int c, const uint16_t *p)
{
    return p && w.live ? ldg16((const char *)p + 2u * (uint32_t)((w.n * CH + c) * g.HW + w.q)) : px_zero();
}

} // namespace pf
