// Tiled matrix products for any shape, the device side: C(m,n) = sum_k A(m,k) B(k,n) on one BM x BN tile.
//
// Operands reach LDS in 16-byte pieces that keep the direction they have in memory: along k ("KC": tile rows of BK
// elements) or along the row / column index ("MC": one tile row per k).  MC tiles of bf16 are read with the
// transposing LDS read, MC tiles of float one element per lane, so neither needs a transposed copy.  A piece may start
// at any element (rows of odd length): the load is then an unaligned 16-byte load, which costs the memory pipeline
// about three aligned ones and is still four times cheaper than eight element loads.  Edges never branch per element: the
// address of a piece that would leave its row is pulled back inside the row and the piece is shifted into place when
// it is written to LDS; what lies past K is written as zero, what lies past M or N is never stored.
//
// The pieces of NS chunks of the contraction are in flight in registers while one of two LDS buffers is multiplied
// and the other is filled: one barrier per chunk.  The main loop has no condition on its loads (a load past the last
// chunk repeats a valid address), and the last chunks have a copy of their own: with a load that may or may not have
// been issued the compiler can only wait for all of them (8192 x 2048 x 512, bf16, 128 x 128 tiles: 45 -> 33 us, 510
// TFLOP/s; the fragments' LDS traffic, 96 KB per chunk at 128 bytes per clock, is then what bounds them).  A chunk is 64 (bf16) or 32 (float) deep, so that a workgroup has
// 16 to 64 KB outstanding: with few workgroups per compute unit it is the latency of the loads, not their number, that
// bounds these products.  float sums every chunk on its own before adding it to the total (the rounding error then
// grows with K / 32).
#pragma once

#include "pf_common.h"

#include <type_traits>

namespace pf {

template <typename CT>
struct TileEl;
template <>
struct TileEl<bf16_t> {
    typedef uint16_t elem;
    static constexpr int V = 8, BK = 64, PAD = 8;
};
template <>
struct TileEl<float> {
    typedef float elem;
    static constexpr int V = 4, BK = 32, PAD = 4;
};

// BM x BN tile, 4 DEEP wavefronts, WM x WN of them over the tile; those that share a block split the contraction, whose chunks are
// DEEP times as long
template <int BM_, int BN_, int WM_, int WN_, int NS_, int DEEP_ = 1>
struct TileCfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_, DEEP = DEEP_, WK = 4 * DEEP / (WM_ * WN_);
    // Wavefronts per SIMD that a kernel of plain products is compiled for: the registers would allow fewer if the compiler
    // had its way (float, 64 x 64: one workgroup per compute unit -> three, 8192 x 1024 x 256 60 -> 49 us, 88 TFLOP/s)
    template <typename CT>
    static constexpr int OCC = sizeof(CT) == 2 ? (BM_ * BN_ <= 64 * 64 ? 4 : 2)
                                               : (BM_ * BN_ <= 32 * 32 ? 3 : BM_ * BN_ <= 64 * 128 ? 2 : 1);
};

constexpr int TILE_THREADS = 256;

// ------------------------------------------------------------------ 16-byte pieces
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));

__device__ __forceinline__ uint4 ldg16(const void *p)
{
    const u32x4_any v = *(const u32x4_any *)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void stg16(void *p, uint4 v)
{
    u32x4_any w;
    w.x = v.x, w.y = v.y, w.z = v.z, w.w = v.w;
    *(u32x4_any *)p = w;
}

// An array of less than 2^31 bytes seen through a buffer descriptor: a load from beyond its end (BUF_OUT always is) gives zeros, a store
// there is dropped.  So neither needs a branch, and the compiler can count what is in flight: after a load under a condition it waits for
// everything that was issued since.
constexpr uint32_t BUF_OUT = 0x80000000u;
struct BufSrc {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ BufSrc(const void *p, i64 bytes) : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, p ? (int)bytes : 0, 0x00027000)) {}
    __device__ __forceinline__ uint4 load(uint32_t at) const
    {
        typedef unsigned int v4 __attribute__((ext_vector_type(4)));
        const v4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 0, 0);
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    __device__ __forceinline__ void store(uint32_t at, uint4 u) const
    {
        typedef unsigned int v4 __attribute__((ext_vector_type(4)));
        const v4 v = {u.x, u.y, u.z, u.w};
        __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)at, 0, 0);
    }
};

// element e of the result is element e + s of r (0 where that is outside the piece)
template <int EB>
__device__ __forceinline__ uint4 piece_shift(uint4 r, int s)
{
    // towards the front by s >= 0; a shift to the back is one to the front of the piece with four zero words before it
    const int b = 8 * EB * s + (s < 0 ? 128 : 0); // bits
    const bool back = s < 0;
    const uint32_t w0 = back ? 0u : r.x, w1 = back ? 0u : r.y, w2 = back ? 0u : r.z, w3 = back ? 0u : r.w;
    const uint32_t w4 = back ? r.x : 0u, w5 = back ? r.y : 0u, w6 = back ? r.z : 0u, w7 = back ? r.w : 0u;
    if (b >= 128 || b < 0) return make_uint4(0, 0, 0, 0);
    const bool q1 = b & 32, q2 = b & 64;
    const uint32_t a0 = q2 ? w2 : w0, a1 = q2 ? w3 : w1, a2 = q2 ? w4 : w2, a3 = q2 ? w5 : w3, a4 = q2 ? w6 : w4,
                   a5 = q2 ? w7 : w5;
    const uint32_t c0 = q1 ? a1 : a0, c1 = q1 ? a2 : a1, c2 = q1 ? a3 : a2, c3 = q1 ? a4 : a3, c4 = q1 ? a5 : a4;
    const int f = b & 31;
    return make_uint4((uint32_t)((((uint64_t)c1 << 32) | c0) >> f), (uint32_t)((((uint64_t)c2 << 32) | c1) >> f),
                      (uint32_t)((((uint64_t)c3 << 32) | c2) >> f), (uint32_t)((((uint64_t)c4 << 32) | c3) >> f));
}

// Masks of a piece's elements are bytes (bit e: keep element e); a table in LDS holds the piece-wide mask of every byte.
template <int V>
struct MaskTable {
    static constexpr int N = 1 << V, BYTES = 16 * N;
    static __device__ __forceinline__ void build(unsigned char *tab, int tid)
    {
        if (tid < N) {
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                w[e] = V == 4 ? (tid >> e & 1 ? 0xffffffffu : 0u)
                              : (tid >> (2 * e) & 1 ? 0xffffu : 0u) | (tid >> (2 * e + 1) & 1 ? 0xffff0000u : 0u);
            ((uint4 *)tab)[tid] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    static __device__ __forceinline__ uint4 apply(const unsigned char *tab, uint32_t m, uint4 r)
    {
        const uint4 k = ((const uint4 *)tab)[m];
        return make_uint4(r.x & k.x, r.y & k.y, r.z & k.z, r.w & k.w);
    }
};

template <typename CT>
__device__ __forceinline__ void piece_floats(uint4 r, float *f)
{
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
    if (sizeof(CT) == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(w[e]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f[2 * e] = __uint_as_float(w[e] << 16);
            f[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
        }
    }
}
template <typename CT>
__device__ __forceinline__ uint4 floats_piece(const float *f)
{
    if (sizeof(CT) == 4)
        return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]),
                      pack_bf16x2(f[6], f[7]));
}

// ------------------------------------------------------------------ operand loaders
// A loader owns CH pieces of a tile per thread.  load() issues the loads of the next chunk, store() writes the oldest
// outstanding chunk to LDS; both walk the same sequence of chunks.  XF words travel with a chunk's pieces (row
// scales, taps).  SUM (weight gradients) adds up what passes.

// Matrix stored [rows][K] with k contiguous, leading dimension ld; SEG: k comes in segments of `seg` (whole pieces), each a
// matrix of its own that starts `jump` elements after the one before
template <typename CT, int ROWS, bool SEG = false, int DEEP = 1>
struct LoadKC {
    typedef typename TileEl<CT>::elem elem;
    static constexpr bool KC = true;
    static constexpr int V = TileEl<CT>::V, BK = TileEl<CT>::BK * DEEP, PITCH = BK + TileEl<CT>::PAD, CPR = BK / V, NT = TILE_THREADS * DEEP,
                         CH = ROWS * CPR / NT, LDS = ROWS * PITCH, XF = 1;
    const elem *rp[CH];
    int K, kc, row, kl, ks;
    int seg = 0;
    i64 jump = 0;

    __device__ __forceinline__ void init(const void *p, i64 ld, int rows, int K_, int row0, int kbeg, int tid)
    {
        K = K_;
        kc = (tid % CPR) * V;
        row = tid / CPR;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = min(row0 + row + i * (NT / CPR), rows - 1);
            rp[i] = (const elem *)p + (i64)r * ld;
        }
        kl = ks = kbeg;
    }
    __device__ __forceinline__ void load(uint4 (&r)[CH], int (&x)[XF])
    {
        const int k = min(kl + kc, K - V);
        const i64 at = SEG && seg > 0 ? k + (k / seg) * (jump - seg) : k;
#pragma unroll
        for (int i = 0; i < CH; ++i) r[i] = ldg16(rp[i] + at);
        kl += BK;
    }
    template <bool EDGE>
    __device__ __forceinline__ void store(elem *lds, uint4 (&r)[CH], int (&x)[XF])
    {
        const bool tail = EDGE && ks + BK > K;
        const int s = ks + kc - min(ks + kc, K - V);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            uint4 v = r[i];
            if (tail) v = piece_shift<sizeof(elem)>(v, s);
            *(uint4 *)&lds[(row + i * (NT / CPR)) * PITCH + kc] = v;
        }
        ks += BK;
    }
};

// Matrix stored [K][cols] with the row / column index contiguous; kscale (nullable): row k is multiplied by kscale[k].
// SUM of floats: a thread may see a thousand rows of an unsplit gradient, so it adds them in runs of sixteen chunks (16384 rows of
// zero mean: one chain 4.3e-7 off, relative, runs 1.4e-7).
template <typename CT, int ROWS, bool SUM = false, bool SCALE = false, int DEEP = 1>
struct LoadMC {
    typedef typename TileEl<CT>::elem elem;
    static constexpr bool KC = false;
    static constexpr int V = TileEl<CT>::V, BK = TileEl<CT>::BK * DEEP, PITCH = ROWS + TileEl<CT>::PAD, CPR = ROWS / V, NT = TILE_THREADS * DEEP,
                         CH = BK * CPR / NT, LDS = BK * PITCH, KSTEP = NT / CPR, XF = SCALE ? CH : 1;
    const elem *p;
    const float *kscale;
    i64 ld;
    int K, mc, shift, krow, kl, ks;
    static constexpr bool RUNS = SUM && sizeof(CT) == 4;
    float sum[SUM ? V : 1], total[RUNS ? V : 1];

    __device__ __forceinline__ void init(const void *p_, i64 ld_, int cols, int K_, int col0, int kbeg, int tid,
                                         const float *kscale_ = nullptr)
    {
        K = K_;
        ld = ld_;
        mc = (tid % CPR) * V;
        krow = tid / CPR;
        const int m = min(col0 + mc, cols - V);
        shift = col0 + mc - m;
        p = (const elem *)p_ + m;
        kscale = kscale_;
        kl = ks = kbeg;
        if (SUM) {
#pragma unroll
            for (int e = 0; e < V; ++e) sum[SUM ? e : 0] = total[RUNS ? e : 0] = 0.f;
        }
    }
    __device__ __forceinline__ void load(uint4 (&r)[CH], int (&x)[XF])
    {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int k = min(kl + krow + i * KSTEP, K - 1);
            r[i] = ldg16(p + (i64)k * ld);
            if (SCALE) x[SCALE ? i : 0] = kscale ? __float_as_int(kscale[k]) : 0;
        }
        kl += BK;
    }
    template <bool EDGE>
    __device__ __forceinline__ void store(elem *lds, uint4 (&r)[CH], int (&x)[XF])
    {
        const bool tail = EDGE && ks + BK > K;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            uint4 v = r[i];
            const int k = ks + krow + i * KSTEP;
            if (shift) v = piece_shift<sizeof(elem)>(v, shift);
            if (tail && k >= K) v = make_uint4(0, 0, 0, 0);
            if (SCALE && kscale) {
                const float s = __int_as_float(x[SCALE ? i : 0]);
                float f[8];
                piece_floats<CT>(v, f);
#pragma unroll
                for (int e = 0; e < V; ++e) f[e] *= s;
                v = floats_piece<CT>(f);
            }
            *(uint4 *)&lds[(krow + i * KSTEP) * PITCH + mc] = v;
            if (SUM) {
                float f[8];
                piece_floats<CT>(v, f);
#pragma unroll
                for (int e = 0; e < V; ++e) sum[SUM ? e : 0] += f[e];
            }
        }
        if (RUNS && (ks / BK & 15) == 15) {
#pragma unroll
            for (int e = 0; e < V; ++e) total[RUNS ? e : 0] += sum[SUM ? e : 0], sum[SUM ? e : 0] = 0.f;
        }
        ks += BK;
    }
    // column sums: the KSTEP threads that share columns meet in LDS (KSTEP * ROWS floats), added in a fixed order
    template <class PUT>
    __device__ __forceinline__ void put_sums(float *red, int tid, PUT put)
    {
#pragma unroll
        for (int e = 0; e < V; ++e) red[krow * ROWS + mc + e] = RUNS ? total[RUNS ? e : 0] + sum[SUM ? e : 0] : sum[SUM ? e : 0];
        __syncthreads();
        if (tid < ROWS) {
            float v = 0.f;
#pragma unroll
            for (int q = 0; q < KSTEP; ++q) v += red[q * ROWS + tid];
            put(tid, v);
        }
    }
};

// An operand that comes as up to TILE_MAX_SLICES partial sums in float, `stride` floats apart: the launch that formed them split its
// contraction, and the sum is taken on the way to LDS, in order, instead of by a launch of its own (3 to 4 us where the products
// themselves take 4 to 9).  All slices of a piece are requested together; one past the last re-reads the last and counts zero times.
constexpr int TILE_MAX_SLICES = 4;
template <typename CT>
struct SlicePiece {
    static constexpr int V = TileEl<CT>::V, W = V / 4, CH = TILE_MAX_SLICES * W; // 16-byte loads of a piece
    static __device__ __forceinline__ void load(const float *p, int slices, i64 stride, uint4 *r)
    {
#pragma unroll
        for (int s = 0; s < TILE_MAX_SLICES; ++s)
#pragma unroll
            for (int w = 0; w < W; ++w) r[s * W + w] = ldg16(p + min(s, slices - 1) * stride + 4 * w);
    }
    static __device__ __forceinline__ uint4 sum(const uint4 *r, int slices)
    {
        float v[V];
#pragma unroll
        for (int w = 0; w < W; ++w) piece_floats<float>(r[w], v + 4 * w);
#pragma unroll
        for (int s = 1; s < TILE_MAX_SLICES; ++s) {
            float t[V];
#pragma unroll
            for (int w = 0; w < W; ++w) piece_floats<float>(r[s * W + w], t + 4 * w);
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = s < slices ? v[e] + t[e] : v[e];
        }
        return floats_piece<CT>(v);
    }
};

// LoadKC of such an operand; copy (nullable): the sums leave once more, in the call's type and with the operand's leading dimension
template <typename CT, int ROWS, int DEEP = 1>
struct LoadKCS {
    typedef typename TileEl<CT>::elem elem;
    typedef SlicePiece<CT> SP;
    static constexpr bool KC = true;
    static constexpr int V = TileEl<CT>::V, BK = TileEl<CT>::BK * DEEP, PITCH = BK + TileEl<CT>::PAD, CPR = BK / V, NT = TILE_THREADS * DEEP,
                         P = ROWS * CPR / NT, CH = P * SP::CH, LDS = ROWS * PITCH, XF = 1;
    const float *rp[P];
    elem *copy;
    i64 ld, stride, jump;
    int K, kc, row, row0, rows, kl, ks, slices, seg;

    __device__ __forceinline__ void init(const void *p, i64 ld_, int rows_, int K_, int row0_, int kbeg, int tid, int slices_, i64 stride_,
                                         int seg_, i64 jump_, void *copy_)
    {
        ld = ld_, K = K_, rows = rows_, row0 = row0_, slices = slices_, stride = stride_, seg = seg_, jump = jump_;
        copy = (elem *)copy_;
        kc = (tid % CPR) * V;
        row = tid / CPR;
#pragma unroll
        for (int i = 0; i < P; ++i) rp[i] = (const float *)p + (i64)min(row0 + row + i * (NT / CPR), rows - 1) * ld;
        kl = ks = kbeg;
    }
    __device__ __forceinline__ void load(uint4 (&r)[CH], int (&x)[XF])
    {
        const int k = min(kl + kc, K - V);
        const i64 at = seg > 0 ? k + (k / seg) * (jump - seg) : k;
#pragma unroll
        for (int i = 0; i < P; ++i) SP::load(rp[i] + at, slices, stride, &r[i * SP::CH]);
        kl += BK;
    }
    template <bool EDGE>
    __device__ __forceinline__ void store(elem *lds, uint4 (&r)[CH], int (&x)[XF])
    {
        const int k = min(ks + kc, K - V), s = ks + kc - k;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            uint4 v = SP::sum(&r[i * SP::CH], slices);
            const int m = row0 + row + i * (NT / CPR);
            if (copy && m < rows) stg16(copy + (i64)m * ld + k, v); // (a piece that was pulled back holds what its neighbour writes)
            if (EDGE && s) v = piece_shift<sizeof(elem)>(v, s);
            *(uint4 *)&lds[(row + i * (NT / CPR)) * PITCH + kc] = v;
        }
        ks += BK;
    }
};

// LoadMC of such an operand
template <typename CT, int ROWS, int DEEP = 1>
struct LoadMCS {
    typedef typename TileEl<CT>::elem elem;
    typedef SlicePiece<CT> SP;
    static constexpr bool KC = false;
    static constexpr int V = TileEl<CT>::V, BK = TileEl<CT>::BK * DEEP, PITCH = ROWS + TileEl<CT>::PAD, CPR = ROWS / V, NT = TILE_THREADS * DEEP,
                         P = BK * CPR / NT, CH = P * SP::CH, LDS = BK * PITCH, KSTEP = NT / CPR, XF = 1;
    const float *p;
    i64 ld, stride;
    int K, mc, shift, krow, kl, ks, slices;

    __device__ __forceinline__ void init(const void *p_, i64 ld_, int cols, int K_, int col0, int kbeg, int tid, int slices_, i64 stride_)
    {
        K = K_, ld = ld_, slices = slices_, stride = stride_;
        mc = (tid % CPR) * V;
        krow = tid / CPR;
        const int m = min(col0 + mc, cols - V);
        shift = col0 + mc - m;
        p = (const float *)p_ + m;
        kl = ks = kbeg;
    }
    __device__ __forceinline__ void load(uint4 (&r)[CH], int (&x)[XF])
    {
#pragma unroll
        for (int i = 0; i < P; ++i) SP::load(p + (i64)min(kl + krow + i * KSTEP, K - 1) * ld, slices, stride, &r[i * SP::CH]);
        kl += BK;
    }
    template <bool EDGE>
    __device__ __forceinline__ void store(elem *lds, uint4 (&r)[CH], int (&x)[XF])
    {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            uint4 v = SP::sum(&r[i * SP::CH], slices);
            if (shift) v = piece_shift<sizeof(elem)>(v, shift);
            if (EDGE && ks + krow + i * KSTEP >= K) v = make_uint4(0, 0, 0, 0);
            *(uint4 *)&lds[(krow + i * KSTEP) * PITCH + mc] = v;
        }
        ks += BK;
    }
};

// ------------------------------------------------------------------ convolution operands
constexpr int TILE_MAX_TAPS = 25;

// An activation tensor [N][CH][plane] seen through a filter's taps over a grid of pixels gH x gW per image:
// (channel, tap, pixel (y, x)) is the element (y s + dy[tap], x s + dx[tap]) of the channel's H x W plane, or zero
// outside it.  Pixels of an image are padded to whole 16-byte pieces: pixel index = image * HC * V + position.
// Without stride, and with gW == W, the pixels of a piece are neighbours in memory whatever the tap, so a piece is
// one 16-byte load at an element offset plus a mask of the elements that lie in the plane.
struct PixView {
    const void *p;
    i64 total; // elements of the tensor
    int N, CH, H, W, gH, gW, s, HC, ntap;
    signed char dy[TILE_MAX_TAPS], dx[TILE_MAX_TAPS];
};

// (mask of the elements of the piece at position pos that the tap finds inside the plane)
template <int V>
__device__ __forceinline__ uint32_t pix_mask(const PixView &g, int pos, int tap)
{
    uint32_t m = 0;
    int y = pos / g.gW, x = pos - y * g.gW;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int iy = y * g.s + g.dy[tap], ix = x * g.s + g.dx[tap];
        if (y < g.gH && iy >= 0 && iy < g.H && ix >= 0 && ix < g.W) m |= 1u << e;
        if (++x == g.gW) x = 0, ++y;
    }
    return m;
}

// A 16-byte piece at element `off` of a tensor, off pulled back inside [0, last] (what is missing is shifted in later).
// 32-bit byte offsets from a uniform base: the address of a load is one register.
template <typename elem>
__device__ __forceinline__ uint4 ldg16_at(const elem *p, int off)
{
    return ldg16((const char *)p + (uint32_t)(off * (int)sizeof(elem)));
}

// With stride 2, and gW a multiple of a piece, the pixels of a piece are every second element from one on: two 16-byte loads,
// the second V - 1 elements after the first, hold them (the even ones of the first, the odd ones of the second).  What travels with
// the piece: the second load, where the two wanted to be, and which elements lie in the plane; at the ends of the tensor, where the
// loads were pulled back, the elements are fetched one by one when the piece is stored.
template <typename elem, int V>
struct Strided {
    static constexpr int XF = 6;
    static __device__ __forceinline__ void load(const elem *p, int off, int total, uint32_t keep, uint4 &r, int *x)
    {
        const int a = min(max(off, 0), max(total - (2 * V - 1), 0));
        r = ldg16_at(p, a);
        const uint4 t = ldg16_at(p, a + V - 1);
        x[0] = off, x[1] = (int)keep;
        x[2] = (int)t.x, x[3] = (int)t.y, x[4] = (int)t.z, x[5] = (int)t.w;
    }
    static __device__ __forceinline__ uint4 piece(const elem *p, int total, const unsigned char *lut, uint4 r, const int *x)
    {
        const int off = x[0];
        if (off < 0 || off + 2 * V - 1 > total) {
            elem v[V];
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = (x[1] >> e & 1) ? p[off + 2 * e] : elem(0);
            return *(const uint4 *)v;
        }
        const uint32_t t0 = x[2], t1 = x[3], t2 = x[4], t3 = x[5];
        if constexpr (sizeof(elem) == 4)
            r = make_uint4(r.x, r.z, t1, t3);
        else
            r = make_uint4((r.x & 0xffffu) | r.y << 16, (r.z & 0xffffu) | r.w << 16, t0 >> 16 | (t1 & 0xffff0000u), t2 >> 16 | (t3 & 0xffff0000u));
        return MaskTable<V>::apply(lut, (uint32_t)x[1], r);
    }
};

// B operand (k = (channel, tap), n = pixel): one tile row per k, pixels contiguous.  Tables in LDS: offset of every tap,
// mask of every (tap, piece of the tile).
template <typename CT, int ROWS, bool GATHER>
struct LoadPixMC {
    typedef typename TileEl<CT>::elem elem;
    static constexpr bool KC = false;
    static constexpr int V = TileEl<CT>::V, BK = TileEl<CT>::BK, PITCH = ROWS + TileEl<CT>::PAD, CPR = ROWS / V,
                         CH = BK * CPR / TILE_THREADS, LDS = BK * PITCH, KSTEP = TILE_THREADS / CPR, XF = GATHER ? 6 * CH : CH;
    static constexpr int TAPS = (TILE_MAX_TAPS + 3) / 4 * 16; // bytes of the offset table
    static constexpr int TAB = MaskTable<V>::BYTES + TAPS + TILE_MAX_TAPS * CPR;
    const elem *p;
    const unsigned char *tab;
    int pos0, last; // element of channel 0 at the piece's position; last element a piece may start at
    int HW, ntap, K, mc, col, krow, kl, ks, inc_c, inc_t;
    bool masked, pairs; // (pairs: strided pieces by two loads)
    int lc[CH], lt[CH]; // (first element of the channel, tap) of the rows to load next
    int pixoff[GATHER ? V : 1];

    __device__ __forceinline__ int toff(int t) const { return ((const int *)(tab + MaskTable<V>::BYTES))[t]; }
    __device__ __forceinline__ uint32_t tmask(int t) const { return tab[MaskTable<V>::BYTES + TAPS + t * CPR + col]; }

    // tab: TAB bytes of LDS; ends with a barrier
    __device__ __forceinline__ void init(const PixView &g, int n0, int kbeg, int tid, unsigned char *tab_)
    {
        p = (const elem *)g.p;
        tab = tab_;
        HW = g.H * g.W;
        ntap = g.ntap;
        K = g.CH * g.ntap;
        col = tid % CPR;
        mc = col * V;
        krow = tid / CPR;
        masked = g.ntap > 1 || g.gH * g.gW % V != 0 || GATHER;
        if (tid < g.ntap) ((int *)(tab_ + MaskTable<V>::BYTES))[tid] = g.dy[tid] * g.W + g.dx[tid];
        if (masked) {
            MaskTable<V>::build(tab_, tid);
            for (int j = tid; j < g.ntap * CPR; j += TILE_THREADS) {
                const int t = j / CPR, c = n0 / V + j % CPR;
                tab_[MaskTable<V>::BYTES + TAPS + j] = (unsigned char)pix_mask<V>(g, c % g.HC * V, t);
            }
        }
        const int cidx = n0 / V + col, img = min(cidx / g.HC, g.N - 1), pos = cidx % g.HC * V;
        pos0 = img * g.CH * HW;
        if (GATHER) {
            int y = pos / g.gW, x = pos - y * g.gW;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                pixoff[GATHER ? e : 0] = y * g.s * g.W + x * g.s;
                if (++x == g.gW) x = 0, ++y;
            }
        } else {
            pos0 += pos;
        }
        last = (int)g.total - V;
        pairs = GATHER && g.s == 2 && g.gW % V == 0 && g.total >= 2 * V - 1;
        inc_c = BK / g.ntap;
        inc_t = BK - inc_c * g.ntap;
        inc_c *= HW;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int k = kbeg + krow + i * KSTEP, c = k / g.ntap;
            lc[i] = c * HW;
            lt[i] = k - c * g.ntap;
        }
        kl = ks = kbeg;
        __syncthreads();
    }
    __device__ __forceinline__ void load(uint4 (&r)[CH], int (&x)[XF])
    {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int off = pos0 + lc[i] + toff(lt[i]);
            if (GATHER && pairs) {
                const uint32_t m = kl + krow + i * KSTEP < K ? tmask(lt[i]) : 0u;
                Strided<elem, V>::load(p, off + pixoff[0], last + V, m, r[i], &x[GATHER ? 6 * i : 0]);
            } else if (GATHER) {
                const uint32_t m = kl + krow + i * KSTEP < K ? tmask(lt[i]) : 0u;
                elem v[V];
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] = (m >> e & 1) ? p[off + pixoff[GATHER ? e : 0]] : elem(0);
                r[i] = *(const uint4 *)v;
            } else {
                const int a = min(max(off, 0), last);
                r[i] = ldg16_at(p, a);
                // the tap, and how far the piece was pulled back (rows past K: anything, they become zero)
                x[i] = (min(max(off - a, -V), V) + V) << 8 | lt[i];
            }
            lc[i] += inc_c;
            lt[i] += inc_t;
            if (lt[i] >= ntap) {
                lt[i] -= ntap;
                lc[i] += HW;
            }
        }
        kl += BK;
    }
    template <bool EDGE>
    __device__ __forceinline__ void store(elem *lds, uint4 (&r)[CH], int (&x)[XF])
    {
        const bool tail = EDGE && ks + BK > K;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            uint4 v = r[i];
            if (GATHER && pairs) v = Strided<elem, V>::piece(p, last + V, tab, v, &x[GATHER ? 6 * i : 0]);
            if (!GATHER) {
                const int s = (x[i] >> 8) - V;
                if (s != 0) v = piece_shift<sizeof(elem)>(v, s);
                if (masked) v = MaskTable<V>::apply(tab, tmask(x[i] & 255), v);
                if (tail && ks + krow + i * KSTEP >= K) v = make_uint4(0, 0, 0, 0);
            }
            *(uint4 *)&lds[(krow + i * KSTEP) * PITCH + mc] = v;
        }
        ks += BK;
    }
};

// Weight gradients: row = (channel, tap), k = pixel.  The contraction runs over the pieces of whole images
// [img0, img1).  Tables in LDS: mask of every (tap, piece of a plane), with stride also the offset of every pixel.
template <typename CT, int ROWS, bool GATHER, bool SUM = false>
struct LoadPixKC {
    typedef typename TileEl<CT>::elem elem;
    static constexpr bool KC = true;
    static constexpr int V = TileEl<CT>::V, BK = TileEl<CT>::BK, PITCH = BK + TileEl<CT>::PAD, CPR = BK / V,
                         CH = ROWS * CPR / TILE_THREADS, LDS = ROWS * PITCH, XF = 1;
    const elem *p;
    const unsigned char *lut, *tmask;
    const int *pix;
    int image, last, HC, N, img1, kc, row, limg, lpc, simg, spc;
    bool masked;
    int ro[CH], tap[CH]; // offset of the row's channel and tap; first mask of the tap
    float sum[SUM ? CH : 1];

    static __host__ __device__ int table_bytes(const PixView &g)
    {
        return (g.ntap > 1 || g.gH * g.gW % V != 0 || GATHER ? MaskTable<V>::BYTES + (g.ntap * g.HC + 15) / 16 * 16 : 0) +
               (GATHER ? 4 * V * g.HC : 0);
    }
    // tab: table_bytes() of LDS; the caller's barrier follows
    __device__ __forceinline__ void init(const PixView &g, int row0, int img0, int img1_, int tid, unsigned char *tab)
    {
        p = (const elem *)g.p;
        HC = g.HC;
        N = g.N;
        img1 = img1_;
        kc = (tid % CPR) * V;
        row = tid / CPR;
        masked = g.ntap > 1 || g.gH * g.gW % V != 0 || GATHER;
        const int HW = g.H * g.W;
        image = g.CH * HW;
        last = (int)g.total - V;
        lut = tab;
        tmask = tab + MaskTable<V>::BYTES;
        pix = (const int *)(tmask + (g.ntap * g.HC + 15) / 16 * 16);
        if (masked) {
            MaskTable<V>::build(tab, tid);
            for (int j = tid; j < g.ntap * HC; j += TILE_THREADS)
                tab[MaskTable<V>::BYTES + j] = (unsigned char)pix_mask<V>(g, j % HC * V, j / HC);
        }
        if (GATHER)
            for (int j = tid; j < HC * V; j += TILE_THREADS)
                ((int *)pix)[j] = (j / g.gW) * g.s * g.W + (j % g.gW) * g.s;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = min(row0 + row + i * (TILE_THREADS / CPR), g.CH * g.ntap - 1);
            const int c = r / g.ntap, t = r - c * g.ntap;
            tap[i] = t * HC;
            ro[i] = c * HW + g.dy[t] * g.W + g.dx[t];
            if (SUM) sum[i] = 0.f;
        }
        limg = img0;
        lpc = tid % CPR;
        wrap(limg, lpc);
        simg = limg;
        spc = lpc;
    }
    __device__ __forceinline__ void wrap(int &img, int &pc)
    {
        while (pc >= HC) pc -= HC, ++img;
    }
    __device__ __forceinline__ void load(uint4 (&r)[CH], int (&x)[XF])
    {
        const int b = min(limg, N - 1) * image + (GATHER ? 0 : lpc * V);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (GATHER) {
                const uint32_t m = limg < img1 ? tmask[tap[i] + lpc] : 0u;
                elem v[V];
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] = (m >> e & 1) ? p[b + ro[i] + pix[lpc * V + e]] : elem(0);
                r[i] = *(const uint4 *)v;
            } else {
                r[i] = ldg16_at(p, min(max(b + ro[i], 0), last));
            }
        }
        lpc += CPR;
        wrap(limg, lpc);
    }
    template <bool EDGE>
    __device__ __forceinline__ void store(elem *lds, uint4 (&r)[CH], int (&x)[XF])
    {
        const int b = min(simg, N - 1) * image + spc * V;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            uint4 v = r[i];
            if (!GATHER) {
                const int off = b + ro[i], s = off - min(max(off, 0), last);
                if (s != 0) v = piece_shift<sizeof(elem)>(v, min(max(s, -V), V));
                if (masked) v = MaskTable<V>::apply(lut, tmask[tap[i] + spc], v);
                if (EDGE && simg >= img1) v = make_uint4(0, 0, 0, 0);
            }
            *(uint4 *)&lds[(row + i * (TILE_THREADS / CPR)) * PITCH + kc] = v;
            if (SUM) {
                float f[8];
                piece_floats<CT>(v, f);
#pragma unroll
                for (int e = 0; e < V; ++e) sum[SUM ? i : 0] += f[e];
            }
        }
        spc += CPR;
        wrap(simg, spc);
    }
    template <class PUT>
    __device__ __forceinline__ void put_sums(float *, int, PUT put)
    {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            float v = sum[SUM ? i : 0];
#pragma unroll
            for (int d = 1; d < CPR; d <<= 1) v += __shfl_xor(v, d, 64);
            if (kc == 0) put(row + i * (TILE_THREADS / CPR), v);
        }
    }
};

// ------------------------------------------------------------------ fragments
// 8 (bf16) or 4 (float) values of row / column c0 + lane % 32 at k = step * 16 (8) + (lane / 32) * 8 (4) ..
template <bool KC, int PITCH>
__device__ __forceinline__ bf16x8_t tile_frag(const uint16_t *lds, int c0, int step, int lane)
{
    if (KC) return *(const bf16x8_t *)&lds[(c0 + (lane & 31)) * PITCH + step * 16 + (lane >> 5) * 8];
    return lds_frag_tr(lds, PITCH, step * 16, c0, lane);
}
template <bool KC, int PITCH>
__device__ __forceinline__ f32x4_t tile_frag(const float *lds, int c0, int step, int lane)
{
    if (KC) return *(const f32x4_t *)&lds[(c0 + (lane & 31)) * PITCH + step * 8 + (lane >> 5) * 4];
    const float *q = &lds[(step * 8 + (lane >> 5) * 4) * PITCH + c0 + (lane & 31)];
    f32x4_t f = {q[0], q[PITCH], q[2 * PITCH], q[3 * PITCH]};
    return f;
}

// ------------------------------------------------------------------ the product
template <typename CT, class CFG, class LA, class LB>
struct TileSize {
    static constexpr int loop = 2 * (LA::LDS + LB::LDS) * (int)sizeof(typename TileEl<CT>::elem);
    static constexpr int cpitch = CFG::BN + 4;
    static constexpr int out = CFG::WK * CFG::BM * cpitch * 4;
    static constexpr int bytes = loop > out ? loop : out;
};

// nch chunks; the sums end up in smem as WK tiles [BM][BN + 4] of floats (ends with a barrier)
template <typename CT, class CFG, class LA, class LB>
__device__ __forceinline__ void tile_product(LA &la, LB &lb, int nch, unsigned char *smem, int tid)
{
    typedef typename TileEl<CT>::elem elem;
    constexpr int NS = CFG::NS, MI = CFG::BM / 32 / CFG::WM, NI = CFG::BN / 32 / CFG::WN;
    constexpr int STEPS = 4 * CFG::DEEP / CFG::WK; // a chunk has four steps, or DEEP times that
    static_assert(NS % 2 == 0, "the LDS buffer of a stage is its parity");
    elem *As[2], *Bs[2];
    As[0] = (elem *)smem;
    As[1] = As[0] + LA::LDS;
    Bs[0] = As[1] + LA::LDS;
    Bs[1] = Bs[0] + LB::LDS;
    const int lane = tid & 63, wave = tid >> 6;
    const int wk = wave / (CFG::WM * CFG::WN), wm = wave / CFG::WN % CFG::WM, wn = wave % CFG::WN;
    uint4 ra[NS][LA::CH], rb[NS][LB::CH];
    int xa[NS][LA::XF], xb[NS][LB::XF];
    f32x16_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    auto load = [&](int st) __attribute__((always_inline)) {
        la.load(ra[st], xa[st]);
        lb.load(rb[st], xb[st]);
    };
    auto compute = [&](int cur) __attribute__((always_inline)) {
        if constexpr (sizeof(elem) == 2) {
#pragma unroll
            for (int q = 0; q < STEPS; ++q) {
                const int step = wk * STEPS + q;
                bf16x8_t a[MI], b[NI];
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    a[i] = tile_frag<LA::KC, LA::PITCH>(As[cur], (wm * MI + i) * 32, step, lane);
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    b[j] = tile_frag<LB::KC, LB::PITCH>(Bs[cur], (wn * NI + j) * 32, step, lane);
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        } else {
            f32x4_t a[STEPS][MI], b[STEPS][NI];
#pragma unroll
            for (int q = 0; q < STEPS; ++q) {
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    a[q][i] = tile_frag<LA::KC, LA::PITCH>(As[cur], (wm * MI + i) * 32, wk * STEPS + q, lane);
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    b[q][j] = tile_frag<LB::KC, LB::PITCH>(Bs[cur], (wn * NI + j) * 32, wk * STEPS + q, lane);
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    f32x16_t t;
#pragma unroll
                    for (int v = 0; v < 16; ++v) t[v] = 0.f;
#pragma unroll
                    for (int q = 0; q < STEPS; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            t = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][i][e], b[q][j][e], t, 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] += t[v];
                }
        }
    };
#define TILE_STORE(EDGE, st)                                      \
    {                                                             \
        la.template store<EDGE>(As[(st) & 1], ra[(st) % NS], xa[(st) % NS]); \
        lb.template store<EDGE>(Bs[(st) & 1], rb[(st) % NS], xb[(st) % NS]); \
    }
    if (nch > NS) {
#pragma unroll
        for (int s = 0; s < NS; ++s) load(s);
        TILE_STORE(false, 0)
        load(0);
        __syncthreads();
        int c = 0;
        for (; c + NS + 1 < nch; c += NS) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                TILE_STORE(false, s + 1)
                load((s + 1) % NS); // (past the last chunk in the last round: read, never used)
                compute(s & 1);
                __syncthreads();
            }
        }
#pragma unroll
        for (int s = 0; s <= NS; ++s) {
            if (c + s < nch) {
                if (s < NS && c + s + 1 < nch) TILE_STORE(true, s + 1)
                compute(s & 1);
                __syncthreads();
            }
        }
    } else { // (an empty contraction reads nothing)
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (s < nch) load(s);
        if (nch > 0) TILE_STORE(true, 0)
        __syncthreads();
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (s < nch) {
                if (s + 1 < NS && s + 1 < nch) TILE_STORE(true, s + 1)
                compute(s & 1);
                __syncthreads();
            }
        }
    }
#undef TILE_STORE
    float *Cs = (float *)smem + wk * CFG::BM * (CFG::BN + 4);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = (wm * MI + i) * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
                Cs[m * (CFG::BN + 4) + (wn * NI + j) * 32 + (lane & 31)] = acc[i][j][v];
            }
    __syncthreads();
}

// out(m, n, v[V]) for every piece of V neighbouring columns of the tile, in tile coordinates
template <typename CT, class CFG, class OUT>
__device__ __forceinline__ void tile_pieces(const unsigned char *smem, int tid, OUT out)
{
    constexpr int V = TileEl<CT>::V, CPR = CFG::BN / V, P = CFG::BN + 4;
    const float *Cs = (const float *)smem;
#pragma unroll 2
    for (int q = tid; q < CFG::BM * CPR; q += TILE_THREADS * CFG::DEEP) {
        const int m = q / CPR, n = q % CPR * V;
        float v[V];
#pragma unroll
        for (int e = 0; e < V; e += 4) {
            f32x4_t t = *(const f32x4_t *)&Cs[m * P + n + e];
#pragma unroll
            for (int w = 1; w < CFG::WK; ++w) t += *(const f32x4_t *)&Cs[(w * CFG::BM + m) * P + n + e];
#pragma unroll
            for (int x = 0; x < 4; ++x) v[e + x] = t[x];
        }
        out(m, n, v);
    }
}

} // namespace pf
