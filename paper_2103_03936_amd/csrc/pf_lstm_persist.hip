// The recurrence of a stack of LSTM layers, small batches, fp32: one cooperative launch per direction, the factors in registers.
//
// A step of the recurrence is two dependent products with an exchange over the whole chip after each.  As launches
// (pf_lstm_stack.hip) a slot of the wavefront schedule is three to five of them, each of which reads its factors again: at
// 1500 units, rank 375, two layers, 43 MB per slot, 24 us.  Here the workgroups stay, and every one keeps the tile of the factors
// that its columns need in its wavefronts' registers (the 43 MB are 170 KB of a compute unit's 512) for all steps.  A slot is two
// phases; what crosses a phase is written past the L2 of the writer's die (agent-scope stores, complete before the
// workgroup arrives) to addresses that nobody has read before in this launch: every step has its own copy, in whole cache
// lines.  So the readers need no cache invalidation, and share a line through their own L2.
//
// Products run on v_mfma_f32_4x4x1_16b_f32: four rows (batch) by 16 columns by four contraction indices, or 8 columns by
// eight, with one row block broadcast within a group of lanes.  Batch 20 is then five row blocks (as 16 x 16 x 4 it would be
// padded to 32: 21 ns instead of 29 for the same weights).  The contraction is split over the lane groups and over the eight
// wavefronts of a workgroup, so each reads only its share of the exchanged activations, in the lanes' own order, and no LDS is
// needed before the sum.
//
// Between phases a wavefront waits for the tasks whose results it reads, and for no others: a task that is done stores the
// slot's number to its flag, in eight copies, and the readers poll the flags of those that fill their contraction indices (2 at
// 128 units, 48 at most), those of a die in one copy.  Before, a barrier over all workgroups (arrivals counted in eight groups,
// whose last tell eight copies of the group flags) cost 1.9 us a phase: an atomic's round trip more, and everybody waited for the
// slowest.  Whole calls, us: 1500 units, two layers, batch 20, 35 steps 1266 -> 1242; 650 units 818 -> 762; 256 units, three
// layers, batch 4, 70 steps 865 -> 762.
// (One copy of the flags: 1376; the pollers get in each other's way.)  What a slot of 11 us consists of now at 1500 units, forward:
// two hand-overs of 0.9, the first reads of what was handed over 0.8 each, matrix instructions 0.8 and 2.4, the wavefronts' sums 0.3
// and 0.6, gates 0.7.
#include "pf_lstm_persist_index.h"


namespace pf {

int launch_zero_f32(hipStream_t s, float *p, i64 n);

// The argument block where the launch put it (indexed by layer, the by-value copy would go to scratch memory).
__device__ __forceinline__ const LpArgs &lp_args(const LpArgs &a)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const LpArgs *)(const __attribute__((address_space(4))) LpArgs *)__builtin_amdgcn_kernarg_segment_ptr();
#else
    return a;
#endif
}

__device__ __forceinline__ float lp_sigmoid(float z) { return 1.0f / (1.0f + expf(-z)); }
__device__ __forceinline__ void lp_share(float *p, float v) // a store that other dies' first read of the line will see
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ phases
// The end of a task's part of a slot: everything that the workgroup has shared is visible, then its flag (all threads)
__device__ __forceinline__ void lp_publish(unsigned *flags, int flag, unsigned epoch)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
    __syncthreads();
    if (threadIdx.x < LP_GROUPS) __hip_atomic_store(flags + threadIdx.x * LP_COPY + flag, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// All workgroups of a cooperative launch are resident, so every flag comes; a wait is bounded all the same (by polls, of
// about a microsecond each: a process that is suspended does not count), and everyone leaves when one gives up, with NaN in
// what it has not written.
__device__ __forceinline__ bool lp_poll(const unsigned *flag, unsigned epoch, unsigned *failed)
{
    bool good = false;
    for (int spin = 0; spin < 4000000; ++spin) {
        const unsigned v = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!__any((int)(v - epoch) < 0)) {
            good = true;
            break;
        }
        if ((spin & 255) == 255 && __hip_atomic_load(failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
    }
    if (!good && (threadIdx.x & 63) == 0) __hip_atomic_store(failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" ::: "memory"); // no read of shared data before this
#endif
    return good;
}
// A wavefront's wait; *ok (LDS, 1 at first) tells the workgroup after its next __syncthreads
__device__ __forceinline__ void lp_await(const unsigned *flag, unsigned epoch, unsigned *failed, int *ok)
{
    if (!lp_poll(flag, epoch, failed)) *ok = 0;
}

// A barrier of n workgroups, once in a launch: they count arrivals in eight groups (an atomic each on a line of its own), the last
// of a group tells eight copies of the group flags, and everybody polls one of the copies.
struct LpSync {
    unsigned *base;
    int wg;
    int *ok; // LDS

    // everything this workgroup has shared is visible; then it counts itself in (all threads)
    __device__ __forceinline__ void arrive(int n)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
        __syncthreads();
        if (threadIdx.x < 64) {
            const int g = wg % LP_GROUPS, members = n / LP_GROUPS; // (n: a multiple)
            unsigned *flags = base + LP_GROUPS * 64;
            int before = 0;
            if (threadIdx.x == 0)
                before = (int)__hip_atomic_fetch_add(base + g * 64, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            before = __builtin_amdgcn_readfirstlane(before);
            if (before == members - 1 && threadIdx.x < LP_GROUPS)
                __hip_atomic_store(flags + threadIdx.x * 64 + g, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __device__ __forceinline__ bool wait()
    {
        if (threadIdx.x < 64) {
            const unsigned *flags = base + LP_GROUPS * 64 + (wg % LP_GROUPS) * 64;
            const bool good = lp_poll(flags + min((int)threadIdx.x, LP_GROUPS - 1), 1u, base + LP_FAILED);
            if (threadIdx.x == 0) *ok = good;
        }
        __syncthreads();
        const bool all = *ok != 0;
        __syncthreads(); // (nobody clears it before all have read it)
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" ::: "memory"); // no read of shared data before this
#endif
        return all;
    }
};

// ------------------------------------------------------------------ a wavefront's product
// Exchanged matrices [4 RB rows][K]: groups of 32 indices, in each the row blocks, in each 16 index pairs of four rows: lane
// 4 p + i of a wavefront reads row i, indices 2 p and 2 p + 1 of a group as eight bytes.
template <int RB>
__device__ __forceinline__ int lp_place(int k, int m)
{
    return ((k >> 5) * RB + (m >> 2)) * 128 + ((k >> 1) & 15) * 8 + (m & 3) * 2 + (k & 1);
}
// The instruction's A operand comes from one lane of each group of four (block) in 4 << (CB - 2)... lanes: with CB = 2 four
// groups of 16 lanes, each with 16 columns and its own four index pairs; with CB = 1 eight groups of 8 lanes, 8 columns, two
// index pairs.  weights [tile][group][s + 2 b]: index 2 p + s of the group, p = (lane group) 2^CB + b.
template <int NT, int KG, int CB, class F>
__device__ __forceinline__ void lp_weights(float (&w)[NT][KG][2 << CB], int g0, int ng, F at)
{
    const int lane = threadIdx.x & 63, col = lane & ((4 << CB) - 1), lg = lane >> (2 + CB);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int j = 0; j < (2 << CB); ++j) {
                w[nt][g][j] = 0.f;
                if (g < ng) w[nt][g][j] = at(nt, g0 + g, 2 * ((lg << CB) + (j >> 1)) + (j & 1), col);
            }
}
// The same where a column's indices are contiguous: row(nt, g, col, in) is the address of group g's first, in: the column exists;
// left(g): how many of the group's indices exist.  16 columns: a lane's eight weights of a group are neighbours.
template <int NT, int KG, class ROW, class LEFT>
__device__ __forceinline__ void lp_weights_rows(float (&w)[NT][KG][8], int g0, int ng, ROW row, LEFT left)
{
    struct __attribute__((packed, aligned(4))) F4 {
        float f[4];
    };
    const int lane = threadIdx.x & 63, o = (lane >> 4) * 8;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            float v[8] = {};
            bool in = false;
            if (g < ng) {
                const float *p = row(nt, g0 + g, lane & 15, in);
                const int n = left(g0 + g);
                if (n >= 32) {
                    const F4 x = *(const F4 *)(p + o), y = *(const F4 *)(p + o + 4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = x.f[j], v[4 + j] = y.f[j];
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float x = p[min(o + j, n - 1)];
                        v[j] = o + j < n ? x : 0.f;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) w[nt][g][j] = in ? v[j] : 0.f;
        }
}
// acc[nt][rb] += (sum of the SL slices, ss apart, of A)[rows 4 rb..][groups 0 .. ng - 1 from A on] W; D groups of A are in flight
template <int CB, int J>
__device__ __forceinline__ f32x4_t lp_mfma(float a, float b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, CB, J, 0);
}
template <int CB>
__device__ __forceinline__ f32x4_t lp_mfma_block(int b, float x, float w, f32x4_t c)
{
    if (b == 0) return lp_mfma<CB, 0>(x, w, c);
    if (b == 1) return lp_mfma<CB, 1>(x, w, c);
    if constexpr (CB == 2) return b == 2 ? lp_mfma<CB, 2>(x, w, c) : lp_mfma<CB, 3>(x, w, c);
    return c;
}
struct alignas(8) LpPair {
    float f[2];
};
template <int RB, int D, int SL>
__device__ __forceinline__ void lp_load(LpPair (&a)[D][RB][SL], int d, const float *A, int ss, int g, int ng)
{
    const float *p = A + min(g, ng - 1) * (RB * 128);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int sl = 0; sl < SL; ++sl) a[d][rb][sl] = *(const LpPair *)(p + sl * ss + rb * 128 + (threadIdx.x & 63) * 2);
}
// groups G .. of the product (a recursion: a loop with an exit in it is not unrolled, and the weights would go to scratch memory)
template <int CB, int G, int D, int SL, int NT, int RB, int KG>
__device__ __forceinline__ void lp_groups(f32x4_t (&acc)[NT][RB], const float (&w)[NT][KG][2 << CB], LpPair (&a)[D][RB][SL], int ntn, const float *A,
                                          int ss, int ng)
{
    if constexpr (G < KG) {
        if (G >= ng) return;
        LpPair x[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            x[rb] = a[G % D][rb][0];
#pragma unroll
            for (int sl = 1; sl < SL; ++sl) x[rb].f[0] += a[G % D][rb][sl].f[0], x[rb].f[1] += a[G % D][rb][sl].f[1];
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (NT == 1 || nt < ntn) {
#pragma unroll
                for (int j = 0; j < (2 << CB); ++j)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        acc[nt][rb] = lp_mfma_block<CB>(j >> 1, x[rb].f[j & 1], w[nt][G][j], acc[nt][rb]);
            }
        }
        if constexpr (G + D < KG) lp_load(a, G % D, A, ss, G + D, ng);
        lp_groups<CB, G + 1>(acc, w, a, ntn, A, ss, ng);
    }
}
template <int CB, int D, int SL, int NT, int RB, int KG>
__device__ __forceinline__ void lp_multiply(f32x4_t (&acc)[NT][RB], const float (&w)[NT][KG][2 << CB], int ntn, const float *A, int ss, int ng)
{
    if (ng <= 0) return;
    LpPair a[D][RB][SL];
#pragma unroll
    for (int d = 0; d < D; ++d) lp_load(a, d, A, ss, d, ng);
    lp_groups<CB, 0>(acc, w, a, ntn, A, ss, ng);
}

template <int NT, int RB>
__device__ __forceinline__ void lp_zero(f32x4_t (&t)[NT][RB])
{
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) t[nt][rb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
}

// A tile's four accumulators (rows) are summed over the lane groups: lanes 16 q + c keep column c of row {0, 2, 1, 3}[q].
template <int CB>
__device__ __forceinline__ float lp_fold(f32x4_t v)
{
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[1]), false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2]), __float_as_uint(v[3]), false, false);
    const float s = __uint_as_float(x[0]) + __uint_as_float(x[1]), t = __uint_as_float(y[0]) + __uint_as_float(y[1]);
    const auto z = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(t), false, false);
    float u = __uint_as_float(z[0]) + __uint_as_float(z[1]);
    if (CB == 1) // (8 columns: both halves of a row of 16 lanes hold sums)
        u += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(u), 0x128, 0xf, 0xf, false));
    return u;
}
__device__ __forceinline__ int lp_lane(int m, int c) { return ((m & 1) << 1 | (m >> 1 & 1)) * 16 + c; }
// The wavefronts' tiles meet in LDS: red[wavefront][NT][RB][64]
template <int CB, int NT, int RB>
__device__ __forceinline__ void lp_exchange(float *red, const f32x4_t (&acc)[NT][RB])
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) red[((w * NT + nt) * RB + rb) * 64 + lane] = lp_fold<CB>(acc[nt][rb]);
    __syncthreads();
}
template <int NT, int RB>
__device__ __forceinline__ float lp_sum(const float *red, int nt, int m, int c)
{
    const float *p = red + (nt * RB + (m >> 2)) * 64 + lp_lane(m, c);
    float s[LP_WAVES];
#pragma unroll
    for (int w = 0; w < LP_WAVES; ++w) s[w] = p[w * NT * RB * 64];
    return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// element o of an exchanged matrix: row m, index k
template <int RB>
__device__ __forceinline__ void lp_element(int o, int &k, int &m)
{
    k = (o / (128 * RB)) * 32 + ((o >> 3) & 15) * 2 + (o & 1);
    m = ((o >> 7) % RB) * 4 + ((o >> 1) & 3);
}
// T (or dT) of one task: TN tiles of TW columns from col0 on, to the exchange and (out, whole sums only) to the tensor that is kept
template <int TN, int TW, int RB>
__device__ __forceinline__ void lp_put_T(const LpArgs &a, const float *red, float *xt, float *out, int col0, int ncol)
{
#pragma unroll
    for (int it = 0; it < (TN * TW * 4 * RB + LP_NT - 1) / LP_NT; ++it) {
        const int e = threadIdx.x + LP_NT * it, pr = e >> 3, nt = pr / (TW / 2 * RB), rb = (pr / (TW / 2)) % RB;
        const int c = pr % (TW / 2) * 2 + (e & 1), m = 4 * rb + ((e >> 1) & 3), cp = col0 + TW * nt + c;
        if (nt < TN && TW * nt < ncol) {
            const float v = lp_sum<TN, RB>(red, nt, m, c);
            lp_share(xt + lp_place<RB>(cp, m), v);
            if (out) {
                const int q = cp / a.rp, cc = cp - q * a.rp;
                if (m < a.B && cc < a.r) out[(i64)m * a.gr + q * a.r + cc] = v;
            }
        }
    }
}

// groups of A in flight: as registers allow beside the weights of both phases and the accumulators
constexpr int lp_depth(int RB, int KG, int NT, int weights, int SL = 1)
{
    int d = (190 - weights - 4 * NT * RB) / (2 * RB * SL);
    const int most = (SL == 1 ? 64 : 96) / (2 * RB * SL);
    if (d > most) d = most;
    if (d > KG) d = KG;
    return d < 1 ? 1 : d;
}

// ------------------------------------------------------------------ forward
// Slot s handles the layers l with a step t = s - l: first T = h_{t-1} Vh (and x_t Vx above the first layer), then
// z = Th Uh^T + Tx Ux^T + b with eq. (2) where z is formed: a workgroup owns 4 NT units (one factor pair for all gates: a tile is
// four units by four gates, wavefronts 0-3 have Th, 4-7 Tx, a quarter of the contraction each) or 16 (a pair per gate: wavefront
// w has gate w % 4 of path w / 4).  c_t stays with its thread.
template <int RB, int NT, bool G4>
__global__ __launch_bounds__(LP_NT) void lstm_run_fwd_kernel(LpArgs by_value)
{
    constexpr int TN = G4 ? 3 : 1, TKG = 6, KG = G4 ? 12 : 3, U = G4 ? 16 : 4 * NT;
    constexpr int WR = TN * TKG * 4 + NT * KG * 8;
    const LpArgs &a = lp_args(by_value);
    __shared__ __attribute__((aligned(16))) float red[LP_WAVES * (NT > TN ? NT : TN) * RB * 64];
    __shared__ int ok;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), wg = blockIdx.x;
    const int T = a.T, B = a.B, BT = a.BT, h = a.h, r = a.r, gr = a.gr, L = a.L, hp = a.hp, rp = a.rp, G = G4 ? 4 : 1;
    LpSync sync = {a.sync, wg, &ok};
    unsigned *flags = a.sync + LP_BAR, *failed = a.sync + LP_FAILED;
    const bool in2 = wg < a.n2;
    // the initial states and the first layer's Tx into the lanes' order
    if (in2) {
        // (the few states by the last workgroups, which have one element less of the other)
        for (LpWalk at(hp * 4 * RB, (a.n2 - 1 - wg) * LP_NT + tid, a.n2 * LP_NT); at.row < L; at.next()) {
            int k, m;
            lp_element<RB>(at.o, k, m);
            const float v = a.l[at.row].h0[(i64)min(m, B - 1) * h + min(k, h - 1)];
            lp_share(lp_xh(a, at.row, 0) + at.o, k < h ? v : 0.f);
        }
        for (LpWalk at(G * rp * 4 * RB, wg * LP_NT + tid, a.n2 * LP_NT); at.row < T; at.next()) {
            int k, m;
            lp_element<RB>(at.o, k, m);
            const int q = k / rp, cc = k - q * rp;
            const float v = a.l[0].Tx[((i64)at.row * BT + min(m, B - 1)) * gr + q * r + min(cc, r - 1)];
            lp_share(lp_xt(a, 0, 1, at.row) + at.o, cc < r ? v : 0.f);
        }
        sync.arrive(a.n2);
    }
    // phase 1: columns tcol .. tcol + tncol - 1 of a product; groups tg0 .. of h
    const LpColumns cols = lp_columns(a, wg, a.n1, G * rp, 8, 1);
    const bool has1 = cols.has;
    const int tl = cols.l, tpath = cols.path, tcol = cols.col, tncol = cols.n;
    const LpShare share1 = lp_fwd_share1(a, cols, w, U);
    const int tg0 = share1.first, tng = share1.n;
    float wt[TN][TKG][4];
    {
        const float *V = tpath ? a.l[tl].Vx : a.l[tl].Vh;
        lp_weights<TN, TKG, 1>(wt, tg0, tng, [&](int nt, int g, int i, int c) __attribute__((always_inline)) {
            const int q = (tcol + 8 * nt) / rp, cc = tcol + 8 * nt - q * rp + c, k = 32 * g + i;
            const float v = V[(i64)min(k, h - 1) * gr + min(q, G - 1) * r + min(cc, r - 1)];
            return k < h && q < G && cc < r && 8 * nt < tncol ? v : 0.f;
        });
    }
    // phase 2: units u0 .. of layer zl
    const LpUnits units = lp_units(a, wg, a.n2, U);
    const bool has2 = units.has;
    const LpShare share2 = lp_fwd_share2(a, units, w);
    const int zl = units.l, u0 = units.u0, zx = w >> 2, zg0 = share2.first, zng = share2.n;
    float wz[NT][KG][8];
    {
        const float *Um = zx ? a.l[zl].Ux : a.l[zl].Uh;
        lp_weights_rows<NT, KG>(
            wz, zg0, zng,
            [&](int nt, int g, int c, bool &in) __attribute__((always_inline)) {
                const int unit = G4 ? u0 + c : u0 + 4 * nt + (c >> 2), q = G4 ? w & 3 : c & 3;
                in = unit < h;
                return Um + ((i64)q * h + min(unit, h - 1)) * r + 32 * g - (G4 ? (w & 3) * rp : 0);
            },
            [&](int g) __attribute__((always_inline)) { return r - 32 * g + (G4 ? (w & 3) * rp : 0); });
    }
    // its elements: row m, unit un of thread tid (at most one: U 4 RB <= threads)
    const int ekp = (tid >> 3) % (U / 2), eu = ekp * 2 + (tid & 1), em = ((tid >> 3) / (U / 2)) * 4 + ((tid >> 1) & 3), un = u0 + eu;
    const bool el = has2 && em < 4 * RB && un < hp, kept = el && em < B && un < h;
    float pb[4] = {0.f, 0.f, 0.f, 0.f}, c_prev = 0.f;
    if (kept) {
        c_prev = a.l[zl].c0[(i64)em * h + un];
#pragma unroll
        for (int g = 0; g < 4; ++g) pb[g] = a.l[zl].bias ? a.l[zl].bias[(i64)g * h + un] : 0.f;
    }
    const unsigned *mine = flags + wg % LP_GROUPS * LP_COPY;
    const unsigned *await1 = mine + lp_flag(2, share1.on.task(tid & 63)), *await2 = mine + lp_flag(1, share2.on.task(tid & 63));
    int slot = 0;
    bool lost = !sync.wait(); // a wait gave up
    for (; !lost && slot < T + L - 1; ++slot) {
        if (has1) {
            const int t = slot - tl;
            if (t >= 0 && t < T) {
                if (share1.waits && t + tpath > 0) lp_await(await1, slot, failed, &ok);
                f32x4_t acc[TN][RB];
                lp_zero(acc);
                lp_multiply<1, lp_depth(RB, TKG, TN, WR), 1>(acc, wt, (tncol + 7) / 8,
                                                             (tpath ? lp_xh(a, tl - 1, t + 1) : lp_xh(a, tl, t)) + tg0 * RB * 128, 0, tng);
                lp_exchange<1>(red, acc);
                if ((lost = !ok)) break;
                lp_put_T<TN, 8, RB>(a, red, lp_xt(a, tl, tpath, t), (tpath ? a.l[tl].Tx : a.l[tl].Th) + (i64)t * BT * gr, tcol, tncol);
            }
            lp_publish(flags, lp_flag(1, cols.task), slot + 1);
        }
        if (has2) {
            const int t = slot - zl;
            float gv[4] = {}, cv = 0.f, hv = 0.f;
            const bool active = t >= 0 && t < T;
            if (active) {
                if (share2.waits) lp_await(await2, slot + 1, failed, &ok);
                f32x4_t acc[NT][RB];
                lp_zero(acc);
                lp_multiply<2, lp_depth(RB, KG, NT, WR), 1>(acc, wz, NT, lp_xt(a, zl, zx, t) + zg0 * RB * 128, 0, zng);
                lp_exchange<2>(red, acc);
                if ((lost = !ok)) break;
                float z[4];
                const int rb = min(em >> 2, RB - 1);
                if constexpr (G4) {
                    const float *p = red + rb * 64 + lp_lane(em, eu);
#pragma unroll
                    for (int g = 0; g < 4; ++g) z[g] = p[g * RB * 64] + p[(g + 4) * RB * 64] + pb[g];
                } else {
                    f32x4_t s[LP_WAVES];
#pragma unroll
                    for (int v = 0; v < LP_WAVES; ++v)
                        s[v] = *(const f32x4_t *)(red + ((v * NT + (eu >> 2)) * RB + rb) * 64 + lp_lane(em, (eu & 3) * 4));
                    const f32x4_t sum = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
#pragma unroll
                    for (int g = 0; g < 4; ++g) z[g] = sum[g] + pb[g];
                }
                gv[0] = lp_sigmoid(z[0]), gv[1] = lp_sigmoid(z[1]), gv[2] = tanhf(z[2]), gv[3] = lp_sigmoid(z[3]);
                cv = gv[1] * c_prev + gv[0] * gv[2];
                hv = gv[3] * tanhf(cv);
                if (el) lp_share(lp_xh(a, zl, t + 1) + lp_place<RB>(un, em), un < h ? hv : 0.f);
                c_prev = cv;
            }
            lp_publish(flags, lp_flag(2, units.task), slot + 1); // the others need h only
            if (active && kept) {
                const LstmRunLayer &y = a.l[zl];
                const i64 idx = (i64)t * BT * h + (i64)em * h + un, base = ((i64)t * BT + em) * 4 * h + un;
                y.h_all[idx] = hv;
                y.c_all[idx] = cv;
#pragma unroll
                for (int g = 0; g < 4; ++g) y.gates[base + (i64)g * h] = gv[g];
            }
        }
    }
    if (lost) lp_void_fwd(a, cols, units, slot, tid);
}

// ------------------------------------------------------------------ backward
// Slot u handles the layers l with a step t = T - 1 - (u - (L - 1 - l)): first dh_t = (what arrives from outside) +
// dTh_{t+1} Vh^T + dTx of the layer above at t times its Vx^T, and the gate derivatives where dh is formed (a workgroup owns
// 16 NT units; below the top layer wavefronts 0-3 have the own path, 4-7 the one from above); then dTh = dz Uh and (above the
// first layer) dTx = dz Ux.  One slot more for the gradient that reaches the first layer's initial state.  dc_t stays with
// its thread.
template <int RB, int NT, int SL, bool G4>
__global__ __launch_bounds__(LP_NT) void lstm_run_bwd_kernel(LpArgs by_value)
{
    constexpr int TCB = G4 ? 1 : 2, TW = 4 << TCB, TN = G4 ? 3 : 1, TKG = G4 ? 6 : SL == 3 ? 8 : 12, KG = G4 ? 12 : 3;
    constexpr int NIT = (64 * NT * RB + LP_NT - 1) / LP_NT;
    constexpr int WR = TN * TKG * (2 << TCB) + NT * KG * 8;
    const LpArgs &a = lp_args(by_value);
    __shared__ __attribute__((aligned(16))) float red[LP_WAVES * (NT > TN ? NT : TN) * RB * 64];
    __shared__ int ok;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), wg = blockIdx.x;
    const int T = a.T, B = a.B, BT = a.BT, h = a.h, r = a.r, gr = a.gr, L = a.L, hp = a.hp, rp = a.rp, G = G4 ? 4 : 1;
    unsigned *flags = a.sync + LP_BAR, *failed = a.sync + LP_FAILED;
    if (tid == 0) ok = 1; // (waits that give up clear it)
    __syncthreads();
    // phase 1: units u0 .. of layer zl
    const LpUnits units = lp_units(a, wg, a.n1, 16 * NT);
    const bool has1 = units.has;
    const int zl = units.l, u0 = units.u0;
    const bool two = zl + 1 < L;
    const LpShare share1 = lp_bwd_share1(a, units, w, SL);
    const int zx = two ? w >> 2 : 0, zg0 = share1.first, zng = share1.n;
    float wz[NT][KG][8];
    {
        const float *V = zx ? a.l[zl + 1].Vx : a.l[zl].Vh;
        lp_weights_rows<NT, KG>(
            wz, zg0, zng,
            [&](int nt, int g, int c, bool &in) __attribute__((always_inline)) {
                const int unit = u0 + 16 * nt + c, q = G4 ? 32 * g / rp : 0;
                in = unit < h;
                return V + (i64)min(unit, h - 1) * gr + q * r + 32 * g - q * rp;
            },
            [&](int g) __attribute__((always_inline)) { return r - (G4 ? 32 * g % rp : 32 * g); });
    }
    // phase 2: columns tcol .. of a product (of gate tq, or slice tq of the contraction); groups tg0 .. of dz
    const LpColumns cols = lp_columns(a, wg, a.n2, rp, TW, G4 ? 4 : SL);
    const bool has2 = cols.has;
    const int tq = cols.q, tl = cols.l, tpath = cols.path, tcol = cols.col, tncol = cols.n;
    const LpShare share2 = lp_bwd_share2(a, cols, w, SL, 16 * NT);
    const int tg0 = share2.first, tng = share2.n;
    float wt[TN][TKG][2 << TCB];
    {
        const float *Um = tpath ? a.l[tl].Ux : a.l[tl].Uh;
        lp_weights<TN, TKG, TCB>(wt, tg0, tng, [&](int nt, int g, int i, int c) __attribute__((always_inline)) {
            const int cc = tcol + TW * nt + c, q = G4 ? tq : 32 * g / hp, unit = 32 * g - (G4 ? 0 : q * hp) + i;
            const float v = Um[((i64)min(q, 3) * h + min(unit, h - 1)) * r + min(cc, r - 1)];
            return q < 4 && unit < h && cc < r && TW * nt < tncol ? v : 0.f;
        });
    }
    float dcs[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) dcs[it] = 0.f;
    const unsigned *mine = flags + wg % LP_GROUPS * LP_COPY;
    const unsigned *await1 = mine + lp_flag(2, share1.on.task(tid & 63)), *await2 = mine + lp_flag(1, share2.on.task(tid & 63));
    int u = 0;
    bool lost = false; // a wait gave up
    for (; u < T + L; ++u) {
        if (has1) {
            const LstmRunLayer &y = a.l[zl];
            const int t = T - 1 - (u - (L - 1 - zl));
            const bool active = t >= -1 && t < T, own = t + 1 < T, above = t >= 0 && two;
            float pa[NIT], pg[NIT][4], pcp[NIT], pco[NIT];
            auto element = [&](int it, int &m, int &un) __attribute__((always_inline)) {
                const int e = tid + LP_NT * it, p = e >> 3;
                un = u0 + (p % (8 * NT)) * 2 + (e & 1);
                m = (p / (8 * NT)) * 4 + ((e >> 1) & 3);
            };
            if (active) { // (nothing of this depends on the phase before)
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    int m, un;
                    element(it, m, un);
                    const bool in = m < B && un < h && t >= 0;
                    const i64 idx = (i64)min(m, B - 1) * h + min(un, h - 1), at = (i64)max(t, 0) * BT * h + idx;
                    const i64 base = ((i64)max(t, 0) * BT + min(m, B - 1)) * 4 * h + min(un, h - 1);
                    pa[it] = (in && zl == L - 1 ? a.dh_top[at] : 0.f) + (in && t == T - 1 && y.dhT ? y.dhT[idx] : 0.f);
#pragma unroll
                    for (int g = 0; g < 4; ++g) pg[it][g] = in ? y.gates[base + (i64)g * h] : 0.f;
                    pcp[it] = in ? (t > 0 ? y.c_all + (i64)(t - 1) * BT * h : y.c0)[idx] : 0.f;
                    pco[it] = in ? y.c_all[at] : 0.f;
                    if (t == T - 1) dcs[it] = in && y.dcT ? y.dcT[idx] : 0.f;
                }
            }
            if (active) {
                f32x4_t acc[NT][RB];
                lp_zero(acc);
                if (share1.waits && (zx ? above : own)) {
                    lp_await(await1, u, failed, &ok);
                    lp_multiply<2, lp_depth(RB, KG, NT, WR, SL), SL>(acc, wz, NT, (zx ? lp_xt(a, zl + 1, 1, t) : lp_xt(a, zl, 0, t + 1)) + zg0 * RB * 128,
                                                                     rp * 4 * RB, zng);
                }
                lp_exchange<2>(red, acc);
                if ((lost = !ok)) break;
                float *xz = lp_xh(a, zl, max(t, 0));
                float dv[NIT][4], dcv[NIT];
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    int m, un;
                    element(it, m, un);
                    const float dh = pa[it] + lp_sum<NT, RB>(red, (un - u0) >> 4, min(m, 4 * RB - 1), (un - u0) & 15);
                    if (t < 0) {
                        if (m < B && un < h) y.dh0[(i64)m * h + un] = dh;
                        continue;
                    }
                    const float ig = pg[it][0], fg = pg[it][1], gg = pg[it][2], og = pg[it][3], tc = tanhf(pco[it]);
                    const float dc = dcs[it] + dh * og * (1.f - tc * tc);
                    dcs[it] = dcv[it] = dc * fg;
                    dv[it][0] = dc * gg * ig * (1.f - ig);
                    dv[it][1] = dc * pcp[it] * fg * (1.f - fg);
                    dv[it][2] = dc * ig * (1.f - gg * gg);
                    dv[it][3] = dh * tc * og * (1.f - og);
                    if (m < 4 * RB && un < hp) { // (zeros in the padding: its gates are)
#pragma unroll
                        for (int g = 0; g < 4; ++g) lp_share(xz + lp_place<RB>(g * hp + un, m), un < h ? dv[it][g] : 0.f);
                    }
                }
                lp_publish(flags, lp_flag(1, units.task), u + 1);
                if (t >= 0) {
#pragma unroll
                    for (int it = 0; it < NIT; ++it) {
                        int m, un;
                        element(it, m, un);
                        if (m < B && un < h) {
                            if (t == 0) y.dc0[(i64)m * h + un] = dcv[it];
#pragma unroll
                            for (int g = 0; g < 4; ++g) y.dz[((i64)t * BT + m) * 4 * h + (i64)g * h + un] = dv[it][g];
                        }
                    }
                }
            }
        }
        if (has2 && u + 1 < T + L) {
            const int t = T - 1 - (u - (L - 1 - tl));
            if (t >= 0 && t < T) {
                if (share2.waits) lp_await(await2, u + 1, failed, &ok);
                f32x4_t acc[TN][RB];
                lp_zero(acc);
                lp_multiply<TCB, lp_depth(RB, TKG, TN, WR), 1>(acc, wt, (tncol + TW - 1) / TW, lp_xh(a, tl, t) + ((G4 ? tq * (hp / 32) : 0) + tg0) * RB * 128,
                                                               0, tng);
                lp_exchange<TCB>(red, acc);
                if ((lost = !ok)) break;
                lp_put_T<TN, TW, RB>(a, red, lp_xt(a, tl, tpath, t) + (SL > 1 ? tq * rp * 4 * RB : 0),
                                     SL > 1 ? nullptr : (tpath ? a.l[tl].dTx : a.l[tl].dTh) + (i64)t * BT * gr, (G4 ? tq * rp : 0) + tcol, tncol);
                lp_publish(flags, lp_flag(2, cols.task), u + 1);
            }
        }
    }
    if (SL > 1) { // the slices' sums: all of dT is there
        LpSync sync = {a.sync, wg, &ok};
        if (!lost && wg < a.n2) sync.arrive(a.n2);
        if (!lost && wg < a.n1) lost = !sync.wait();
    }
    if (lost) {
        lp_void_bwd(a, cols, units, u, SL, RB, wg, tid);
        return;
    }
    if (SL > 1 && wg < a.n1) {
        const int nx = rp * 4 * RB;
        for (LpWalk at(nx, wg * LP_NT + tid, a.n1 * LP_NT); at.row < (2 * L - 1) * T; at.next()) {
            const int o = at.o, pr = at.row / T, t = at.row - pr * T, l = lp_layer(pr), path = lp_path(pr);
            int k, m;
            lp_element<RB>(o, k, m);
            if (k >= r || m >= B) continue;
            const float *x = lp_xt(a, l, path, t) + o;
            float v = x[0];
#pragma unroll
            for (int sl = 1; sl < SL; ++sl) v += x[sl * nx];
            (path ? a.l[l].dTx : a.l[l].dTh)[((i64)t * BT + m) * gr + k] = v;
        }
    }
}

// ------------------------------------------------------------------ host side
// compute units of the current device that a launch may use, 0 if it cannot run cooperative launches
static int lp_cus()
{
    const int n = cooperative_cus();
    return n < LP_MOST_CUS ? n : LP_MOST_CUS;
}

static bool lp_fits(const LstmGeom &g, bool bwd, size_t room)
{
    const size_t n = lp_floats(g, bwd);
    return n > 0 && n <= room && lp_rows_at_once(g, bwd, lp_cus()) > 0;
}

static int lp_launch(void (*kernel)(LpArgs), const LpArgs &a, bool bwd, hipStream_t s)
{
    TimingScope ts(bwd ? "lstm_run_bwd" : "lstm_run_fwd", s);
    LpArgs args = a;
    void *list[] = {(void *)&args};
    const hipError_t e = hipLaunchCooperativeKernel((const void *)kernel, dim3(a.nwg), dim3(LP_NT), list, 0, s);
    return e == hipSuccess ? PF_OK : set_hip_error(e);
}
typedef void (*LpKernel)(LpArgs);
template <int RB>
static LpKernel lp_kernel_rb(const LpPlan &p, int G, bool bwd)
{
    if constexpr (RB < 8) {
        if (G != 1) return bwd ? (LpKernel)lstm_run_bwd_kernel<RB, 1, 1, true> : lstm_run_fwd_kernel<RB, 1, true>;
        if (!bwd && p.NT == 3) return lstm_run_fwd_kernel<RB, 3, false>;
        if (bwd && p.NT == 2)
            return p.SL == 1 ? lstm_run_bwd_kernel<RB, 2, 1, false> : p.SL == 2 ? lstm_run_bwd_kernel<RB, 2, 2, false> : lstm_run_bwd_kernel<RB, 2, 3, false>;
    }
    if constexpr (RB <= 3) {
        if (!bwd && p.NT == 5) return lstm_run_fwd_kernel<RB, 5, false>;
    }
    if (bwd) return p.SL == 1 ? lstm_run_bwd_kernel<RB, 1, 1, false> : p.SL == 2 ? lstm_run_bwd_kernel<RB, 1, 2, false> : lstm_run_bwd_kernel<RB, 1, 3, false>;
    return p.NT == 1 ? lstm_run_fwd_kernel<RB, 1, false> : lstm_run_fwd_kernel<RB, 2, false>;
}
static LpKernel lp_kernel(const LpPlan &p, int G, bool bwd)
{
    switch (p.RB) {
    case 1: return lp_kernel_rb<1>(p, G, bwd);
    case 2: return lp_kernel_rb<2>(p, G, bwd);
    case 3: return lp_kernel_rb<3>(p, G, bwd);
    case 5: return lp_kernel_rb<5>(p, G, bwd);
    default: return lp_kernel_rb<8>(p, G, bwd);
    }
}

static int lp_run(const LstmGeom &g, const LstmRunLayer *l, const float *dh_top, bool bwd, float *ws, hipStream_t s)
{
    LstmGeom some = g;
    const int rows = lp_rows_at_once(g, bwd, lp_cus());
    for (int b0 = 0; b0 < g.B; b0 += rows) { // (one after the other: the workspace is theirs in turn)
        some.B = g.B - b0 < rows ? g.B - b0 : rows;
        const LpPlan p = lp_plan(some, bwd, lp_cus());
        LpArgs a;
        lp_fill(a, p, some, l, dh_top, ws, b0, g.B);
        int st = launch_zero_f32(s, (float *)a.sync, LP_SYNC);
        if (st == PF_OK) st = lp_launch(lp_kernel(p, g.G, bwd), a, bwd, s);
        if (st != PF_OK) return st;
    }
    return PF_OK;
}

namespace {
struct Install {
    Install() { lstm_recurrence = LstmRecurrence{lp_wants, lp_fits, lp_run}; }
} install;
} // namespace

} // namespace pf
