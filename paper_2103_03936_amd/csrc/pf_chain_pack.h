// The chain kernel's packed weights, one 16-byte fragment slot at a time (device side, shared by the kernels that write them).
#pragma once

#include "pf_conv_chain.h"

namespace pf {

__device__ __forceinline__ void pack_w1_item(const PackW1 &p, int g)
{
    // one 16-byte fragment slot: ((s * RB + b) * 64 + lane)
    const int lane = g & 63, fb = g >> 6, b = fb % p.RB, s = fb / p.RB;
    const int rho = 32 * b + (lane & 31), tap = s % p.T;
    int c0 = 16 * (s / p.T) + 8 * (lane >> 5), cs = 1; // first channel of the slot and the step between its channels
    if (p.il_cw) { // k-step S of wavefront w = S / (cw / 16): channels 256 sub + 4 (16 t + 8 (lane / 32) + i) + w
        const int S = s / p.T, per = p.il_cw / 16, wv = S / per, rem = S - wv * per;
        c0 = 256 * (rem >> 2) + 4 * (16 * (rem & 3) + 8 * (lane >> 5)) + wv;
        cs = 4;
    }
    uint32_t e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = p.src[rho * p.s_rho + (c0 + cs * i) * p.s_c + tap * p.s_tap];
    if (p.cscale) {
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = float_to_bf16_bits(bf16_bits_to_float((uint16_t)e[i]) * p.cscale[c0 + cs * i]);
    }
    p.dst[g] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
}

__device__ __forceinline__ void pack_w2_item(const PackW2 &p, int g)
{
    // ((ob * S2 + s2) * 64 + lane)
    const int lane = g & 63, fb = g >> 6, s2 = fb % p.S2, ob = fb / p.S2;
    const int o = 32 * ob + (lane & 31), tap = s2 / p.R16, rho0 = 16 * (s2 % p.R16) + 8 * (lane >> 5);
    uint32_t e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = p.src[p.base + o * p.s_o + (rho0 + i) * p.s_rho + tap * p.s_tap];
    p.dst[g] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
}

} // namespace pf
