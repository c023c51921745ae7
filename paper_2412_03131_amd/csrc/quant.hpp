// quant.hpp -- the group quantizer of Sec. 2.2, bit-exact with the IEEE fp32
// definition, in two mappings: one 32-dim group over a 16-lane row, two values per
// lane (quant_pair: the generation step, one token per wave), and over a quad,
// eight values per lane (quant_oct: the append's page jobs, four tokens per wave
// at a time; the group's extremes and scale cost a quarter per value).
#pragma once

#include "common.hpp"

namespace dkv {

// Min / max over a 16-lane row with DPP (quad swaps, then half-row and row mirrors).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row16_min(float x)
{
    x = fminf(x, dpp_f32<0xB1>(x));   // quad_perm [1,0,3,2]
    x = fminf(x, dpp_f32<0x4E>(x));   // quad_perm [2,3,0,1]
    x = fminf(x, dpp_f32<0x141>(x));  // row_half_mirror
    return fminf(x, dpp_f32<0x140>(x));  // row_mirror
}
__device__ __forceinline__ float row16_max(float x)
{
    x = fmaxf(x, dpp_f32<0xB1>(x));
    x = fmaxf(x, dpp_f32<0x4E>(x));
    x = fmaxf(x, dpp_f32<0x141>(x));
    return fmaxf(x, dpp_f32<0x140>(x));
}

// clamp(rint(d / s), 0, lb) for two values, with d / s the IEEE fp32
// quotient.  The quotient through the hardware reciprocal (v_rcp_f32, within
// 1 ulp) and one rounded product is within 1.5 * 2^-23 relative, i.e. 2^-13
// absolute for |d/s| <= 2^9; larger quotients clamp the same way either way.
// It rounds to another integer than the IEEE quotient only if it lies within
// that distance of a half-integer, so lanes within 2^-12 of one (about 1 in
// 2^11) divide exactly, in a branch the compiler may not flatten.
__device__ __forceinline__ void codes_of(float d0, float d1, float s, float lb, uint32_t& c0, uint32_t& c1)
{
#pragma clang fp contract(off)
    const float rs = __builtin_amdgcn_rcpf(s);
    float q0 = d0 * rs, q1 = d1 * rs;
    const bool n0 = fabsf(q0 - rintf(q0)) > 0.5f - 0x1p-12f;
    const bool n1 = fabsf(q1 - rintf(q1)) > 0.5f - 0x1p-12f;
    if (n0 || n1) {
        asm volatile("" ::: "memory");
        if (n0) q0 = d0 / s;
        if (n1) q1 = d1 / s;
    }
    c0 = (uint32_t)fminf(fmaxf(rintf(q0), 0.0f), lb);
    c1 = (uint32_t)fminf(fmaxf(rintf(q1), 0.0f), lb);
}

// Quantize one 32-dim group spread over a 16-lane row (2 values per lane).
// Arithmetic is IEEE fp32 with no contraction, identical to the text of the
// quantizer: s = fp16((max-min)/L), z = fp16(min), code = clamp(rint((x-z)/s)).
__device__ __forceinline__ void quant_pair(uint32_t xbits, int lb, uint32_t& sz, uint32_t& c0,
                                           uint32_t& c1)
{
#pragma clang fp contract(off)
    float x0 = h2f(xbits & 0xffffu) + 0.0f;
    float x1 = h2f(xbits >> 16) + 0.0f;
    float mn = row16_min(fminf(x0, x1));
    float mx = row16_max(fmaxf(x0, x1));
    float s32 = (mx - mn) / (float)lb;
    uint32_t s16 = f2h_rne(s32);
    uint32_t z16 = f2h_rne(mn);
    float s = h2f(s16), z = h2f(z16);
    if (s16 == 0) {
        c0 = c1 = 0;
    } else {
        codes_of(x0 - z, x1 - z, s, (float)lb, c0, c1);
    }
    sz = s16 | (z16 << 16);
}

// RN(d / LB) for the code ranges LB = 1, 3, 15, 255 from RN(1 / LB): one Newton
// step on the rounded product, which gives the IEEE quotient for every 24-bit
// d (checked for all significands of each LB; d is 0 or at least 2^-24, so nothing
// underflows).  Infinities and NaN pass through as they do in a division.
template <int LB>
__device__ __forceinline__ float div_by_range(float d)
{
#pragma clang fp contract(off)
    if constexpr (LB == 1) return d;
    constexpr float y = 1.0f / (float)LB;
    const float q0 = d * y;
    const float q = __builtin_fmaf(__builtin_fmaf(-(float)LB, q0, d), y, q0);
    return d < INFINITY ? q : d;
}

typedef _Float16 q_half2 __attribute__((ext_vector_type(2)));

template <int CTRL>
__device__ __forceinline__ q_half2 dpp_h2(q_half2 x)
{
    return __builtin_bit_cast(q_half2, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}

// Quantize one 32-dim group spread over a quad of lanes, eight consecutive
// values each (four fp16 pairs), to codes 0 .. LB, as floats.  The arithmetic
// is quant_pair's: extremes (exact in fp16), s = fp16((max - min) / LB),
// z = fp16(min), code = clamp(rint((x - z) / s)) with the quotient through the
// hardware reciprocal and divided exactly within 2^-12 of a half-integer (the
// clamp comes first: its bounds are integers, so it commutes with the
// rounding, and x >= z).
template <int LB>
__device__ __forceinline__ void quant_oct(const uint4& x, uint32_t& sz, float (&code)[8])
{
#pragma clang fp contract(off)
    const q_half2 a = __builtin_bit_cast(q_half2, x.x), b = __builtin_bit_cast(q_half2, x.y);
    const q_half2 c = __builtin_bit_cast(q_half2, x.z), d = __builtin_bit_cast(q_half2, x.w);
    q_half2 lo = __builtin_elementwise_min(__builtin_elementwise_min(a, b), __builtin_elementwise_min(c, d));
    q_half2 hi = __builtin_elementwise_max(__builtin_elementwise_max(a, b), __builtin_elementwise_max(c, d));
    lo = __builtin_elementwise_min(lo, dpp_h2<0xB1>(lo));  // quad_perm [1,0,3,2]
    hi = __builtin_elementwise_max(hi, dpp_h2<0xB1>(hi));
    lo = __builtin_elementwise_min(lo, dpp_h2<0x4E>(lo));  // quad_perm [2,3,0,1]
    hi = __builtin_elementwise_max(hi, dpp_h2<0x4E>(hi));
    const float mn = fminf((float)lo.x, (float)lo.y) + 0.0f;  // -0 counts as +0
    const float mx = fmaxf((float)hi.x, (float)hi.y) + 0.0f;
    const uint32_t s16 = f2h_rne(div_by_range<LB>(mx - mn));
    const uint32_t z16 = f2h_rne(mn);
    const float s = h2f(s16), z = h2f(z16);
    const float rs = s16 == 0 ? 0.0f : __builtin_amdgcn_rcpf(s);  // scale 0: every code 0
    sz = s16 | (z16 << 16);
    const float v[8] = {(float)a.x, (float)a.y, (float)b.x, (float)b.y, (float)c.x, (float)c.y, (float)d.x, (float)d.y};
    float q[8], far = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        q[i] = __builtin_amdgcn_fmed3f((v[i] - z) * rs, 0.0f, (float)LB);
        code[i] = rintf(q[i]);
        far = fmaxf(far, fabsf(q[i] - code[i]));
    }
    if (far > 0.5f - 0x1p-12f) {
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (fabsf(q[i] - code[i]) > 0.5f - 0x1p-12f) {
                asm volatile("" ::: "memory");
                code[i] = fminf(rintf((v[i] - z) / s), (float)LB);
            }
        }
    }
}

}  // namespace dkv
