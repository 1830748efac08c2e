// Arithmetic of the activation producers, in one place for every kernel that runs them: the same
// operations in the same order give the same codes.
#pragma once
#include "flexq_device.h"

namespace {

// Over the 64 lanes, every lane with the result.  A butterfly, lane i with i ^ 32, 16, 8, 4, 2, 1 in
// turn (which fixes the order of the sum), by lane swaps and DPP instead of shuffles through LDS:
// after the step over 8 a row repeats every eight lanes, so that a rotation by four is i ^ 4.
// A reduction is a few tens of cycles instead of six trips through LDS one after the other; with
// one workgroup per token that is 0.3 us of a small launch's 4 to 5 (10240 x 8192 at 16 tokens behind
// an RMS norm 21.2 -> 20.9 us, LLaMA-2-7B's block at 8 tokens 57.2 -> 56.4).
template <class Op>
__device__ __forceinline__ unsigned wave_all(unsigned v, const Op &op)
{
    auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = op(s[0], s[1]);
    s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = op(s[0], s[1]);
#define FLEXQ_DPP(ctrl) (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, false)
    v = op(v, FLEXQ_DPP(0x128));      // row_ror:8
    v = op(v, FLEXQ_DPP(0x124));      // row_ror:4
    v = op(v, FLEXQ_DPP(0x4e));       // quad_perm [2, 3, 0, 1]
    v = op(v, FLEXQ_DPP(0xb1));       // quad_perm [1, 0, 3, 2]
#undef FLEXQ_DPP
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
    return __uint_as_float(wave_all(__float_as_uint(v), [](unsigned a, unsigned b) {
        return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
    }));
}
__device__ __forceinline__ float wave_sum(float v)
{
    return __uint_as_float(wave_all(__float_as_uint(v), [](unsigned a, unsigned b) {
        return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
    }));
}
__device__ __forceinline__ unsigned wave_max_bits(unsigned v)
{
    return wave_all(v, [](unsigned a, unsigned b) { return max(a, b); });
}

__device__ __forceinline__ unsigned pack_h2(float lo, float hi)
{
    return (unsigned)f2h(lo) | ((unsigned)f2h(hi) << 16);
}

// g / (1 + e^-g) through v_exp_f32 and v_rcp_f32: each is good to an ulp of
// fp32 and the product g * log2(e) to |g| * 2^-24 in the exponent, orders of
// magnitude inside the half ulp of the fp16 result.  e^-g overflowing to
// infinity gives g * 0 = -0, the correctly rounded value there.
__device__ __forceinline__ float silu(float g)
{
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.44269504088896341f));
}

// Eight h values of a chunk from its first operand (x, or the gate half) and its second (gamma, or
// the up half).  MODE as in producers.hip: 0 RMS norm, 1 gated SiLU, 2 identity.
template <int MODE>
__device__ __forceinline__ uint4 produce_h(const uint4 &a, const uint4 &b, float inv)
{
    if (MODE == 2) return a;
    unsigned a4[4] = {a.x, a.y, a.z, a.w}, b4[4] = {b.x, b.y, b.z, b.w}, o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float alo = h2f((uint16_t)(a4[i] & 0xffffu)), ahi = h2f((uint16_t)(a4[i] >> 16));
        const float blo = h2f((uint16_t)(b4[i] & 0xffffu)), bhi = h2f((uint16_t)(b4[i] >> 16));
        if (MODE == 0)
            o[i] = pack_h2((alo * inv) * blo, (ahi * inv) * bhi);
        else
            o[i] = pack_h2(silu(alo) * blo, silu(ahi) * bhi);
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
}

// The sum of squares of a chunk, added to ss.
__device__ __forceinline__ void add_squares(const uint4 &v, float &ss)
{
    unsigned w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = h2f((uint16_t)(w4[i] & 0xffffu)), b = h2f((uint16_t)(w4[i] >> 16));
        ss += a * a;
        ss += b * b;
    }
}

// The largest magnitude of a chunk (fp16 magnitudes of finite values order like their bits).
__device__ __forceinline__ unsigned max_bits(const uint4 &v, unsigned best)
{
    unsigned w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        best = max(best, w4[i] & 0x7fffu);
        best = max(best, (w4[i] >> 16) & 0x7fffu);
    }
    return best;
}

// fp16(absmax / qmax), 1 where that is zero.
__device__ __forceinline__ uint16_t token_scale(float amax, float qmax)
{
    const uint16_t bits = f2h(amax / qmax);
    return amax == 0.0f || h2f(bits) == 0.0f ? (uint16_t)0x3c00 : bits;
}

}  // namespace
