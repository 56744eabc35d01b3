// GELU of a Transformer layer's first feed-forward layer and its int8 codes, shared by the row quantiser and by the GEMM
// that writes the codes itself.
#pragma once
#include "common.hpp"

namespace egeria {

__device__ __forceinline__ float gelu_exact(float v)
{
    const double d = (double)v;
    return (float)(0.5 * d * (1.0 + erf(d * 0.70710678118654752440)));
}

constexpr float kGeluShortcutMin = 0.5f;   // gelu(0.5) = 0.346 exceeds max |gelu| over v < 0 (0.17)
// Beyond the shortcut the largest |gelu| may be that of a negative value.  |gelu| falls on both sides of the minimum of gelu at
// kGeluArgMin (within 2e-8; it is flat there: the neighbouring fp32 values round to the same gelu), so it is the largest
// one's, or that of the value nearest below the minimum, or of the nearest above it.
constexpr float kGeluArgMin = -0.75179154f;
// multiplier and scale of the codes of a tensor whose largest |gelu| is absmax
__device__ __forceinline__ float gelu_code_scale(float absmax, bool bad, float *scale)
{
    if (bad) absmax = 0.0f;
    float sc = (float)((double)absmax / 127.0);
    float inv = (float)(127.0 / (double)absmax);
    if (!(inv <= 3.402823466e+38f) || !(sc > 0.0f)) { sc = 1.0f; inv = 0.0f; }
    *scale = sc;
    return inv;
}

// fp32 GELU from a table of cubic pieces (gelu_table.inc: a piece of width 1/16 around every multiple of 1/16 in
// [-8, 8), generated with the measured error of the fp32 evaluation; from kGeluTop on gelu(v) rounds to v, below -8 it lies within
// 5e-15 of the table's first value).  |approximation - gelu| <= kGeluErrAbs + kGeluErrRel * |gelu|.
#include "gelu_table.inc"
constexpr float kGeluTop = 7.9375f;

// The table's value at v, times inv if the coefficients in LDS have been (scale_gelu_entry).  Adding 1.5 * 2^19 rounds v to the
// multiple of 1/16 that is its piece's centre and leaves the piece's number in the low byte.  BIG: values of kGeluTop and more
// may occur (the caller knows the tensor's maximum); otherwise the test is left out.
template <bool BIG>
__device__ __forceinline__ float gelu_table(float v, float inv, const float4 *__restrict__ tab)
{
    constexpr float kRound = 786432.0f;
    const float vc = BIG ? fminf(fmaxf(v, -8.0f), kGeluTop) : fmaxf(v, -8.0f);
    const float u = vc + kRound;
    const float t = vc - (u - kRound);
    const float4 c = *(const float4 *)((const uint8_t *)tab + (__float_as_uint(u) << 4 & 0xff0u));
    const float g = fmaf(fmaf(fmaf(c.w, t, c.z), t, c.y), t, c.x);
    return (BIG && v >= kGeluTop) ? v * inv : g;
}
__device__ __forceinline__ float4 scale_gelu_entry(float4 c, float inv) { return make_float4(c.x * inv, c.y * inv, c.z * inv, c.w * inv); }

__device__ __forceinline__ uint32_t code_of(float t)
{
    float r = rintf(t);
    r = fminf(fmaxf(r, -127.0f), 127.0f);
    return (uint32_t)((int)r) & 0xffu;
}

// Code of a value that a table leaves open, in fp64: 0 for -infinity and NaN, whose gelu is a NaN here, as the cubic table has it
// (it clamps v from below).  +infinity leaves inv = 0 and a NaN: code -127, and the tensor is flagged.
__device__ __forceinline__ uint32_t settle_gelu(float v, float inv)
{
    return v >= -3.402823466e+38f ? code_of(gelu_exact(v) * inv) : 0u;
}

// Code of gelu(v) from the table scaled by inv, in the low byte of the result.  The code clamp(rne(fp32(g * inv))) is monotone in
// g, so when both ends of the interval that the error bound leaves for g * inv round to the same integer, that integer is the
// code of the exact value; *unsure is set otherwise (a few values per 100 000) and the caller takes the fp64 form.
// room = 1/2 - kGeluErrAbs * inv.  (The relative part also covers the rounding of the scaled coefficients and of the product.)
// (The interval [t - e, t + e] rounds to one integer if |t - rne(t)| + e < 1/2.  No clamp: the scale is the
// tensor's exact maximum of |gelu| over 127, so |t| stays below 127.5 by the table's error bound; with a
// non-finite maximum inv is 0, and so is every code but that of +infinity, which is left unsure.)  25 vector instructions a value with the conversions spelt out (floor,
// int and back, rint), 18 this way.
template <bool BIG>
__device__ __forceinline__ uint32_t quant_gelu_fast(float v, float inv, float room, const float4 *__restrict__ tab, bool *unsure)
{
    constexpr float kRound = 12582912.0f;                        // 1.5 * 2^23
    const float t = gelu_table<BIG>(v, inv, tab);
    const float r = t + kRound;
    *unsure = !(fabsf(t - (r - kRound)) < fmaf(-(kGeluErrRel + 3.0e-7f), fabsf(t), room));
    return __float_as_uint(r);
}
// The same from straight lines (gelu_lines.inc), for the GEMM that writes the codes: half the bytes per look-up and 8 instructions
// less than the cubic pieces; about one value in 20 000 is left open.  lines: gelu_lines.inc scaled by inv, room = 1/2 -
// kGeluLineErr * inv.  Adding 1.5 * 2^15 + 6 rounds v to the multiple of 1/256 whose line is looked up and leaves its number in
// the low bits.  (Relative part: the scaled coefficients, the sum, and the exact form's two steps, each 2^-24 |t|.)  A value
// that is not finite makes t a NaN and stays unsure.
#include "gelu_lines.inc"
__device__ __forceinline__ uint32_t quant_gelu_lines(float v, float room, const float2 *__restrict__ lines, bool *unsure)
{
    constexpr float kRound = 12582912.0f, kLine = 49158.0f;      // 1.5 * 2^23, 1.5 * 2^15 + 6
    const float u = __builtin_amdgcn_fmed3f(v, -6.0f, 5.99609375f) + kLine;
    // the sum's bits: 0x47400000 + number; their lower 24 times 8, less what belongs to the constant, is the line's address
    uint32_t at;
    asm("v_mad_u32_u24 %0, %1, 8, %2" : "=v"(at) : "v"(u), "s"(0u - 0x400000u * 8u));
    const float2 c = *(const float2 *)((const uint8_t *)lines + at);
    const float t = fmaf(c.y, v, c.x);
    const float r = t + kRound;
    *unsure = !(fabsf(t - (r - kRound)) < fmaf(-4.0e-7f, fabsf(t), room));
    return __float_as_uint(r);
}

// the low bytes of four words
__device__ __forceinline__ uint32_t pack_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, 0x0c0c0400u), __builtin_amdgcn_perm(b, a, 0x0c0c0400u), 0x05040100u);
}

}  // namespace egeria
