// Per-token INT8 codes of FP16 values (Section 6.1 of arXiv 2405.04532), as the activation quantizer and the GEMM kernel that
// quantizes its own tokens decide them.
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qoq {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ h2 half2_of(uint32_t w) { return __builtin_bit_cast(h2, w); }

// round_half_away(x / s), clamped to [-127, 127], for FP16 values x and s > 0 (held in FP32), without a division.
// x and s have 11-bit significands, so the exact quotient is either exactly on a rounding midpoint k + 1/2 or at
// least 2^-12 away from every midpoint (|x / s| < 256); x * fl(1 / s) is within 3e-5 of the quotient, and pushing
// it 1e-4 away from zero sends exact midpoints up and nothing else across: the result is the one the correctly
// rounded division followed by round-half-away gives, bit for bit (checked against exact rational arithmetic on
// the FP16 neighbours of all midpoints of several thousand scales, and on the GPU against the CPU reference).
__device__ __forceinline__ int quantize_code(float x, float inv_s)
{
    const float t = x * inv_s;
    const int a = (int)(t + copysignf(0.5f + 1e-4f, t));   // conversion truncates toward zero
    return max(-127, min(127, a));
}

// sx = fp16(absmax / 127): the FP32 quotient of an FP16 value by 127 never lies close enough to an FP16 rounding midpoint for
// the intermediate rounding to matter.  A row of zeros gets 1.
__device__ __forceinline__ __half scale_of_row(float amax)
{
    const __half s = __float2half_rn(amax / 127.0f);
    return __half2float(s) == 0.f ? __float2half_rn(1.0f) : s;
}

// The codes of eight FP16 values for a normal FP16 scale, two instructions each: x * (1/s) pushed away from zero by a relative
// 2^-20 and added to 1.5 * 2^23 in one fused multiply-add leaves round(x / s) in the low byte of the sum.  As in quantize_code
// the exact quotient is on a rounding midpoint or at least 2^-12 away from every one; the push (at most 1.4e-4 at 127, and at
// least 2^-20 - 2^-23 of the quotient, where the reciprocal and the factor are off by 2^-23 together) sends exact midpoints away
// from zero and nothing else across.  No clamp is needed: with a normal FP16 scale |x / s| <= 127 (1 + 2^-11).  Infinities
// (scale infinite, x * 0) and NaN leave a quiet NaN, whose low byte is the code 0 that the conversion of quantize_code gives.
// push = inv_s * (1 + 2^-20); isum += the codes.
__device__ __forceinline__ uint2 codes_of_chunk(const uint4& v, float push, int& isum)
{
    const float magic = 12582912.0f;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t r[8], packed[2];
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = __float_as_uint(fmaf((float)half2_of(w[j >> 1])[j & 1], push, magic));
#pragma unroll
    for (int j = 0; j < 2; ++j) {                      // the four low bytes of r[4j .. 4j + 3]
        packed[j] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(r[4 * j + 3], r[4 * j + 2], 0x0C0C0400u),
                                          __builtin_amdgcn_perm(r[4 * j + 1], r[4 * j], 0x0C0C0400u), 0x05040100u);
        isum = __builtin_amdgcn_sdot4((int)packed[j], 0x01010101, isum, false);
    }
    return make_uint2(packed[0], packed[1]);
}

// The same for a subnormal scale, which is too coarse for that.
__device__ __forceinline__ uint2 codes_of_chunk_clamped(const uint4& v, float inv_s, int& isum)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t packed[2] = {0u, 0u};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int a = quantize_code((float)half2_of(w[j >> 1])[j & 1], inv_s);
        isum += a;
        packed[j >> 2] |= (uint32_t)(a & 0xFF) << (8 * (j & 3));
    }
    return make_uint2(packed[0], packed[1]);
}

// Largest magnitude of eight FP16 values, as FP16 pairs joined with the ones before.
__device__ __forceinline__ h2 max_of_chunk(const uint4& v, h2 mx)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) mx = __builtin_elementwise_max(mx, half2_of(w[j] & 0x7FFF7FFFu));
    return mx;
}

}  // namespace
}  // namespace qoq
