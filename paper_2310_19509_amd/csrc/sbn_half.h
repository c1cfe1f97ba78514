// Device helpers of the kernels on pairs of 16-bit floats (sbn_conv1x1_half.hip, sbn_conv3x3_half.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sbn_half {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

constexpr int kFirstExp = 27;             // exponents run from here, so that a scale stays below 2^127
constexpr int kSpoilt = 255;              // exponent that an infinite activation leaves

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ v4u buf_load(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t scalar_off)
{
    return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)scalar_off, 0));
}
__device__ __forceinline__ float as_float(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_uint(float f) { return __builtin_bit_cast(uint32_t, f); }

// Factor that takes values of exponent e (the biased exponent of the largest) to [2^14, 2^15), times 2^more.
__device__ __forceinline__ float scale_of(int e, int more) { return as_float((uint32_t)(268 + more - e) << 23); }
// As bits - 1: pieces below 2^-27 of the largest activation (their largest value) lie under this; zeros do not.
__device__ __forceinline__ uint32_t tiny_limit(int e) { return ((uint32_t)(e - 26) << 23) - 1u; }

// max(|a|, |b|, c), one instruction; a NaN among them is passed over
__device__ __forceinline__ float max3_abs(float a, float b, float c)
{
    float d;
    asm("v_max3_f32 %0, |%1|, |%2|, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// Largest of 64 lanes' non-negative values, as bits (which order like the values), in a scalar register.
__device__ __forceinline__ uint32_t wave_max(float v)
{
    int m = (int)as_uint(v);
#define SBN_STEP(CTRL) m = max(m, __builtin_amdgcn_update_dpp(0, m, CTRL, 0xF, 0xF, true));
    SBN_STEP(0x111) SBN_STEP(0x112) SBN_STEP(0x114) SBN_STEP(0x118)      // row_shr 1, 2, 4, 8: lane 15 of every row
    SBN_STEP(0x142) SBN_STEP(0x143)                                      // row_bcast 15, 31: lane 63
#undef SBN_STEP
    return (uint32_t)__builtin_amdgcn_readlane(m, 63);
}

// Two values as pairs: hi of both, lo of both.  sc: the scale, sc11: 2048 times the scale.
__device__ __forceinline__ void split2(float a, float b, float sc, float sc11, uint32_t& hi, uint32_t& lo)
{
    const v2h h = __builtin_convertvector((v2f){a * sc, b * sc}, v2h);
    const v2f r = {__builtin_fmaf((float)h.x, -2048.0f, a * sc11), __builtin_fmaf((float)h.y, -2048.0f, b * sc11)};   // exact
    const v2h l = __builtin_convertvector(r, v2h);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

// Four values as pairs, written to LDS: hi at p, lo at p + half.
__device__ __forceinline__ void split4_to(char* p, int half, const v4f& v, float sc, float sc11)
{
    uint32_t h0, h1, l0, l1;
    split2(v.x, v.y, sc, sc11, h0, l0);
    split2(v.z, v.w, sc, sc11, h1, l1);
    *(v2u*)p = (v2u){h0, h1};
    *(v2u*)(p + half) = (v2u){l0, l1};
}

__device__ __forceinline__ v4f relu4(v4f v)                              // as in the 32-bit form
{
    typedef int v4i __attribute__((ext_vector_type(4)));
    const v4i b = __builtin_bit_cast(v4i, v);
    return __builtin_bit_cast(v4f, (v4i){b.x > 0 ? b.x : 0, b.y > 0 ? b.y : 0, b.z > 0 ? b.z : 0, b.w > 0 ? b.w : 0});
}

}  // namespace sbn_half
