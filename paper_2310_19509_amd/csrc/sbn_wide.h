// Device helpers of the kernels on triples of bfloat16 (sbn_conv1x1_wide.hip, sbn_conv3x3_wide.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sbn_wide {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef __bf16 v2b __attribute__((ext_vector_type(2)));

// Magnitudes are compared as twice their bits (the sign drops out) less one (zero comes out largest).
constexpr uint32_t kTiny = 2u * 0x0D800000u - 1u;                      // 2^-100

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ v4u buf_load(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t scalar_off)
{
    return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)scalar_off, 0));
}
__device__ __forceinline__ uint32_t as_uint(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ uint32_t magnitude(float f) { return (as_uint(f) << 1) - 1u; }
__device__ __forceinline__ uint32_t least_magnitude(const v4f& v, uint32_t least)
{
    return min(min(min(magnitude(v.x), magnitude(v.y)), least), min(magnitude(v.z), magnitude(v.w)));
}

// Two values as triples a + b + c, exact: a the nearest bfloat16, b the nearest one to the rest (16 bits and a
// sign, so that at most 8 bits are left for c).
__device__ __forceinline__ void split2(float v0, float v1, uint32_t& a, uint32_t& b, uint32_t& c)
{
    const v2b h = __builtin_convertvector((v2f){v0, v1}, v2b);
    const float r0 = v0 - (float)h.x, r1 = v1 - (float)h.y;
    const v2b m = __builtin_convertvector((v2f){r0, r1}, v2b);
    const v2b l = __builtin_convertvector((v2f){r0 - (float)m.x, r1 - (float)m.y}, v2b);
    a = __builtin_bit_cast(uint32_t, h);
    b = __builtin_bit_cast(uint32_t, m);
    c = __builtin_bit_cast(uint32_t, l);
}

// Four values as triples, written to LDS: a at p, b at p + part, c at p + 2 * part.
__device__ __forceinline__ void split4_to(char* p, int part, const v4f& v)
{
    uint32_t a0, a1, b0, b1, c0, c1;
    split2(v.x, v.y, a0, b0, c0);
    split2(v.z, v.w, a1, b1, c1);
    *(v2u*)p = (v2u){a0, a1};
    *(v2u*)(p + part) = (v2u){b0, b1};
    *(v2u*)(p + 2 * part) = (v2u){c0, c1};
}

// Lanes of one wave exchange data through LDS without a barrier (a wave's LDS instructions are executed in order): keeps the
// compiler from moving LDS accesses across this point, no instruction.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One instruction each, by the sign bit: for results that are finite.  The others are done again.
__device__ __forceinline__ v4f relu4(v4f v)
{
    typedef int v4i __attribute__((ext_vector_type(4)));
    const v4i b = __builtin_bit_cast(v4i, v);
    return __builtin_bit_cast(v4f, (v4i){b.x > 0 ? b.x : 0, b.y > 0 ? b.y : 0, b.z > 0 ? b.z : 0, b.w > 0 ? b.w : 0});
}

// For results that are done again: NaN becomes 0, as in the 32-bit forms.
__device__ __forceinline__ v4f relu4_of_any(v4f v) { return (v4f){fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f)}; }

// acc[co] += sum over ci of w[co][ci] * x[ci] (the 1x1 tables' order), for a piece that is kept
__device__ __forceinline__ void add_piece(v4f& acc, const v4f (&w)[4], const v4f& x, bool kept)
{
    if (!kept) return;                             // (not multiplied: the activation may be infinite or NaN)
#pragma unroll
    for (int ci = 0; ci < 4; ++ci)
#pragma unroll
        for (int co = 0; co < 4; ++co) acc[co] = __builtin_fmaf(w[co][ci], x[ci], acc[co]);
}
__device__ __forceinline__ v4f sum_over_wave(v4f v)
{
#pragma unroll
    for (int m = 1; m < 64; m *= 2)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] += __shfl_xor(v[i], m);
    return v;
}
// Outputs that a wave has to do again: bit k of a lane's `redo` says that its group of four outputs number k is one.
// A few of a number are done one by one by all lanes together (together(k, lane)), many by their lanes (alone(k)).
// (512 x 512, 12544 pixels, 42 us without any, 32-bit form 60 to 65: one NaN 374 us with lanes alone, 71 so; NaN in every 100th
// pixel 526 and 83; every output 970, bound by the loads of activations that lie a pixel apart.  3x3, 32 x 28 x 28, 128 x 128, 46 us,
// 32-bit form 56: one NaN, which reaches nine pixels, 148; every output 690.)
template <class Together, class Alone>
__device__ __forceinline__ void do_again(uint32_t redo, int n, Together&& together, Alone&& alone)
{
    __builtin_amdgcn_s_waitcnt(0);                 // the wave's stores so far are done: these replace some of them
#pragma unroll 1
    for (int k = 0; k < n; ++k) {
        unsigned long long mine = __builtin_amdgcn_ballot_w64(redo >> k & 1u);
        if (__builtin_popcountll(mine) > 12) {
            if (redo >> k & 1u) alone(k);
            continue;
        }
        for (; mine; mine &= mine - 1) together(k, __builtin_ctzll(mine));
    }
}

// The results of a 32-pixel tile, [group of 4 channels][channel] of 32 channels from ch0 on, to the rows row0 .. row0 + 31
// of y.  Two groups of 32 pixels (lanes 0-31 and 32-63 hold different channels of a pixel) become twice all four groups
// of 16 pixels, so that 64 bytes of a pixel leave in one instruction.  Channels from N on are not written, rows past the
// buffer neither.  AUX 2: streaming.
template <int AUX>
__device__ __forceinline__ void store_tile(const v16f& v, __amdgpu_buffer_rsrc_t yres, int row0, int ch0, int N, bool relu, int lane)
{
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        v4u o[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const auto r = __builtin_amdgcn_permlane16_swap(as_uint(v[8 * k + i]), as_uint(v[8 * k + 4 + i]), false, false);
            o[0][i] = r[0];
            o[1][i] = r[1];
        }
        const int ch = ch0 + 16 * k + ((lane >> 4) & 1) * 8 + (lane >> 5) * 4;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t off = ch < N ? ((uint32_t)((lane & 15) + 16 * u + row0) * (uint32_t)N + (uint32_t)ch) * 4u : 0xFFFFFFF0u;
            if (relu) o[u] = __builtin_bit_cast(v4u, relu4(__builtin_bit_cast(v4f, o[u])));
            __builtin_amdgcn_raw_buffer_store_b128(o[u], yres, (int)off, 0, AUX);
        }
    }
}

}  // namespace sbn_wide
