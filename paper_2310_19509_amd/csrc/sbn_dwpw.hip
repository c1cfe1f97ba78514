// Depthwise 3x3 (+ bias, ReLU) computed inside the staging of the group-sparse 1x1 layer that
// consumes it, for gfx950: the depthwise output never goes to HBM.  (Section 3.2 treats the
// depthwise and the pointwise layer of a separable block as separate operators; on this machine
// the early blocks of MobileNet-v1 are bound by HBM traffic, and the intermediate tensor is
// half of it.)
//
// A workgroup walks 8x8 tiles of output pixels (one per lane) x ALL output channels: four waves
// (64 channels) or eight (128), a wave per bundle, so that the depthwise result of a tile is
// computed once.  As many workgroups as the chip holds; their tiles and sub-chunks of 32 channels are one stream:
//   1. the depthwise layer's input tile with its halo, (7s+3)^2 pixels x 32 channels, goes
//      global -> registers -> LDS (the buffer's bounds give the zeros of the padding); the loads are issued
//      one step ahead, across tiles too;
//   2. every thread computes the depthwise outputs of one or two vertically adjacent pixels x 4
//      channels (weights and bias of the whole layer sit in LDS) and writes them to the activation tile
//      X[64 pixels][32 channels] that the 1x1 arithmetic reads.  For a layer with 3:9 pattern
//      groups of 16 channels (Section 3.2, DwConv3x3; Algorithm 2's per-group pattern information;
//      template parameter PAT) a wave works on ONE 16-channel half of the sub-chunk, which is one
//      pattern group: the group's kept taps are a wave-uniform word, and one scalar branch picks
//      the body that loads and multiplies only those six taps;
//   3. the wave walks the bundle's entries of the sub-chunk exactly as the 1x1 kernel does: a
//      16-byte LDS read per entry, 4 v_mfma_f32_4x4x1 per present group.
// With a stem in front (STEM) step 1 works out the 10x10 pixels of the stem's output under a tile instead: each wave 16 of the 32
// channels of 64 pixels, 108 multiplies, from inputs that its lanes loaded a tile ahead.
// Results are turned round between four lanes and leave as 64 bytes per pixel, without LDS or a barrier.
// MobileNet-v1's first three blocks at batch 64, 50 % (us, a workgroup per tile / so): 82 / 75, 81 / 60, 85 / 69.  The workgroup per tile spent half of
// its vector instructions on tile coordinates (integer divisions) and on padding, and three round trips on the parameters before its first
// load; vector and matrix instructions now take 41 to 45 us of the issue port, the traffic (309, 309 and 206 MB) 60, 60 and 40 us.
// The stem in front of the first: 36 + 74 us and 450 MB of tensors in two launches, 96 and 244 MB (301 counted) in one (3456 of 5500 matrix cycles per tile are the stem's: 28 of
// the 128 lanes that work out its 100 pixels idle, and 1.56 of them per pixel of the tile; instructions take 61 us of the issue port).
// Used when the 1x1 layer has at most 128 input and 128 output channels; wider layers are bound by
// the matrix pipe, not by memory traffic, and keep the two launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sbn_internal.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v3f __attribute__((ext_vector_type(3)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int TH = 8, TW = 8;          // output tile: 64 pixels, lane = oy * 8 + ox
constexpr int KC = 32;                 // channels per sub-chunk
constexpr int XS = KC + 4;             // row stride of the activation tile in floats (no bank conflicts)
constexpr int KMAX = 128;              // most input channels (depthwise parameters held in LDS)

template <int ABID>
__device__ __forceinline__ v4f mfma_bcast(float w, float x, v4f c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(w, x, c, 4, ABID, 0);
}

// group G of entry Q: lanes 4*AB..4*AB+3 of w hold [co 0..3], the components the four input channels
template <int Q, int G>
__device__ __forceinline__ void group_fma(const v4f& w, const v4f& xv, v4f (&acc)[4][2])
{
    constexpr int AB = (Q & 3) * 4 + G;
    acc[G][0] = mfma_bcast<AB>(w.x, xv.x, acc[G][0]);
    acc[G][1] = mfma_bcast<AB>(w.y, xv.y, acc[G][1]);
    acc[G][0] = mfma_bcast<AB>(w.z, xv.z, acc[G][0]);
    acc[G][1] = mfma_bcast<AB>(w.w, xv.w, acc[G][1]);
}

template <int Q>
__device__ __forceinline__ void entry_fma(uint32_t m, const v4f& w, const v4f& xv, v4f (&acc)[4][2])
{
    if (__builtin_expect((m & 1u) != 0, 1)) group_fma<Q, 0>(w, xv, acc);
    if (__builtin_expect((m & 2u) != 0, 1)) group_fma<Q, 1>(w, xv, acc);
    if (__builtin_expect((m & 4u) != 0, 1)) group_fma<Q, 2>(w, xv, acc);
    if (__builtin_expect((m & 8u) != 0, 1)) group_fma<Q, 3>(w, xv, acc);
}

// One instruction; NaN becomes 0.
__device__ __forceinline__ float relu(float v)
{
    float r;
    asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ v4f relu4(v4f v) { return (v4f){relu(v.x), relu(v.y), relu(v.z), relu(v.w)}; }

constexpr uint32_t kOutside = 0x80000000u;             // offset past the end of every buffer here

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

struct Record8 {
    uint32_t d[8];
};

// A stem in front (3 -> 32 channels, 3x3, stride 2): x is then its input, and every tile's 10 x 10 pixels of its output are worked out where
// the others are loaded.  w [9][3][32], b [32]; h, w_in: extents of its input.
struct StemArgs {
    const float* w;
    const float* b;
    int h, w_in, act;
};

// Pair P = (input k, group g of 4 channels) of 16 channels: its weights lie in block P % 16 of register P / 16
template <int P>
__device__ __forceinline__ void stem_pairs(const float (&wreg)[7], const float (&xin)[27], v4f (&acc)[4])
{
    if constexpr (P < 27 * 4) {
        acc[P % 4] = mfma_bcast<P % 16>(wreg[P / 16], xin[P / 4], acc[P % 4]);
        stem_pairs<P + 1>(wreg, xin, acc);
    }
}

// Four lanes' v[0 .. 3] turned round among them: lane q of a quad then holds in v[k] what lane k held in v[q].
__device__ __forceinline__ void turn_quad(v4f (&v)[4], int lane)
{
    auto step = [&](auto ctrl_c, int bit, v4f& lo, v4f& hi) {          // lo stays where the bit is clear, hi where it is set
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a = lo[i], b = hi[i];
            const float a_of = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, a), decltype(ctrl_c)::value, 0xF, 0xF, true));
            const float b_of = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, b), decltype(ctrl_c)::value, 0xF, 0xF, true));
            lo[i] = lane & bit ? b_of : a;
            hi[i] = lane & bit ? b : a_of;
        }
    };
    constexpr std::integral_constant<int, 0xB1> by1{};                 // quad_perm [1, 0, 3, 2]
    constexpr std::integral_constant<int, 0x4E> by2{};                 // quad_perm [2, 3, 0, 1]
    step(by1, 1, v[0], v[1]);
    step(by1, 1, v[2], v[3]);
    step(by2, 2, v[0], v[2]);
    step(by2, 2, v[1], v[3]);
}

// Waves per SIMD that the registers leave room for, and with that the workgroups of a compute unit.  (One more wave per SIMD, 96 registers: the forms of
// four waves and of stride 2 spill, 73 -> 173 and 63 -> 79 us; the other 68 either way; with the stem 96 -> 120.)
// Stride 2 with four waves comes with two and, LEAN, with three: launch_dwpw.
constexpr int waves_per_simd(int stride, int nwv, bool stem, bool lean, bool exact)
{
    return exact ? 2 : stem || lean ? 3 : stride == 2 && nwv == 4 ? 2 : 4;
}

// EXACT: with a stem, where the launch has so few tiles that the 1x1 layer by itself would run in the few-pixel form: no 32-bit sum runs over more than 4
// products (four sets of accumulators), and they and the bias are added in 64 bits, so that the error is that form's (0.98 to 1.01 of it; with one set and the
// bias added in 32 bits 1.02 to 1.10).  60 sizes of up to 64 tiles 9.4 to 10.6 us in three launches, 6.0 to 6.5 with one set, 6.5 to 7.0 so.
template <int STRIDE, int NWV, bool PAT, bool STEM, bool LEAN, bool EXACT>
__global__ __launch_bounds__(64 * NWV, waves_per_simd(STRIDE, NWV, STEM, LEAN, EXACT)) void dwpw_kernel(const float* __restrict__ x, float* __restrict__ y,
                                                   const float* __restrict__ dw_w, const float* __restrict__ dw_b,
                                                   const uint32_t* __restrict__ dw_taps, int dw_act,
                                                   const uint32_t* __restrict__ records,
                                                   const uint32_t* __restrict__ woff, const float* __restrict__ wts,
                                                   const float* __restrict__ bias, int H, int W, int OH, int OW, int K,
                                                   int N, int n_bundles, int n_sub, int tiles_x,
                                                   int tiles_y, int n_pix_tiles, int step, int step_x, int step_y, int step_n, int act,
                                                   StemArgs stem)
{
    static_assert(!STEM || (STRIDE == 1 && NWV == 4), "the stem joins the form of four waves and stride 1");
    static_assert(!LEAN || (STRIDE == 2 && NWV == 4), "the other forms have one number of waves");
    static_assert(!EXACT || STEM, "one sub-chunk only");
    constexpr int NSET = EXACT ? 4 : 1;
    constexpr int IW = (TW - 1) * STRIDE + 3, IH = (TH - 1) * STRIDE + 3;     // input tile
    constexpr int NPIX = IW * IH;
    constexpr int NPIXP = NPIX + (6 - NPIX % 4) % 4;           // = 2 mod 4: the two halves of a pixel pair fill all banks
    constexpr int NSLOT = NPIX * (KC / 4);
    constexpr int NT = 64 * NWV;                               // threads
    constexpr int NL = (NSLOT + NT - 1) / NT;
    constexpr int AS = STEM ? KC + 4 : KC;                     // row stride of the input tile (STEM: a lane writes a pixel)
    constexpr int NO = 8 / NWV;                                // depthwise output pixels per thread
    __shared__ __attribute__((aligned(16))) float lds_a[PAT ? 2 * NPIXP * 16 : (NPIX + 1) * AS];   // input tile [pixel][32], PAT: [16-channel half][pixel][16]
    __shared__ __attribute__((aligned(16))) float lds_x[64 * XS];                     // depthwise result
    __shared__ __attribute__((aligned(16))) float lds_p[10 * KMAX];                   // depthwise weights [9][K], bias [K]

    const int lane = threadIdx.x & 63;
    const int bundle = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = bundle;
    const bool active = bundle < n_bundles;
    const int bsafe = active ? bundle : 0;

    // ---- the workgroup's tiles: every step-th, in steps of the coordinates
    struct At {
        int x, y, n;
    };
    auto next = [&](At t) -> At {
        t.x += step_x;
        t.y += step_y;
        t.n += step_n;
        if (t.x >= tiles_x) {
            t.x -= tiles_x;
            ++t.y;
        }
        if (t.y >= tiles_y) {
            t.y -= tiles_y;
            ++t.n;
        }
        return t;
    };
    int tile = blockIdx.x;
    At at = {tile % tiles_x, tile / tiles_x % tiles_y, tile / (tiles_x * tiles_y)};

    // ---- input tile staging: thread t moves 16-byte slots t, t+NT, ...; slot = pixel * 8 + column.  Slots outside the image
    //      lie outside the buffer and read as zeros.
    const int col4 = (threadIdx.x & 7) * 4;
    auto slot_pixel = [](int i, int tid) {
        const int pix = i * (NT / 8) + (tid >> 3);
        return pix < NPIX ? pix : NPIX - 1;
    };
    // STEM: a wave works out 16 channels of 64 of the tile's 100 pixels, a lane per pixel: its 3 x 3 x 3 inputs are loaded where
    // the others load the tile, pixel by pixel (those outside the input lie outside the buffer).
    const int spix = (bundle & 1) * 64 + lane, shalf = bundle >> 1;
    const int spy = min(spix, NPIX - 1) / IW, spx = min(spix, NPIX - 1) % IW;
    __amdgpu_buffer_rsrc_t xres;
    constexpr int NPLACE = STEM || LEAN ? 1 : NL, NOFF = STEM ? 9 : NL;
    uint32_t place[NPLACE], off[NOFF];                       // of the slots: from the tile's corner, from the buffer's start
    if constexpr (STEM) {
        place[0] = (uint32_t)(spy * 2 * stem.w_in + spx * 2) * 12u;
    } else if constexpr (!LEAN) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int pix = slot_pixel(i, threadIdx.x);
            place[i] = (uint32_t)(((pix / IW) * W + pix % IW) * K + col4) * 4u;
        }
    }
    auto aim = [&](const At& t) {
        if constexpr (STEM) {
            const int iy0 = t.y * (2 * TH) - 3, ix0 = t.x * (2 * TW) - 3, r0 = max(iy0, 0);
            xres = make_rsrc(x + ((long long)t.n * stem.h + r0) * stem.w_in * 3, (uint32_t)(min(stem.h - r0, 2 * IH + 1) * stem.w_in) * 12u);
            const uint32_t first = place[0] + (uint32_t)((iy0 - r0) * stem.w_in + ix0) * 12u;
            const bool border = iy0 < 0 || ix0 < 0 || iy0 + 2 * IH + 1 > stem.h || ix0 + 2 * IW + 1 > stem.w_in;
#pragma unroll
            for (int k = 0; k < 9; ++k) off[k] = first + (uint32_t)(k / 3 * stem.w_in + k % 3) * 12u;
            if (border) {
                const int iy = iy0 + 2 * spy, ix = ix0 + 2 * spx;
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    if ((uint32_t)(iy + k / 3) >= (uint32_t)stem.h || (uint32_t)(ix + k % 3) >= (uint32_t)stem.w_in) off[k] = kOutside;
            }
            return;
        }
        const int iy0 = t.y * (TH * STRIDE) - 1, ix0 = t.x * (TW * STRIDE) - 1, r0 = max(iy0, 0);
        xres = make_rsrc(x + ((long long)t.n * H + r0) * W * K, (uint32_t)(min(H - r0, IH) * W * K) * 4u);
        const uint32_t corner = (uint32_t)(((iy0 - r0) * W + ix0) * K) * 4u;
        const bool border = iy0 < 0 || ix0 < 0 || iy0 + IH > H || ix0 + IW > W;
        if constexpr (!LEAN) {
#pragma unroll
            for (int i = 0; i < NL; ++i) off[i] = place[STEM ? 0 : i] + corner;
        }
        if (LEAN || border) {
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));                    // (worked out here: kept across the tiles the slots' pixels cost registers)
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const int pix = slot_pixel(i, tid);
                const int iy = iy0 + pix / IW, ix = ix0 + pix % IW;
                if constexpr (LEAN) off[i] = (uint32_t)((pix / IW * W + pix % IW) * K + col4) * 4u + corner;
                if ((uint32_t)iy >= (uint32_t)H || (uint32_t)ix >= (uint32_t)W) off[i] = kOutside;
            }
        }
    };
    float xin[STEM ? 27 : 1], swreg[STEM ? 7 : 1];
    if constexpr (STEM) {
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int e = min(i * 64 + lane, 27 * 16 - 1);    // [input][16 channels]
            swreg[i] = stem.w[(e >> 4) * 32 + shalf * 16 + (e & 15)];
        }
    }
    v4f stage_reg[NL];
    auto issue_a = [&](int sc) {                             // K is a multiple of 32: always inside
        if constexpr (STEM) {
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const v3f v = __builtin_bit_cast(v3f, __builtin_amdgcn_raw_buffer_load_b96(xres, (int)off[k], 0, 0));
                xin[k * 3] = v.x;
                xin[k * 3 + 1] = v.y;
                xin[k * 3 + 2] = v.z;
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < NL; ++i)
            stage_reg[i] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(xres, (int)off[i], sc * (KC * 4), 0));
    };
    auto write_a = [&](const At& t) {                        // (slots past the tile go to a pixel behind it: no branch)
        if constexpr (STEM) {
            v4f o[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) o[g] = *(const v4f*)(stem.b + shalf * 16 + g * 4);
            stem_pairs<0>(swreg, xin, o);
            const int sy = t.y * TH - 1 + spy, sx = t.x * TW - 1 + spx, pix = min(spix, NPIX);
            const bool real = (uint32_t)sy < (uint32_t)H && (uint32_t)sx < (uint32_t)W;      // (outside: the depthwise layer's padding)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
#pragma unroll
                for (int i = 0; i < 4; ++i) o[g][i] = real ? o[g][i] : 0.f;
                if (stem.act == SBN_ACT_RELU) o[g] = relu4(o[g]);
                *(v4f*)(PAT ? lds_a + (shalf * NPIXP + pix) * 16 + g * 4 : lds_a + pix * AS + shalf * 16 + g * 4) = o[g];
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int pix = min(i * (NT / 8) + (int)(threadIdx.x >> 3), NPIX);
            *(v4f*)(PAT ? lds_a + ((col4 >> 4) * NPIXP + pix) * 16 + (col4 & 15) : lds_a + pix * AS + col4) = stage_reg[i];
        }
    };

    // ---- depthwise: thread t -> channels col4..col4+3 of the sub-chunk, output pixels (oyp .. oyp +
    //      NO - 1, oxp) of the tile; the (NO - 1) * STRIDE + 3 input rows under them are read once
    const int oxp = (threadIdx.x >> 3) & 7, oyp = (threadIdx.x >> 6) * NO;
    auto dw_dense = [&](int sc) {
        const int ch = sc * KC + col4;
        const float* wp = lds_p + ch;
        const v4f b = *(const v4f*)(lds_p + 9 * KMAX + ch);
        v4f o[NO];
#pragma unroll
        for (int jo = 0; jo < NO; ++jo) o[jo] = b;
        const float* a0 = lds_a + ((oyp * STRIDE) * IW + oxp * STRIDE) * AS + col4;
#pragma unroll
        for (int r = 0; r < (NO - 1) * STRIDE + 3; ++r) {
            v4f a[3];
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) a[kx] = *(const v4f*)(a0 + (r * IW + kx) * AS);
#pragma unroll
            for (int jo = 0; jo < NO; ++jo) {
                const int ky = r - jo * STRIDE;
                if (ky >= 0 && ky < 3) {
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) o[jo] += *(const v4f*)(wp + (ky * 3 + kx) * KMAX) * a[kx];
                }
            }
        }
#pragma unroll
        for (int jo = 0; jo < NO; ++jo) {
            v4f v = o[jo];
            if (dw_act == SBN_ACT_RELU) v = relu4(v);
            *(v4f*)(lds_x + ((oyp + jo) * TW + oxp) * XS + col4) = v;
        }
    };

    // ---- depthwise with pattern groups: a wave takes one 16-channel half of the sub-chunk (one group) and
    //      2 * NO rows of the tile; lane -> channel quad, column, row pair.  Output pixels (oyp ..
    //      oyp + NO - 1, oxp); the (NO - 1) * STRIDE + 3 input rows under them are read once.
    const int half = wave & 1, quad4 = (lane & 3) * 4;
    const int oxq = (lane >> 2) & 7, oyq = (wave >> 1) * (2 * NO) + (lane >> 5) * NO;
    const float* aq = lds_a + (half * NPIXP + (oyq * STRIDE) * IW + oxq * STRIDE) * 16 + quad4;
    float* xo = lds_x + (oyq * TW + oxq) * XS + half * 16 + quad4;
    // TAPS: bit ky * 3 + kx set = the tap is kept by every channel of the group (removed taps hold
    // zeros in dw_w, so a body that multiplies more taps than needed is still right)
    auto dw_body = [&](int sc, auto taps_c) {
        constexpr uint32_t TAPS = decltype(taps_c)::value;
        const int ch = sc * KC + half * 16 + quad4;
        const float* wp = lds_p + ch;                          // weights are read where they are used: few live registers
        const v4f b = *(const v4f*)(lds_p + 9 * KMAX + ch);
        v4f o[NO];
#pragma unroll
        for (int jo = 0; jo < NO; ++jo) o[jo] = b;
#pragma unroll
        for (int r = 0; r < (NO - 1) * STRIDE + 3; ++r) {
            v4f a[3];
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                bool needed = false;
#pragma unroll
                for (int jo = 0; jo < NO; ++jo) {
                    const int ky = r - jo * STRIDE;
                    if (ky >= 0 && ky < 3 && ((TAPS >> (ky * 3 + kx)) & 1u)) needed = true;
                }
                if (needed) a[kx] = *(const v4f*)(aq + (r * IW + kx) * 16);
            }
#pragma unroll
            for (int jo = 0; jo < NO; ++jo) {
                const int ky = r - jo * STRIDE;
                if (ky >= 0 && ky < 3) {
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx)
                        if ((TAPS >> (ky * 3 + kx)) & 1u) o[jo] += *(const v4f*)(wp + (ky * 3 + kx) * KMAX) * a[kx];
                }
            }
        }
#pragma unroll
        for (int jo = 0; jo < NO; ++jo) {
            v4f v = o[jo];
            if (dw_act == SBN_ACT_RELU) v = relu4(v);
            *(v4f*)(xo + jo * TW * XS) = v;
        }
    };
    // the 3:9 family: row r keeps columns {0, 1} (mask 3) or {1, 2} (mask 6)
#define SBN_TAPS(R0, R1, R2) std::integral_constant<uint32_t, (R0) | ((R1) << 3) | ((R2) << 6)>()
    auto dw_pattern = [&](int sc) {
        const uint32_t taps = dw_taps ? __builtin_amdgcn_readfirstlane(dw_taps[sc * (KC / 16) + half]) : 0x1FFu;
        switch (taps) {
        case 6 | (6 << 3) | (6 << 6): dw_body(sc, SBN_TAPS(6, 6, 6)); break;
        case 3 | (6 << 3) | (6 << 6): dw_body(sc, SBN_TAPS(3, 6, 6)); break;
        case 6 | (3 << 3) | (6 << 6): dw_body(sc, SBN_TAPS(6, 3, 6)); break;
        case 3 | (3 << 3) | (6 << 6): dw_body(sc, SBN_TAPS(3, 3, 6)); break;
        case 6 | (6 << 3) | (3 << 6): dw_body(sc, SBN_TAPS(6, 6, 3)); break;
        case 3 | (6 << 3) | (3 << 6): dw_body(sc, SBN_TAPS(3, 6, 3)); break;
        case 6 | (3 << 3) | (3 << 6): dw_body(sc, SBN_TAPS(6, 3, 3)); break;
        case 3 | (3 << 3) | (3 << 6): dw_body(sc, SBN_TAPS(3, 3, 3)); break;
        default: dw_body(sc, SBN_TAPS(7, 7, 7)); break;
        }
    };
#undef SBN_TAPS

    auto dw_compute = [&](int sc) {
        if constexpr (PAT)
            dw_pattern(sc);
        else
            dw_dense(sc);
    };

    // ---- the 1x1 layer's tables: one record of 8 descriptors and one first-entry index per sub-chunk;
    //      a 16-byte weight load per lane covers four entries
    const uint32_t* wo = woff + (size_t)bsafe * (n_sub + 1);
    const Record8* recs = (const Record8*)__builtin_assume_aligned(records, 32) + (size_t)bsafe * n_sub;
    auto load_weights = [&](int sc, v4f (&w)[2]) {
        const uint32_t e0 = __builtin_amdgcn_readfirstlane(wo[sc]);
        const v4f* src = (const v4f*)(wts + (size_t)e0 * 64) + lane;
        w[0] = src[0];
        w[1] = src[64];
    };
    auto multiply = [&](const Record8& r, const v4f (&w)[2], v4f (&acc)[NSET][4][2]) {
        const char* xl = (const char*)lds_x + lane * (XS * 4);
        v4f xa, xb;
#define SBN_ENTRY(Q, XC, XN)                                             \
    if (__builtin_expect(r.d[Q] == 0, 0)) goto sub_chunk_done;           \
    if (Q + 1 < 8) XN = *(const v4f*)(xl + (r.d[(Q + 1) & 7] >> 8));      \
    entry_fma<Q>(r.d[Q], w[Q / 4], XC, acc[Q / 2 % NSET]);
        xa = *(const v4f*)(xl + (r.d[0] >> 8));
        SBN_ENTRY(0, xa, xb)
        SBN_ENTRY(1, xb, xa)
        SBN_ENTRY(2, xa, xb)
        SBN_ENTRY(3, xb, xa)
        SBN_ENTRY(4, xa, xb)
        SBN_ENTRY(5, xb, xa)
        SBN_ENTRY(6, xa, xb)
        SBN_ENTRY(7, xb, xa)
#undef SBN_ENTRY
    sub_chunk_done:;
    };

    // ---- bias, activation, rows of 64 bytes.  Pixels past the image and channels past c_out lie outside the buffer and are dropped.
    const uint32_t yplace = bundle * 16 + (lane & 3) * 4 < N
                                ? (uint32_t)(((lane >> 3) * OW + (lane & 4)) * N + bundle * 16 + (lane & 3) * 4) * 4u
                                : kOutside;
    auto finish = [&](const At& t, v4f (&acc)[NSET][4][2]) {
        v4f o[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const v4f b = *(const v4f*)(bias + bundle * 16 + g * 4);
            if constexpr (EXACT) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    double sum = (double)b[i];
#pragma unroll
                    for (int h = 0; h < 2 * NSET; ++h) sum += (double)acc[h / 2][g][h % 2][i];
                    o[g][i] = (float)sum;
                }
            } else {
                o[g] = acc[0][g][0] + acc[0][g][1] + b;
            }
        }
        turn_quad(o, lane);
        if (act == SBN_ACT_RELU) {                     // (behind the turn: the compiler does not see an asm's write in front of a lane move's read)
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = relu4(o[k]);
        }
        const int oy0 = t.y * TH, ox0 = t.x * TW;
        const __amdgpu_buffer_rsrc_t yres = make_rsrc(y + ((long long)t.n * OH + oy0) * OW * N, (uint32_t)(min(OH - oy0, TH) * OW * N) * 4u);
        // (The place within the row goes into the lane's offset: behind a store with a scalar offset the compiler writes
        // the data's registers again in the next instruction, and the store has then been seen to take the new value.)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t to = ox0 + (lane & 4) + k < OW ? yplace + (uint32_t)((ox0 + k) * N * 4) : kOutside;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o[k]), yres, (int)to, 0, 0);
        }
    };

    aim(at);
    issue_a(0);
    // the depthwise layer's parameters, asked for together behind the first input tile
    {
        constexpr int NP = (10 * KMAX / 4 + NT - 1) / NT;
        v4f v[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int s = i * NT + threadIdx.x, row = s / (KMAX / 4), ch = s % (KMAX / 4) * 4;
            v[i] = *(const v4f*)(row < 9 ? dw_w + row * K + min(ch, K - 4) : dw_b + min(ch, K - 4));
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int s = i * NT + threadIdx.x;
            if (s < 10 * KMAX / 4) *(v4f*)(lds_p + s * 4) = v[i];
        }
    }
    v4f acc[NSET][4][2];
    // (in one place and out of the compiler's sight: it otherwise keeps several sets of them, over 200 registers)
    auto pin = [&] {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int h = 0; h < 2 * NSET; ++h) {
                if constexpr (STEM || LEAN) asm volatile("" : "+v"(acc[h / 2][g][h % 2]));
                else asm volatile("" : "+a"(acc[h / 2][g][h % 2]));
            }
    };
    auto start = [&] {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int h = 0; h < 2 * NSET; ++h) acc[h / 2][g][h % 2] = (v4f){0.f, 0.f, 0.f, 0.f};
        pin();
    };
    // A workgroup barrier for LDS alone: memory accesses stay in flight across it.
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    start();
    int sc = 0;
    v4f w[2];
    load_weights(0, w);
    write_a(at);
    for (;;) {
        barrier();                               // input tile visible (and the parameters); X free
        const Record8 r = recs[sc];
        const bool last = sc + 1 == n_sub;
        const int scn = last ? 0 : sc + 1;
        const int tile_next = last ? tile + step : tile;
        const bool again = tile_next < n_pix_tiles;
        const At at_next = last && again ? next(at) : at;
        if (last && again) aim(at_next);
        issue_a(scn);                                  // in flight while this sub-chunk is worked on (behind the last tile unused)
        dw_compute(sc);
        barrier();                               // X visible, input tile free
        if (active) multiply(r, w, acc);
        pin();
        load_weights(scn, w);
        write_a(at_next);                              // (in front of the stores: loads and stores come back in order)
        if (last) {
            if (active) finish(at, acc);
            start();
        }
        if (!again) break;
        tile = tile_next;
        at = at_next;
        sc = scn;
    }
}

template <int STRIDE, int NWV, bool PAT, bool STEM = false, bool LEAN = false, bool EXACT = false>
int launch(const sbn_packed* p, const float* x, float* y, const float* dw_w, const float* dw_b, const uint32_t* dw_taps,
           int dw_act, int n, int h, int w, hipStream_t st, const StemArgs& stem = {})
{
    const sbn::DeviceLayout& L = p->dev;
    const int oh = (h - 1) / STRIDE + 1, ow = (w - 1) / STRIDE + 1;
    const int tiles_x = (ow + TW - 1) / TW, tiles_y = (oh + TH - 1) / TH;
    const long long n_pix_tiles = (long long)n * tiles_x * tiles_y;
    const long long grid = std::min<long long>(n_pix_tiles, 4ll * waves_per_simd(STRIDE, NWV, STEM, LEAN, EXACT) / NWV * L.cus);
    hipLaunchKernelGGL((dwpw_kernel<STRIDE, NWV, PAT, STEM, LEAN, EXACT>), dim3((unsigned)grid), dim3(64 * NWV), 0, st, x, y, dw_w, dw_b, dw_taps, dw_act, L.d_records32,
                       L.d_woff32, L.d_wts, L.d_bias, h, w, oh, ow, p->c_in, p->c_out, L.n_bundles, L.n_chunks32,
                       tiles_x, tiles_y, (int)n_pix_tiles, (int)grid, (int)(grid % tiles_x), (int)(grid / tiles_x % tiles_y),
                       (int)(grid / tiles_x / tiles_y), p->act, stem);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sbn::fail(SBN_EHIP, "fused depthwise + 1x1 launch: %s", hipGetErrorString(e));
    return SBN_OK;
}

}  // namespace

namespace sbn {

bool dwpw_fusable(const sbn_packed* p, int channels, int stride)
{
    return p->kind == SBN_CONV1X1 && p->c_in == channels && channels % KC == 0 && channels <= KMAX && p->c_out <= 128 &&
           (stride == 1 || stride == 2);
}

int launch_dwpw(const sbn_packed* p, const float* x, float* y, const float* dw_w, const float* dw_b,
                const uint32_t* dw_taps, int dw_stride, int dw_act, int n, int h, int w, void* stream)
{
    if (!dwpw_fusable(p, p->c_in, dw_stride) || !dwpw_extents_fit(p, dw_stride, n, h, w))
        return fail(SBN_EINVAL, "internal error: fused depthwise + 1x1 launch for a layer it does not cover");
    hipStream_t st = (hipStream_t)stream;
    const bool wide = p->dev.n_bundles > 4;      // more than 64 output channels: eight waves cover up to 128
#define SBN_DWPW(S, NWV, PAT) launch<S, NWV, PAT>(p, x, y, dw_w, dw_b, dw_taps, dw_act, n, h, w, st)
#define SBN_DWPW_LEAN(PAT) launch<2, 4, PAT, false, true>(p, x, y, dw_w, dw_b, dw_taps, dw_act, n, h, w, st)
    // Four waves, stride 2: three workgroups per compute unit (LEAN: a tile's places in memory are worked out anew at every tile, which spares the
    // registers) or two.  us, two / three: 576 tiles, 32 x 64 10.6 / 9.2, 560, 64 x 60 14.4 / 12.4, 540, 128 x 24 20.8 / 17.1, 11820, 32 x 32 94 / 76;
    // two where a unit gets more than four tiles of several sub-chunks: 12168, 64 x 60 162 / 174, 11880, 128 x 52 274 / 280 (4500 random sizes,
    // two / three, least and median: up to 4 tiles per unit 0.94, 1.06; up to 8 0.89, 1.03; more than 16 0.88, 0.98, with 32 channels 0.89, 1.03).
    const long long tiles = (long long)n * (((h - 1) / dw_stride + TH) / TH) * (((w - 1) / dw_stride + TW) / TW);
    const bool lean = p->c_in == KC || tiles <= 4ll * p->dev.cus;
    // Pattern bodies everywhere but in the eight-wave stride-2 form: there they need 134 registers,
    // one workgroup per CU instead of two (with a workgroup per tile 109 us against 79 us for MobileNet-v1's second block at
    // batch 64), so that form multiplies the stored zeros of the removed taps instead.
    if (dw_taps && !(wide && dw_stride == 2)) {
        if (wide) return SBN_DWPW(1, 8, true);
        if (dw_stride == 2) return lean ? SBN_DWPW_LEAN(true) : SBN_DWPW(2, 4, true);
        return SBN_DWPW(1, 4, true);
    }
    if (wide) return dw_stride == 2 ? SBN_DWPW(2, 8, false) : SBN_DWPW(1, 8, false);
    if (dw_stride == 2) return lean ? SBN_DWPW_LEAN(false) : SBN_DWPW(2, 4, false);
    return SBN_DWPW(1, 4, false);
#undef SBN_DWPW_LEAN
#undef SBN_DWPW
}

bool stem_dwpw_fusable(const sbn_packed* p, int c_in, int c_out, int stride, int dw_stride)
{
    return c_in == 3 && c_out == 32 && stride == 2 && dw_stride == 1 && dwpw_fusable(p, 32, 1) && p->dev.n_bundles <= 4;
}

int launch_stem_dwpw(const sbn_packed* p, const float* x, float* y, const float* stem_w, const float* stem_b, int stem_act, const float* dw_w,
                     const float* dw_b, const uint32_t* dw_taps, int dw_act, int n, int h, int w, bool exact, void* stream)
{
    const int sh = (h - 1) / 2 + 1, sw = (w - 1) / 2 + 1;      // (21 rows of 2 sw pixels, 12 bytes each, are less than 17 of sw with 32 channels)
    if (!stem_dwpw_fusable(p, 3, 32, 2, 1) || !dwpw_extents_fit(p, 1, n, sh, sw))
        return fail(SBN_EINVAL, "internal error: fused stem + depthwise + 1x1 launch for a layer it does not cover");
    const StemArgs stem = {stem_w, stem_b, h, w, stem_act};
    hipStream_t st = (hipStream_t)stream;
#define SBN_STEM(PAT, EXACT) launch<1, 4, PAT, true, false, EXACT>(p, x, y, dw_w, dw_b, dw_taps, dw_act, n, sh, sw, st, stem)
    if (exact) return dw_taps ? SBN_STEM(true, true) : SBN_STEM(false, true);
    return dw_taps ? SBN_STEM(true, false) : SBN_STEM(false, false);
#undef SBN_STEM
}

}  // namespace sbn
