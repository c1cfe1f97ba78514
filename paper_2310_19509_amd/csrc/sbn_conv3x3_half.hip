// Kernel-level group-sparse 3x3 convolution, stride 1, on pairs of 16-bit floats, for gfx950.
//
// The arithmetic is that of sbn_conv1x1_half.hip (operands s * (hi + lo / 2048), three
// v_mfma_f32_16x16x32_f16 per product, sums in 32-bit floats, 32-bit multiply-adds for data outside the
// pairs' range): one multiply per 32 channels and tap, over blocks filled up with the removed kernels' zeros.
//
// Mapping.  Output pixels are numbered through the images (image, row, column); a workgroup owns
// T = 64 * WPX consecutive ones x 64 output channels, so no lane multiplies padding whatever the extents.  With
// stride 1 the tap (ky, kx) of pixel p is pixel p + (ky - 1) * W + kx - 1 of the same numbering, so the
// tile's input is one run of T + 2 * W + 2 pixels.  Per 32 channels it goes global -> registers -> pairs ->
// LDS, once for all nine taps; a lane whose tap lies outside the image reads a row of zeros instead (nine
// bits per pixel, worked out once).  The scale of the pairs is shared by the workgroup: it is known after
// a barrier that the single LDS buffer needs anyway.
//
// Three forms (70 % sparsity, batch 32, the 32-bit form's time first):
//   WPX = 2, NB = 2: 128 x 64 tiles, a wave 64 pixels x 32 channels.  56 x 56 x 64: 38 -> 33 us, 28 x 28 x 128:
//     40 -> 27 us, 14 x 14 x 256: 43 -> 30 us.
//   WPX = 1, NB = 1: 64 x 64 tiles, a wave 64 pixels x 16 channels, for launches of fewer tiles than 0.7 per
//     compute unit of the first form (3 x 23 x 23 x 128 at 50 %: 17.6 -> 13.0 us, 128 x 64 tiles 18.0).
//   the same with S = 2 slices of waves that share the input channels, up to one workgroup per compute unit
//     (7 x 7 x 512: 51 -> 36 us, one slice 45; 3 x 9 x 9 x 256 at 50 %: 32 -> 18 us, one slice 21).
// The large form runs at 0.8 PFLOP/s of 16-bit multiplies; the small ones wait: fetching weights a whole
// sub-chunk, activations two sub-chunks or LDS reads two halves ahead changed none of their times.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sbn_half.h"
#include "sbn_internal.h"

namespace {

using namespace sbn_half;

constexpr int KC = 32;                    // channels staged at a time
constexpr int PT = 4;                     // 16-pixel tiles per wave (two halves)

// Outputs [pix0, pix0 + npix) x [ch0, ch0 + nch) by 32-bit multiply-adds over the kept kernels.  One
// wave; reached only for data outside the pairs' range.
__device__ __forceinline__ void exact_outputs(const float* __restrict__ x, float* __restrict__ y,
                                              const uint32_t* __restrict__ records, const uint32_t* __restrict__ woff,
                                              const float* __restrict__ wts, const float* __restrict__ bias, int H, int W,
                                              int K, int N, int n_sub, long long pix0, int npix, int ch0, int nch, int act)
{
    for (int o = threadIdx.x & 63; o < npix * nch; o += 64) {
        const long long pix = pix0 + o / nch;
        const int ch = ch0 + o % nch, b = ch >> 4, g = (ch >> 2) & 3, co = ch & 3;
        const int ox = (int)(pix % W), oy = (int)(pix / W % H);
        float acc = bias[ch];
        for (int c = 0; c < n_sub; ++c) {
            const uint32_t* r = records + ((size_t)b * n_sub + c) * 8;
            const float* w = wts + (size_t)woff[(size_t)b * (n_sub + 1) + c] * 576 + g * 16 + co;
#pragma unroll 1
            for (int q = 0; q < 8 && r[q] != 0; ++q, w += 576) {
                if (!(r[q] >> g & 1u)) continue;
#pragma unroll 1
                for (int t = 0; t < 9; ++t) {
                    const int dy = t / 3 - 1, dx = t % 3 - 1;
                    if (oy + dy < 0 || oy + dy >= H || ox + dx < 0 || ox + dx >= W) continue;
                    const float* xp = x + (pix + (long long)dy * W + dx) * K + c * KC + (int)(r[q] >> 12) * 4;
                    for (int ci = 0; ci < 4; ++ci) acc = __builtin_fmaf(w[t * 64 + ci * 4], xp[ci], acc);
                }
            }
        }
        y[pix * N + ch] = act == SBN_ACT_RELU && __builtin_bit_cast(int, acc) <= 0 ? 0.f : acc;
    }
}

// NL: staged 16-byte slots per lane; NL * 32 >= T + 2 * W + 2 pixels.
// S: slices of four waves; slice s multiplies the sub-chunks s, s + S, ... out of its own image, with its own
// exponent, and the sums meet at the end.
template <int NB, int WPX, int NL, int S>
__global__ __launch_bounds__(256 * S, 2) void conv3x3_half_kernel(
    const float* __restrict__ x, float* __restrict__ y, const uint16_t* __restrict__ wh, const int* __restrict__ wh_exp,
    const float* __restrict__ bias, const uint32_t* __restrict__ records, const uint32_t* __restrict__ woff,
    const float* __restrict__ wts, int M, int H, int W, int K, int N, int n_bundles, int n_sub, int n_col_tiles, int n_pix_tiles,
    int act)
{
    constexpr int T = 64 * WPX;
    constexpr int ROWS = NL * 32, PLANE = (ROWS + 16) * 16, HALF = 4 * PLANE;      // row ROWS of every plane is zero
    static_assert(NB * 4 == 4 * WPX, "a workgroup owns 64 channels");
    // LDS image, hi and lo alike: per 8 channels a plane of one 16-byte row per pixel (all planes begin at
    // the same bank, so a read of 16 neighbouring pixels from each of four planes is free of conflicts)
    static_assert(S == 1 || (2 * HALF >= 4 * PT * NB * 1024), "the slices' sums fit one image");
    __shared__ __attribute__((aligned(16))) char lds_all[S][2 * HALF];
    __shared__ uint32_t wave_top_all[S][4];
    __shared__ int wave_tiny_all[S][4], slice_exp[S];

    const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;                // column tiles of one pixel tile on one XCD
    const int pix_tile = (jj / n_col_tiles) * 8 + xcd, col_tile = jj % n_col_tiles;
    if (pix_tile >= n_pix_tiles) return;
    const int tid = threadIdx.x & 255, lane = tid & 63;                  // thread of the slice
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slice = S == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    char* const lds = lds_all[slice];
    uint32_t* const wave_top = wave_top_all[slice];
    int* const wave_tiny = wave_tiny_all[slice];
    const int wpx = wave % WPX;
    const int bundle = col_tile * 4 + (wave / WPX) * NB;                 // first of NB
    const bool active = bundle < n_bundles;
    const int p0 = pix_tile * T, q0 = p0 - W - 1;                        // first output pixel, first staged one
    const int rows_valid = M - p0 < T ? M - p0 : T;

    // ---- this lane's pixels: LDS offset of the top left tap, and which taps lie inside the image
    int at[PT];
    uint32_t inside[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t) {
        const int l = wpx * 64 + t * 16 + (lane & 15), p = p0 + l;
        const int ox = p % W, oy = p / W % H;
        uint32_t m = 0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int iy = oy + k / 3 - 1, ix = ox + k % 3 - 1;
            if (iy >= 0 && iy < H && ix >= 0 && ix < W) m |= 1u << k;
        }
        inside[t] = p < M ? m : 0u;
        at[t] = (lane >> 4) * PLANE + l * 16;
    }
    const int zero_at = (lane >> 4) * PLANE + ROWS * 16;
    if (tid < 8 * 16) *(uint32_t*)(lds + (tid >> 4) * PLANE + ROWS * 16 + (tid & 15) * 4) = 0u;

    // ---- activations: slot i = staged pixel i * 32 + tid / 8, channels 4 * (tid % 8).  Pixels before the
    // first and past the last one, and channels past c_in, lie outside the buffer and read as zero.
    const int quad = tid & 7;
    const int staged = M - q0 < T + 2 * W + 2 ? M - q0 : T + 2 * W + 2;
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(x + (long long)q0 * K, (uint32_t)staged * (uint32_t)K * 4u);
    auto slot_off = [&](int i) {
        const int r = i * 32 + (tid >> 3);
        return q0 + r >= 0 ? ((uint32_t)r * (uint32_t)K + (uint32_t)quad * 4u) * 4u : 0x80000000u;
    };
    v4f stage[NL];
    auto issue_x = [&](int c) {
        const uint32_t outside = c * KC + quad * 4 < K ? 0u : 0x80000000u;
#pragma unroll
        for (int i = 0; i < NL; ++i) stage[i] = __builtin_bit_cast(v4f, buf_load(xres, slot_off(i) | outside, (uint32_t)c * (KC * 4)));
    };
    int run = kFirstExp;                           // running exponent of the workgroup's activations
    uint32_t least = 0xFFFFFFFFu;                  // smallest non-zero piece of four channels (its largest), as bits - 1
    char* const wr = lds + (quad >> 1) * PLANE + (tid >> 3) * 16 + (quad & 1) * 8;

    // ---- weights
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(wh, 0xFFFFFFFFu);      // (the packer keeps the table below 4 GiB)
    auto load_w = [&](int step, v8h (&w)[NB][2]) {                       // step = 9 * sub-chunk + tap
        step = step < n_sub * 9 ? step : 0;                              // (past the end: multiplied with zeros)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int b = bundle + j < n_bundles ? bundle + j : n_bundles - 1;
#pragma unroll
            for (int s = 0; s < 2; ++s)
                w[j][s] = __builtin_bit_cast(v8h, buf_load(wres, (uint32_t)lane * 16u + s * 1024u,
                                                           ((uint32_t)b * (uint32_t)(n_sub * 9) + (uint32_t)step) * 2048u));
        }
    };

    // The matrix unit cuts what it adds to a sum at the sum's own last place, so a long chain of multiplies
    // loses more than its roundings (relative error 4.5e-8 after one step, 7.7e-8 after 4, 2.0e-7 after
    // 32); `main` therefore runs over one row of taps only and is then added to `total`.
    v4f total[PT][NB], main[PT][NB], cross[PT][NB];
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j) total[t][j] = main[t][j] = cross[t][j] = (v4f){0.f, 0.f, 0.f, 0.f};

    // Half a tap: the 16-pixel tiles t and t + 1.  Their reads are issued one half ahead.
    struct Frag {
        v8h hi[2], lo[2];
    };
    auto read_half = [&](int k, int tap_off, int t, Frag& f) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int in = (int)(inside[t + u] << (31 - k)) >> 31;       // all ones if the tap is inside
            const char* p = lds + (((at[t + u] + tap_off) & in) | (zero_at & ~in));
            f.hi[u] = *(const v8h*)p;
            f.lo[u] = *(const v8h*)(p + HALF);
        }
    };
    auto fma_half = [&](int t, const Frag& f, const v8h (&w)[NB][2]) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) cross[t + u][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[j][0], f.lo[u], cross[t + u][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) main[t + u][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[j][0], f.hi[u], main[t + u][j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) cross[t + u][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[j][1], f.hi[u], cross[t + u][j], 0, 0, 0);
    };

    // (Weights a tap ahead, activations a sub-chunk ahead.  With one bundle per wave, weights a whole sub-chunk or
    // activations two ahead changed nothing.)
    v8h w[2][NB][2];
    int tiny = 0;
    issue_x(slice);
    load_w(slice * 9, w[0]);
    // (every slice goes through the same number of barriers; past the last sub-chunk it stages zeros)
    for (int c = slice; c - slice < n_sub; c += S) {
        // measure this wave's share of the sub-chunk
        float top = 0.f;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const float m = max3_abs(stage[i].z, stage[i].w, max3_abs(stage[i].x, stage[i].y, 0.f));
            least = min(least, as_uint(m) - 1u);
            top = fmaxf(top, m);
        }
        const uint32_t wtop = wave_max(top);
        if (lane == 0) wave_top[wave] = wtop;
        __syncthreads();                           // everyone has measured, and has finished with the last sub-chunk's image
        const uint32_t all = max(max(wave_top[0], wave_top[1]), max(wave_top[2], wave_top[3]));
        const int e = (int)((uint32_t)__builtin_amdgcn_readfirstlane((int)all) >> 23);
        if (__builtin_expect(e > run, 0)) {
#pragma unroll
            for (int t = 0; t < PT; ++t)
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        total[t][j][i] = __builtin_amdgcn_ldexpf(total[t][j][i], run - e);
                        cross[t][j][i] = __builtin_amdgcn_ldexpf(cross[t][j][i], run - e);
                    }
            run = e;
        }
        const float sc = scale_of(run, 0), sc11 = scale_of(run, 11);
#pragma unroll
        for (int i = 0; i < NL; ++i) split4_to(wr + i * 512, HALF, stage[i], sc, sc11);
        tiny = __builtin_amdgcn_ballot_w64(least < tiny_limit(run)) != 0;
        if (lane == 0) wave_tiny[wave] = tiny;
        __syncthreads();
        // (opaque: the 36 addresses of a sub-chunk's reads are cheaper to work out again than to keep in registers)
#pragma unroll
        for (int t = 0; t < PT; ++t) asm volatile("" : "+v"(at[t]), "+v"(inside[t]));
        auto tap_off = [&](int k) { return (k / 3 * W + k % 3) * 16; };  // (ky * W + kx) rows of 16 bytes
        Frag f[2];
        read_half(0, 0, 0, f[0]);
#pragma unroll
        for (int i = 0; i < 18; ++i) {
            const int k = i / 2, ahead = i + 1;
            if (i % 2 == 0) {
                load_w(k < 8 ? c * 9 + k + 1 : (c + S) * 9, w[(k + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                if (k == 1) issue_x(c + S);
            }
            if (ahead < 18) read_half(ahead / 2, tap_off(ahead / 2), ahead % 2 * 2, f[ahead & 1]);
            __builtin_amdgcn_sched_barrier(0);
            fma_half(i % 2 * 2, f[i & 1], w[k & 1]);
            __builtin_amdgcn_sched_barrier(0);
            if (i % 6 == 5) {
#pragma unroll
                for (int t = 0; t < PT; ++t)
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        total[t][j] += main[t][j];
                        main[t][j] = (v4f){0.f, 0.f, 0.f, 0.f};
                    }
            }
        }
#pragma unroll
        for (int j = 0; j < NB; ++j)               // nine taps: the next sub-chunk's first weights are in the odd set
#pragma unroll
            for (int s = 0; s < 2; ++s) w[0][j][s] = w[1][j][s];
    }

    // ---- total + cross / 2048 of all slices, in units of the largest exponent
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) total[t][j][i] = __builtin_fmaf(cross[t][j][i], 1.0f / 2048.0f, total[t][j][i]);
    if constexpr (S > 1) {
        if (tid == 0) slice_exp[slice] = run;
        __syncthreads();                           // exponents are known, images are dead
        int e = run;
#pragma unroll
        for (int s = 0; s < S; ++s) e = max(e, __builtin_amdgcn_readfirstlane(slice_exp[s]));
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i) total[t][j][i] = __builtin_amdgcn_ldexpf(total[t][j][i], run - e);
                if (slice > 0) *(v4f*)(lds + ((wave * PT + t) * NB + j) * 1024 + lane * 16) = total[t][j];
            }
        run = e;
        __syncthreads();
        if (slice > 0) return;
#pragma unroll
        for (int s = 1; s < S; ++s)
#pragma unroll
            for (int t = 0; t < PT; ++t)
#pragma unroll
                for (int j = 0; j < NB; ++j) total[t][j] += *(const v4f*)(lds_all[s] + ((wave * PT + t) * NB + j) * 1024 + lane * 16);
    }
    if (!active) return;

    // ---- back to the data's scale, bias, activation, store
    const __amdgpu_buffer_rsrc_t yres = make_rsrc(y + (long long)p0 * N, (uint32_t)rows_valid * (uint32_t)N * 4u);
    const int ch_lane = (lane >> 4) * 4;
    int spoilt = run == kSpoilt;
    tiny = 0;
    for (int s = 0; s < S; ++s) tiny |= wave_tiny_all[s][0] | wave_tiny_all[s][1] | wave_tiny_all[s][2] | wave_tiny_all[s][3];
    const float least_sum = tiny ? (float)K * (9.0f * 16.0f) : 0.0f;     // sums below this may be mostly error: 9 K terms, each off by 2^-20
    float odd = 0.f;                               // NaN once a result is not finite
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int b = bundle + j < n_bundles ? bundle + j : n_bundles - 1;
        const v4f bj = *(const v4f*)(bias + b * 16 + ch_lane);
        const int4 ej = *(const int4*)(wh_exp + b * 16 + ch_lane);
        const int e4[4] = {ej.x, ej.y, ej.z, ej.w};
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            v4f o = total[t][j];
            if (max3_abs(o.z, o.w, max3_abs(o.x, o.y, 0.f)) < least_sum) spoilt = 1;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_ldexpf(o[i], e4[i] + run - 141) + bj[i];
            odd = __builtin_fmaf((o.x + o.y) + (o.z + o.w), 0.f, odd);
            total[t][j] = o;
        }
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(spoilt || odd != odd) != 0, 0)) {
        const int first = wpx * 64;
        const int npix = rows_valid - first < 64 ? rows_valid - first : 64;
        const int nch = N - bundle * 16 < NB * 16 ? N - bundle * 16 : NB * 16;
        if (npix > 0)
            exact_outputs(x, y, records, woff, wts, bias, H, W, K, N, n_sub, (long long)p0 + first, npix, bundle * 16, nch, act);
        return;
    }
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int ch = (bundle + j) * 16 + ch_lane;
            const int row = wpx * 64 + t * 16 + (lane & 15);
            const uint32_t off = ch < N ? ((uint32_t)row * (uint32_t)N + (uint32_t)ch) * 4u : 0xFFFFFFF0u;
            v4f o = total[t][j];
            if (act == SBN_ACT_RELU) o = relu4(o);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o), yres, (int)off, 0, 0);
        }
}

template <int NB, int WPX, int NL, int S>
int launch(const sbn_packed* p, const float* x, float* y, int n, int h, int w, hipStream_t st)
{
    const sbn::DeviceLayout& L = p->dev;
    const long long M = (long long)n * h * w;
    constexpr int T = 64 * WPX;
    const long long n_pix_tiles = (M + T - 1) / T;
    const int n_col_tiles = (L.n_bundles + 3) / 4;
    const long long grid = ((n_pix_tiles + 7) / 8) * 8 * n_col_tiles;
    if (T + 2 * w + 2 > NL * 32) return sbn::fail(SBN_EINVAL, "internal error: the tile's rows do not fit the staged image");
    if (grid > 0x7FFFFFFFll) return sbn::fail(SBN_EINVAL, "too many output tiles for one launch (%lld)", n_pix_tiles);
    hipLaunchKernelGGL((conv3x3_half_kernel<NB, WPX, NL, S>), dim3((unsigned)grid), dim3(256 * S), 0, st, x, y, L.d_wh, L.d_wh_exp,
                       L.d_bias, L.d_records32, L.d_woff32, L.d_wts, (int)M, h, w, p->c_in, p->c_out, L.n_bundles, L.n_chunks32,
                       n_col_tiles, (int)n_pix_tiles, p->act);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sbn::fail(SBN_EHIP, "conv3x3 launch: %s", hipGetErrorString(e));
    return SBN_OK;
}

// the smallest staged image that holds a tile and its halo
template <int NB, int WPX, int S>
int launch_fit(const sbn_packed* p, const float* x, float* y, int n, int h, int w, hipStream_t st)
{
    const int rows = 64 * WPX + 2 * w + 2;
    if (rows <= 160) return launch<NB, WPX, 5, S>(p, x, y, n, h, w, st);
    if (rows <= 256) return launch<NB, WPX, 8, S>(p, x, y, n, h, w, st);
    return launch<NB, WPX, 12, S>(p, x, y, n, h, w, st);
}

}  // namespace

namespace sbn {

// Width: the largest tile's rows, 128 + 2 * w + 2, fit 384 staged ones.  Images of fewer than four rows or
// columns reach few of the taps, so that their sums are short and the 32-bit form loses less
// (an image of one pixel: 3.6e-8 against 5.9e-8).
bool conv3x3_half_takes(const sbn_packed* p, int n, int h, int w)
{
    return p->dev.d_wh && p->stride == 1 && w <= 127 && w >= 4 && h >= 4 && (long long)n * h * w <= 0x70000000ll;
}

int launch_conv3x3_half(const sbn_packed* p, const float* x, float* y, int n, int h, int w, int form, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (!form) {
        const long long M = (long long)n * h * w, cols = (p->dev.n_bundles + 3) / 4, cus = p->dev.cus;
        form = 10 * ((M + 127) / 128 * cols) >= 7 * cus ? 2128 : (M + 63) / 64 * cols <= cus ? 2065 : 2064;
    }
    if (form == 2064) return launch_fit<1, 1, 1>(p, x, y, n, h, w, st);
    if (form == 2065) return launch_fit<1, 1, 2>(p, x, y, n, h, w, st);
    return launch_fit<2, 2, 1>(p, x, y, n, h, w, st);
}

}  // namespace sbn
