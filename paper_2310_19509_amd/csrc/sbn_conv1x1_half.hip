// Group-sparse 1x1 convolution on the wide 16-bit matrix instructions, at the precision of the
// 32-bit form, for gfx950.
//
// v_mfma_f32_16x16x32_f16 multiplies 16 times as many pairs per cycle as the 32-bit instructions, so
// even three of them per product, over blocks filled up with the removed weights' zeros, take a
// fraction of the time of 4x4x1 multiplies over the kept blocks alone.  Every operand is the
// sum of two 16-bit floats, v = s * (hi + lo / 2048): s a power of two, hi the nearest 16-bit float, lo the
// nearest one to 2048 times the rest.  Of the four products three are formed,
//     main += w_hi * x_hi,    cross += w_hi * x_lo,    cross += w_lo * x_hi,
// both sums in 32-bit floats, and main + cross / 2048 is the result.  What is lost, one or two of an
// operand's 24 bits and w_lo * x_lo, is about 9e-8 of the result; in return a sum of K products is
// rounded K / 32 times instead of K times.  sbn_layout.cpp builds the weights' pairs (once, when the
// layer is packed) for the layers where the sum comes out at least as close to the exact result.
//
// Scales.  Weights: one per filter, from its largest weight.  Activations: the wave that stages a
// group of rows takes the largest magnitude among them, as a running maximum over the chunks; when
// a chunk raises it, the sums so far are multiplied by the (exact) power of two.  An activation is
// then off by at most 2^-51 of the group's largest one beyond its own relative error: nothing, as
// long as its piece of four channels holds a value above 2^-27 of the largest.  Groups that hold smaller
// pieces are marked, and there the sums of a filter group that come out small (a pixel whose
// activations are all tiny beside its neighbours') are not taken: the wave computes its outputs
// once more with 32-bit multiply-adds over the kept blocks.  It does the same when a result is not finite (an
// infinite or NaN activation spoils the scale and, times the stored zeros, every output of its pixel).
//
// Mapping.  A workgroup owns T = 16 * PT pixels x 32 * NWV output channels; a wave T pixels x 32 channels
// (two bundles).  Weights are operand A, activations operand B, so a lane ends with four consecutive
// output channels (one filter group) of one pixel: 16-byte stores, no transpose.  Per chunk of 64
// input channels the activations go global -> registers -> pairs -> LDS (two buffers, one barrier per
// chunk), the weights' fragments go straight to registers, one step of 32 channels ahead.  Loads
// return in order, so the weights of a chunk's second step are asked for before the next activations,
// which come from further away.
//
// Two forms, because what bounds a launch differs (512 x 512 layers, batch 64 = 12544 pixels unless stated):
//   PT = 4, NWV = 4: 64 x 128 tiles, a workgroup per tile, three to a compute unit, which cover each
//     other's waits.  Launches of few tiles: 3136 pixels 1024 x 1024 60 -> 34 us (128 x 256 tiles 46).
//   PT = 8, NWV = 8, PIPE: 128 x 256 tiles halve the weights' and the conversions' share of the work; one
//     workgroup per compute unit walks its tiles as one stream of chunks, the next chunk's conversion
//     between the multiplies of this one (the 32-bit form against this: 53 -> 31 us; 100352 pixels
//     298 -> 182 us, 0.87 PFLOP/s of 16-bit multiplies.  A loop of these multiplies alone runs at 1.65
//     on random data, where the clock falls to 1.6 GHz; the rest goes to conversions and LDS reads
//     of the two waves of a SIMD that meet at a chunk's barrier, and to waits for activations).
// The LDS image matters: with rows of 144 bytes every 16-byte read took 7.6 cycles, with the planes
// below 5.6 (stand-alone reads: 5.2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sbn_half.h"
#include "sbn_internal.h"

namespace {

using namespace sbn_half;

constexpr int KC = 64;                    // channels staged at a time

// The outputs [pix0, pix0 + npix) x [ch0, ch0 + nch) by 32-bit multiply-adds over the kept blocks.
// One wave; reached only for data outside the pairs' range.
__device__ __forceinline__ void exact_outputs(const float* __restrict__ x, float* __restrict__ y,
                                                        const uint32_t* __restrict__ records,
                                                        const uint32_t* __restrict__ woff,
                                                        const float* __restrict__ wts, const float* __restrict__ bias,
                                                        int K, int N, int n_chunks, long long pix0, int npix, int ch0,
                                                        int nch, int act)
{
    for (int o = threadIdx.x & 63; o < npix * nch; o += 64) {
        const long long pix = pix0 + o / nch;
        const int ch = ch0 + o % nch, b = ch >> 4, at = ch & 15;         // at = group * 4 + filter of the bundle
        float acc = bias[ch];
        for (int c = 0; c < n_chunks; ++c) {
            const uint32_t* r = records + ((size_t)b * n_chunks + c) * 16;
            const float* w = wts + (size_t)woff[(size_t)b * (n_chunks + 1) + c] * 64 + at * 4;
#pragma unroll 1
            for (int q = 0; q < 16 && r[q] != 0; ++q, w += 64) {
                if (!(r[q] >> (at >> 2) & 1u)) continue;
                const float* xp = x + pix * K + c * 64 + (int)(r[q] >> 12) * 4;
                for (int ci = 0; ci < 4; ++ci) acc = __builtin_fmaf(w[ci], xp[ci], acc);
            }
        }
        const int bits = __builtin_bit_cast(int, acc);
        y[pix * N + ch] = act == SBN_ACT_RELU && bits <= 0 ? 0.f : acc;
    }
}

template <int PT, int NWV, bool PIPE>
__global__ __launch_bounds__(64 * NWV, 2) void conv1x1_half_kernel(
    const float* __restrict__ x, float* __restrict__ y, const uint16_t* __restrict__ wh, const int* __restrict__ wh_exp,
    const float* __restrict__ bias, const uint32_t* __restrict__ records, const uint32_t* __restrict__ woff,
    const float* __restrict__ wts, long long M, int K, int N, int n_bundles, int n_chunks, int n_col_tiles, int n_pix_tiles,
    int pix_stride, int act)
{
    constexpr int T = 16 * PT;                     // pixels of the workgroup
    constexpr int NL = T * 16 / (64 * NWV);        // 16-byte slots per lane and chunk
    constexpr int ROWS = T / NWV;                  // rows that a wave stages: a group that shares a scale
    constexpr int GT = ROWS / 16;                  // 16-pixel tiles per group
    constexpr int NG = NWV;                        // groups of rows
    // LDS image, hi and lo alike: per 8 channels a plane of T rows of 16 bytes.  The 16 rows that a read
    // takes from each of four planes and the 16 that a write stores then cover all banks evenly.
    constexpr int PLANE = T * 16, HALF = 8 * PLANE;
    static_assert(ROWS % 16 == 0 && NG * GT == PT && NL * 4 == ROWS, "tile shape");
    __shared__ __attribute__((aligned(16))) char lds[2][2 * HALF];
    __shared__ int group[2][NWV];                  // per group of rows: exponent, + 256 if it holds tiny pieces

    // A workgroup keeps its column tile and walks every pix_stride-th pixel tile.  Column tiles of one
    // pixel tile run on one XCD (workgroup ids go round the eight XCDs).
    const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;
    int pix_tile = (jj / n_col_tiles) * 8 + xcd;
    const int col_tile = jj % n_col_tiles;
    if (pix_tile >= n_pix_tiles) return;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int bundle = (col_tile * NWV + wave) * 2;                       // first of two
    const bool active = bundle < n_bundles;
    const int b0 = active ? bundle : 0, b1 = bundle + 1 < n_bundles ? bundle + 1 : b0;
    const int n_steps = 2 * n_chunks;
    auto rows_of = [&](int tile) -> int {                                // pixels of the tile that exist
        const long long left = M - (long long)tile * T;
        return (int)(left < 0 ? 0 : left < T ? left : T);
    };

    // ---- activations: slot i of a lane = row wave * ROWS + 16 * (i / 4) + lane / 4, channels
    // 16 * (i % 4) + 4 * (lane % 4) of the chunk.  Rows past the last pixel lie outside the buffer and read
    // as zero; channels past c_in are sent there.
    uint32_t xoff[NL / 4];
#pragma unroll
    for (int i = 0; i < NL / 4; ++i)
        xoff[i] = ((uint32_t)(wave * ROWS + 16 * i + (lane >> 2)) * (uint32_t)K + (uint32_t)(lane & 3) * 4u) * 4u;
    auto issue_x = [&](int tile, int c, v4f (&stage)[NL]) {
        const int rows = rows_of(tile);
        const __amdgpu_buffer_rsrc_t xres = make_rsrc(rows ? x + (long long)tile * T * K : x, (uint32_t)rows * (uint32_t)K * 4u);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const uint32_t outside = c * KC + (i & 3) * 16 + (lane & 3) * 4 < K ? 0u : 0x80000000u;
            stage[i] = __builtin_bit_cast(v4f, buf_load(xres, xoff[i / 4] | outside, (uint32_t)c * (KC * 4) + (i & 3) * 64));
        }
    };
    int run = kFirstExp;                           // running exponent of the rows this wave stages
    uint32_t least = 0xFFFFFFFFu;                  // smallest non-zero piece of four channels (its largest), as bits - 1
    float top = 0.f;
    auto measure_slot = [&](const v4f& v) {
        const float m = max3_abs(v.z, v.w, max3_abs(v.x, v.y, 0.f));
        least = min(least, as_uint(m) - 1u);
        top = fmaxf(top, m);
    };
    auto measured = [&]() {
        const int e = (int)(wave_max(top) >> 23);
        run = e > run ? e : run;
    };
    auto start_measuring = [&]() { run = kFirstExp, least = 0xFFFFFFFFu, top = 0.f; };
    char* const wr = lds[0] + ((lane >> 1) & 1) * PLANE + (wave * ROWS + (lane >> 2)) * 16 + (lane & 1) * 8;
    auto publish_slot = [&](const v4f& v, int i, int buf, float sc, float sc11) {
        split4_to(wr + buf * (2 * HALF) + (i & 3) * (2 * PLANE) + (i / 4) * 256, HALF, v, sc, sc11);
    };
    auto publish_scale = [&](int buf) {
        // a piece below 2^-27 of the largest activation (zeros apart)
        const int tiny = __builtin_amdgcn_ballot_w64(least < tiny_limit(run)) != 0;
        group[buf][wave] = run + tiny * 256;                             // (all lanes write the same)
    };

    // ---- weights: four fragments (two bundles, hi and lo) per step
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(wh, 0xFFFFFFFFu);      // (the packer keeps the table below 4 GiB)
    auto load_w = [&](int step, v8h (&w)[2][2]) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                w[j][s] = __builtin_bit_cast(v8h, buf_load(wres, (uint32_t)lane * 16u + s * 1024u,
                                                           ((uint32_t)(j ? b1 : b0) * (uint32_t)n_steps + (uint32_t)step) * 2048u));
    };

    v4f main[PT][2], cross[PT][2];
    int cur = kFirstExp;                                  // lane g % NG: group's word of group g, whose exponent the sums are in
    auto exponent = [&](int v, int g) { return __builtin_amdgcn_readlane(v, g) & 255; };
    auto rescale = [&](int buf) {
        const int now = group[buf][lane % NG];
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(now != cur) != 0, 0)) {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int d = exponent(cur, g) - exponent(now, g);       // <= 0
#pragma unroll
                for (int t = g * GT; t < (g + 1) * GT; ++t)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            main[t][j][i] = __builtin_amdgcn_ldexpf(main[t][j][i], d);
                            cross[t][j][i] = __builtin_amdgcn_ldexpf(cross[t][j][i], d);
                        }
            }
            cur = now;
        }
    };
    const char* const rd = lds[0] + (lane >> 4) * PLANE + (lane & 15) * 16;
    // A step: per 16-pixel tile the reads of the next tile, six multiplies and a share of the staging
    // of the next chunk.  The share's vector instructions are spread between the multiplies (a
    // multiply holds the matrix unit for 16 cycles and the issue port for 4); the fences between
    // tiles keep the compiler from reading ahead further than the registers allow.
    auto step = [&](int buf, int s, const v8h (&w)[2][2], auto&& share, auto vec_c) {
        constexpr int V = decltype(vec_c)::value;                        // vector instructions after a multiply
        const char* const p = rd + buf * (2 * HALF) + s * (4 * PLANE);
        v8h hi[2], lo[2];
        hi[0] = *(const v8h*)p;
        lo[0] = *(const v8h*)(p + HALF);
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            __builtin_amdgcn_sched_barrier(0);
            if (t + 1 < PT) {
                hi[(t + 1) & 1] = *(const v8h*)(p + (t + 1) * 256);
                lo[(t + 1) & 1] = *(const v8h*)(p + (t + 1) * 256 + HALF);
            }
            const v8h h = hi[t & 1], l = lo[t & 1];
#pragma unroll
            for (int j = 0; j < 2; ++j) cross[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[j][0], l, cross[t][j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 2; ++j) main[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[j][0], h, main[t][j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 2; ++j) cross[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[j][1], h, cross[t][j], 0, 0, 0);
            share(t);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);           // LDS reads
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // a multiply
                __builtin_amdgcn_sched_group_barrier(0x002, V, 0);       // vector
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- main + cross / 2048, back to the data's scale, bias, activation, store
    auto finish = [&](int tile) {
        const long long pix0 = (long long)tile * T;
        const int rows_valid = rows_of(tile);
        const __amdgpu_buffer_rsrc_t yres = make_rsrc(y + pix0 * N, (uint32_t)rows_valid * (uint32_t)N * 4u);
        const int ch_lane = (lane >> 4) * 4, row_lane = lane & 15;
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) main[t][j][i] = __builtin_fmaf(cross[t][j][i], 1.0f / 2048.0f, main[t][j][i]);
        int spoilt = 0;
#pragma unroll
        for (int g = 0; g < NG; ++g) spoilt |= exponent(cur, g) == kSpoilt;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(cur > 255) != 0, 0)) {
            // sums of a filter group below this may be mostly error: K terms, each off by 2^-20 at most
            const float least_sum = (float)K * 16.0f;
#pragma unroll
            for (int t = 0; t < PT; ++t)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (max3_abs(main[t][j].z, main[t][j].w, max3_abs(main[t][j].x, main[t][j].y, 0.f)) < least_sum) spoilt = 1;
        }
        float odd = 0.f;                           // NaN once a result is not finite
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int b = j ? b1 : b0;
            const v4f bj = *(const v4f*)(bias + b * 16 + ch_lane);
            const int4 ej = *(const int4*)(wh_exp + b * 16 + ch_lane);
            const int e4[4] = {ej.x, ej.y, ej.z, ej.w};
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                v4f o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_ldexpf(main[t][j][i], e4[i] + exponent(cur, t / GT) - 141) + bj[i];
                odd = __builtin_fmaf((o.x + o.y) + (o.z + o.w), 0.f, odd);
                main[t][j] = o;
            }
        }
        const bool redo = spoilt || odd != odd;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(redo) != 0, 0)) {
            const int nch = N - bundle * 16 < 32 ? N - bundle * 16 : 32;
            exact_outputs(x, y, records, woff, wts, bias, K, N, n_chunks, pix0, rows_valid, bundle * 16, nch, act);
            return;
        }
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int ch = (bundle + j) * 16 + ch_lane;
                // (A pixel's 128 bytes leave in two instructions.  As streaming stores the halves go to memory one by one,
                // which costs the form that walks many tiles 4 % at 512 channels and 100352 pixels.)
                const uint32_t off = ch < N ? ((uint32_t)(row_lane + t * 16) * (uint32_t)N + (uint32_t)ch) * 4u : 0xFFFFFFF0u;
                v4f o = main[t][j];
                if (act == SBN_ACT_RELU) o = relu4(o);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o), yres, (int)off, 0,
                                                       PIPE ? 0 : 2 /* slc: streaming */);
            }
    };

    // The chunks of all the workgroup's tiles in one stream.  Per chunk: its second step's weights and the
    // activations two chunks on are asked for, the chunk is multiplied, and between the multiplies the
    // next chunk's activations, asked for a chunk ago, are measured (first step) and published (second
    // step).  Past the last tile the loads lie outside the buffer and bring zeros, which are
    // published and never read.
    v8h wa[2][2], wb[2][2];
    v4f x_next[NL], x_far[NL];
    issue_x(pix_tile, 0, x_far);
    load_w(0, wa);
    if constexpr (PIPE) issue_x(pix_tile, 1, x_next);
    start_measuring();
#pragma unroll
    for (int i = 0; i < NL; ++i) measure_slot(x_far[i]);
    measured();
#pragma unroll
    for (int i = 0; i < NL; ++i) publish_slot(x_far[i], i, 0, scale_of(run, 0), scale_of(run, 11));
    publish_scale(0);
    __syncthreads();
    int buf = 0;
    for (; pix_tile < n_pix_tiles; pix_tile += pix_stride) {
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) main[t][j] = cross[t][j] = (v4f){0.f, 0.f, 0.f, 0.f};
        cur = kFirstExp;
        for (int c = 0; c < n_chunks; ++c) {
            if constexpr (PIPE) {
                load_w(2 * c + 1, wb);
                __builtin_amdgcn_sched_barrier(0);
                if (c + 2 < n_chunks)
                    issue_x(pix_tile, c + 2, x_far);
                else
                    issue_x(pix_tile + pix_stride, c + 2 - n_chunks, x_far);
                __builtin_amdgcn_sched_barrier(0);
                rescale(buf);
                if (c + 1 == n_chunks) start_measuring();
                step(buf, 0, wa, [&](int t) {
                    if (t < NL) measure_slot(x_next[t]);
                    if (t == NL) measured();
                }, std::integral_constant<int, 2>());
                load_w(c + 1 < n_chunks ? 2 * c + 2 : 0, wa);
                const float sc = scale_of(run, 0), sc11 = scale_of(run, 11);
                step(buf, 1, wb, [&](int t) {
#pragma unroll
                    for (int i = t * NL / PT; i < (t + 1) * NL / PT; ++i) publish_slot(x_next[i], i, buf ^ 1, sc, sc11);
                }, std::integral_constant<int, 3>());
                publish_scale(buf ^ 1);
#pragma unroll
                for (int i = 0; i < NL; ++i) x_next[i] = x_far[i];
            } else {
                load_w(2 * c + 1, wb);
                __builtin_amdgcn_sched_barrier(0);
                if (c + 1 < n_chunks)
                    issue_x(pix_tile, c + 1, x_far);
                else
                    issue_x(pix_tile + pix_stride, 0, x_far);
                __builtin_amdgcn_sched_barrier(0);
                rescale(buf);
                step(buf, 0, wa, [&](int) {}, std::integral_constant<int, 0>());
                load_w(c + 1 < n_chunks ? 2 * c + 2 : 0, wa);
                step(buf, 1, wb, [&](int) {}, std::integral_constant<int, 0>());
                if (c + 1 == n_chunks) start_measuring();
#pragma unroll
                for (int i = 0; i < NL; ++i) measure_slot(x_far[i]);
                measured();
                const float sc = scale_of(run, 0), sc11 = scale_of(run, 11);
#pragma unroll
                for (int i = 0; i < NL; ++i) publish_slot(x_far[i], i, buf ^ 1, sc, sc11);
                publish_scale(buf ^ 1);
            }
            buf ^= 1;
            __syncthreads();
        }
        if (active) finish(pix_tile);
    }
}

template <int PT, int NWV, bool PIPE>
int launch(const sbn_packed* p, const float* x, float* y, long long M, hipStream_t st)
{
    const sbn::DeviceLayout& L = p->dev;
    constexpr int T = 16 * PT;
    const long long n_pix_tiles = (M + T - 1) / T;
    const int per_tile = 2 * NWV, n_col_tiles = (L.n_bundles + per_tile - 1) / per_tile;
    // PIPE: one workgroup per compute unit, which walks its pixel tiles as one stream of chunks; otherwise a
    // workgroup per tile.  The column tiles of a pixel tile go to one of the eight XCDs.
    const long long room = PIPE ? std::max(1, L.cus / 8 / n_col_tiles) : (n_pix_tiles + 7) / 8;
    const long long pix_slots = 8 * std::min(room, (n_pix_tiles + 7) / 8);
    const long long grid = pix_slots * n_col_tiles;
    if (grid > 0x7FFFFFFFll || n_pix_tiles + pix_slots > 0x7FFFFFFFll)
        return sbn::fail(SBN_EINVAL, "too many pixels for one launch (%lld)", M);
    hipLaunchKernelGGL((conv1x1_half_kernel<PT, NWV, PIPE>), dim3((unsigned)grid), dim3(64 * NWV), 0, st, x, y, L.d_wh, L.d_wh_exp,
                       L.d_bias, L.d_records, L.d_woff, L.d_wts, M, p->c_in, p->c_out, L.n_bundles, L.n_chunks, n_col_tiles,
                       (int)n_pix_tiles, (int)pix_slots, p->act);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sbn::fail(SBN_EHIP, "conv1x1 launch: %s", hipGetErrorString(e));
    return SBN_OK;
}

}  // namespace

namespace sbn {

int launch_conv1x1_half(const sbn_packed* p, const float* x, float* y, long long M, int form, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (!p->dev.d_wh) return fail(SBN_EINVAL, "internal error: the layer has no 16-bit pairs");
    return form == 2256 ? launch<8, 8, true>(p, x, y, M, st) : launch<4, 4, false>(p, x, y, M, st);
}

}  // namespace sbn
