// Group-sparse 1x1 convolution on the wide 16-bit matrix instructions, with every bit of the 32-bit operands,
// for gfx950.
//
// v_mfma_f32_32x32x16_bf16 multiplies 16 times as many pairs per cycle as the 32-bit instructions, so even
// six of them per product, over blocks filled up with the removed weights' zeros, take less time than 4x4x1
// multiplies over the kept blocks where a layer keeps enough of them (conv1x1_wide_pays has the rule).  Every
// operand is the exact sum of three bfloat16, v = a + b + c (8 + 8 + 8 bits; the exponent range is that of
// 32-bit floats, so there is nothing to scale and no value depends on its neighbours).  Of the nine products
// six are formed,
//     main += w_a * x_a,    cross += w_a * x_c + w_c * x_a + w_b * x_b + w_a * x_b + w_b * x_a,
// both sums in 32-bit floats; the other three are at most 2^-24 of the product, 2e-9 of it on average, where one
// rounding of a 32-bit sum is at most 2^-24 and 2.5e-8 on average.  `main`, the only long sum of full-sized terms, is
// rounded c_in / 16 times instead of once per kept weight.  Relative error (2-norm, units of 1e-8, half-zero
// activations, c_in = 128 / 256 / 512 / 1024, 50 % kept): 4.1 / 5.3 / 7.1 / 9.9; one 32-bit sum 10.6 / 14.6 / 20.5 / 28.8,
// two sums 8.2 / 10.8 / 14.9 / 20.6; one active channel per pixel 2.6 against 2.5.  (The splitting is that of the known
// emulations of single precision on bfloat16 units: Henry, Tang, Heinecke, "Leveraging the bfloat16 artificial
// intelligence datatype for higher-precision computations", 2019.)
//
// What bfloat16 cannot hold is done again with 32-bit multiply-adds over the kept blocks, output by output: results that are not finite (an infinite or NaN activation, times the stored
// zeros, reaches every output of its pixel), sums below 2^-100, and, in pixels that hold a non-zero
// activation below 2^-100 (whose last bits can lie below the smallest bfloat16), sums so small that those bits could matter.
//
// Mapping.  A workgroup owns T = 32 * PX pixels x 32 * NWV output channels; a wave T pixels x 32 channels
// (two bundles).  Weights are operand A, activations operand B, so a lane ends with four times four consecutive
// output channels (filter groups) of one pixel: 16-byte stores.  Per chunk of 64 input
// channels the activations go global -> registers -> triples -> LDS (two buffers, one barrier per
// chunk), the weights' fragments go straight to registers, two steps of 16 channels ahead.
//
// Two forms (launch_conv1x1_wide has the rule):
//   PX = 2, NWV = 4: 64 x 128 tiles, a workgroup per tile, three to a compute unit, which cover each
//     other's waits.
//   PX = 4, NWV = 8, PIPE: 128 x 256 tiles halve the weights' and the conversions' share of the work; one
//     workgroup per compute unit walks its tiles as one stream of chunks.
// In both the next chunk's conversion goes between the multiplies of this one.  The matrix unit is busy 63 % of the
// time in the second form (512 x 512, 100352 pixels, 260 us: 1.2 PFLOP/s; a loop of these multiplies alone on random
// data reaches 1.85): activations, weights and LDS reads that arrive late cost 22 %, uneven rounds 13 %.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sbn_internal.h"
#include "sbn_wide.h"

namespace {

using namespace sbn_wide;

constexpr int KC = 64;                    // channels staged at a time
constexpr int STEPS = KC / 16;            // multiplies per chunk, tile and product

// Four output channels ch .. ch + 3 (one filter group) of pixel pix by 32-bit multiply-adds over the kept blocks: by one
// lane, four pieces' loads at a time, or by a wave, a lane per piece of four chunks.
struct Exact {
    const float* __restrict__ x;
    float* __restrict__ y;
    const uint32_t* __restrict__ records;
    const uint32_t* __restrict__ woff;
    const float* __restrict__ wts;
    const float* __restrict__ bias;
    int K, N, n_chunks, act;

    __device__ __forceinline__ void store(v4f acc, long long pix, int ch) const
    {
        acc += *(const v4f*)(bias + ch);
        if (act == SBN_ACT_RELU) acc = relu4_of_any(acc);
        *(v4f*)(y + pix * N + ch) = acc;
    }
    __device__ __forceinline__ void by_lane(long long pix, int ch) const
    {
        const int b = ch >> 4, g = (ch >> 2) & 3;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < n_chunks; ++c) {
            const uint32_t* r = records + ((size_t)b * n_chunks + c) * 16;
            const v4f* w = (const v4f*)(wts + (size_t)woff[(size_t)b * (n_chunks + 1) + c] * 64 + g * 16);
            const float* xc = x + pix * K + c * 64;
            for (int q = 0; q < 16 && r[q] != 0; q += 4, w += 64) {      // (past the record's end: other entries, or the slack behind the table)
                v4f xv[4], wv[4][4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    xv[u] = *(const v4f*)(xc + (int)(r[q + u] >> 12) * 4);
#pragma unroll
                    for (int co = 0; co < 4; ++co) wv[u][co] = w[u * 16 + co];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) add_piece(acc, wv[u], xv[u], r[q + u] >> g & 1u);
            }
        }
        store(acc, pix, ch);
    }
    __device__ __forceinline__ void by_wave(long long pix, int ch, int lane) const
    {
        const int b = ch >> 4, g = (ch >> 2) & 3;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int c = lane >> 4; c < n_chunks; c += 4) {
            const uint32_t r = records[((size_t)b * n_chunks + c) * 16 + (lane & 15)];
            if (!(r >> g & 1u)) continue;
            const v4f* w = (const v4f*)(wts + ((size_t)woff[(size_t)b * (n_chunks + 1) + c] + (lane & 15)) * 64 + g * 16);
            const v4f xv = *(const v4f*)(x + pix * K + c * 64 + (int)(r >> 12) * 4), wv[4] = {w[0], w[1], w[2], w[3]};
            add_piece(acc, wv, xv, true);
        }
        acc = sum_over_wave(acc);
        if (lane == 0) store(acc, pix, ch);
    }
};

template <int PX, int NWV, bool PIPE>
__global__ __launch_bounds__(64 * NWV, PIPE ? 2 : 3) void conv1x1_wide_kernel(
    const float* __restrict__ x, float* __restrict__ y, const uint16_t* __restrict__ wt, uint32_t wt_bytes,
    const float* __restrict__ bias, const uint32_t* __restrict__ records, const uint32_t* __restrict__ woff,
    const float* __restrict__ wts, long long M, int K, int N, int n_bundles, int n_chunks, int n_col_tiles, int n_pix_tiles,
    int pix_stride, float tiny_sum, int act)
{
    constexpr int T = 32 * PX;                     // pixels of the workgroup
    constexpr int NL = T * 16 / (64 * NWV);        // 16-byte slots per lane and chunk
    constexpr int ROWS = 16;                       // rows that a wave stages, four lanes to a row
    // LDS image, a, b and c alike: per 8 channels a plane of T rows of 16 bytes.  The 32 rows that a read
    // takes from each of two planes cover all banks evenly; the two planes that a write goes to lie a multiple of 256
    // bytes apart, so that rows of both meet in a bank.  (Counters: 0.59 conflict cycles per active LDS cycle in the
    // 128 x 256 form, 0.79 in the other.)
    constexpr int PLANE = T * 16, PART = 8 * PLANE, IMAGE = 3 * PART;
    static_assert(ROWS * NWV == T && NL == 4, "tile shape");
    __shared__ __attribute__((aligned(16))) char lds[2][IMAGE];
    __shared__ unsigned long long mark[2][NWV];    // per staging wave: four bits per row, set by lanes that met tiny values in it

    // A workgroup keeps its column tile and walks every pix_stride-th pixel tile.  Column tiles of one
    // pixel tile run on one XCD (workgroup ids go round the eight XCDs).
    const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;
    int pix_tile = (jj / n_col_tiles) * 8 + xcd;
    const int col_tile = jj % n_col_tiles;
    if (pix_tile >= n_pix_tiles) return;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pair = col_tile * NWV + wave;                              // 32 channels, two bundles
    const bool active = pair * 2 < n_bundles;
    const int n_steps = STEPS * n_chunks;
    auto rows_of = [&](int tile) -> int {                                // pixels of the tile that exist
        const long long left = M - (long long)tile * T;
        return (int)(left < 0 ? 0 : left < T ? left : T);
    };

    // ---- activations: slot i of a lane = row wave * 16 + lane / 4, channels 16 * i + 4 * (lane % 4) of the
    // chunk.  Rows past the last pixel lie outside the buffer and read as zero; channels past c_in are sent there.
    const uint32_t xoff = ((uint32_t)(wave * ROWS + (lane >> 2)) * (uint32_t)K + (uint32_t)(lane & 3) * 4u) * 4u;
    auto issue_x = [&](int tile, int c, int i, v4f& to) {
        const int rows = rows_of(tile);
        const __amdgpu_buffer_rsrc_t xres = make_rsrc(rows ? x + (long long)tile * T * K : x, (uint32_t)rows * (uint32_t)K * 4u);
        const uint32_t outside = c * KC + i * 16 + (lane & 3) * 4 < K ? 0u : 0x80000000u;
        to = __builtin_bit_cast(v4f, buf_load(xres, xoff | outside, (uint32_t)c * (KC * 4) + i * 64));
    };
    uint32_t least = 0xFFFFFFFFu;                  // smallest non-zero magnitude of this lane's row so far
    char* const wr = lds[0] + ((lane >> 1) & 1) * PLANE + (wave * ROWS + (lane >> 2)) * 16 + (lane & 1) * 8;
    auto publish_slot = [&](const v4f& v, int i, int buf) {
        least = least_magnitude(v, least);
        split4_to(wr + buf * IMAGE + i * (2 * PLANE), PART, v);
    };
    auto publish_mark = [&](int buf) { mark[buf][wave] = __builtin_amdgcn_ballot_w64(least < kTiny); };  // (all lanes write the same)

    // ---- weights: three fragments (a, b, c) per step of 16 channels
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(wt, wt_bytes);
    const uint32_t w0 = (uint32_t)(active ? pair : 0) * (uint32_t)n_steps * 3072u;
    auto load_w = [&](int step, v8b (&w)[3]) {
#pragma unroll
        for (int s = 0; s < 3; ++s) w[s] = __builtin_bit_cast(v8b, buf_load(wres, (uint32_t)lane * 16u + s * 1024u, w0 + (uint32_t)step * 3072u));
    };

    v16f main[PX], cross[PX];
    const char* const rd = lds[0] + (lane >> 5) * PLANE + (lane & 31) * 16;
    auto read_x = [&](int buf, int s, int t, int part) {
        return *(const v8b*)(rd + buf * IMAGE + s * (2 * PLANE) + t * 512 + part * PART);
    };
    // A step: two 32-pixel tiles at a time, their multiplies in turn (a multiply takes 32 cycles, one that adds to the same
    // sum can follow after 56).  The activations' parts c, a, b are read a phase before they are used, into the
    // registers that the phase before has finished with; a share of the staging of the next chunk goes between the multiplies.
    v8b fa[2], fb[2], fc[2];
    auto step = [&](int buf, int s, const v8b (&w)[3], auto&& share) {
#pragma unroll
        for (int t = 0; t < PX; t += 2) {
            const int tn = t + 2 < PX ? t + 2 : 0, sn = t + 2 < PX ? s : s + 1;
            auto mul = [&](const v8b& wp, const v8b (&xp)[2], v16f* sum) {
#pragma unroll
                for (int u = 0; u < 2; ++u) sum[t + u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wp, xp[u], sum[t + u], 0, 0, 0);
            };
            auto read = [&](int at_s, int at_t, int part, v8b (&to)[2]) {
#pragma unroll
                for (int u = 0; u < 2; ++u) to[u] = read_x(buf, at_s, at_t + u, part);
                __builtin_amdgcn_sched_barrier(0);
            };
            auto spread = [&](auto n_c) {          // vector instructions go between the multiplies
#pragma unroll
                for (int i = 0; i < decltype(n_c)::value; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            read(s, t, 1, fb);
            mul(w[0], fc, cross);
            spread(std::integral_constant<int, 2>());
            if (sn < STEPS) read(sn, tn, 2, fc);
            mul(w[2], fa, cross);
            mul(w[0], fa, main);
            mul(w[1], fa, cross);
            share(t);
            spread(std::integral_constant<int, 6>());
            if (sn < STEPS) read(sn, tn, 0, fa);
            mul(w[1], fb, cross);
            mul(w[0], fb, cross);
            spread(std::integral_constant<int, 4>());
        }
    };

    // ---- main + (cross + bias), activation, store
    auto finish = [&](int tile, uint32_t marked) {
        int l = lane;
        asm volatile("" : "+v"(l));               // (offsets are worked out here: kept across the tiles they cost the loop its registers)
        const long long pix0 = (long long)tile * T;
        const int rows_valid = rows_of(tile);
        const __amdgpu_buffer_rsrc_t yres = make_rsrc(y + pix0 * N, (uint32_t)rows_valid * (uint32_t)N * 4u);
        const __amdgpu_buffer_rsrc_t bres = make_rsrc(bias, (uint32_t)n_bundles * 64u);
        const int ch_lane = pair * 32 + (l >> 5) * 4, row_lane = l & 31;                  // + 8 * g, + 32 * t
        float odd = 0.f;                           // NaN once a result is not finite
        uint32_t low = 0xFFFFFFFFu;                // smallest non-zero sum
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const v4f bg = __builtin_bit_cast(v4f, buf_load(bres, (uint32_t)(ch_lane + 8 * g) * 4u, 0));
#pragma unroll
            for (int t = 0; t < PX; ++t) {
                v4f o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    o[i] = main[t][4 * g + i] + (cross[t][4 * g + i] + bg[i]);
                    low = min(low, magnitude(main[t][4 * g + i]));
                    cross[t][4 * g + i] = o[i];
                }
                odd = __builtin_fmaf((o.x + o.y) + (o.z + o.w), 0.f, odd);
            }
        }
        uint32_t redo = 0;                         // bit 4 * t + g: to be done again
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd != odd || low < kTiny || marked != 0) != 0, 0)) {
#pragma unroll
            for (int t = 0; t < PX; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    bool bad = false;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float o = cross[t][4 * g + i], m = main[t][4 * g + i];
                        bad |= o - o != 0.f || magnitude(m) < kTiny || ((marked >> t & 1u) && __builtin_fabsf(m) < tiny_sum);
                    }
                    if (bad && t * 32 + row_lane < rows_valid && ch_lane + 8 * g < N) redo |= 1u << (4 * t + g);
                }
        }
#pragma unroll
        for (int t = 0; t < PX; ++t) store_tile<PIPE ? 0 : 2>(cross[t], yres, t * 32, pair * 32, N, act == SBN_ACT_RELU, l);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(redo != 0) != 0, 0)) {
            const Exact exact = {x, y, records, woff, wts, bias, K, N, n_chunks, act};
            auto pixel = [&](int k, int ln) { return pix0 + (k >> 2) * 32 + (ln & 31); };
            auto channel = [&](int k, int ln) { return pair * 32 + (ln >> 5) * 4 + 8 * (k & 3); };
            do_again(redo, 4 * PX, [&](int k, int ln) { exact.by_wave(pixel(k, ln), channel(k, ln), l); },
                     [&](int k) { exact.by_lane(pixel(k, l), channel(k, l)); });
        }
    };

    // The chunks of all the workgroup's tiles in one stream.  In step s of a chunk its weights of step s + 2 are asked
    // for, slot s of the next chunk's activations, asked for a chunk ago, is published and, into the same
    // registers, that of the chunk after it asked for.  (Loads return in order: weights two steps ahead leave the
    // activations, which come from further away, three steps.)  Past the last tile the loads lie outside the buffer and
    // bring zeros, which are published and never read.
    v8b w[4][3];
    v4f xs[NL];
    {
        v4f first[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) issue_x(pix_tile, 0, i, first[i]);
        load_w(0, w[0]);
        load_w(1, w[1]);
#pragma unroll
        for (int i = 0; i < NL; ++i) issue_x(pix_tile, 1, i, xs[i]);
#pragma unroll
        for (int i = 0; i < NL; ++i) publish_slot(first[i], i, 0);
    }
    publish_mark(0);
    __syncthreads();
    int buf = 0;
    for (; pix_tile < n_pix_tiles; pix_tile += pix_stride) {
#pragma unroll
        for (int t = 0; t < PX; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) main[t][i] = cross[t][i] = 0.f;
        uint32_t marked = 0;
        for (int c = 0; c < n_chunks; ++c) {
            const bool last = c + 1 == n_chunks;
            if (last) {                            // bit t: the pixel of tile t holds tiny values
                least = 0xFFFFFFFFu;               // (what is published from here on is the next tile's)
#pragma unroll
                for (int t = 0; t < PX; ++t)
                    marked |= ((mark[buf][2 * t + ((lane >> 4) & 1)] >> (4 * (lane & 15))) & 15u) != 0 ? 1u << t : 0u;
            }
            const bool wrap = c + 2 >= n_chunks;   // the chunk after the next is the next tile's
            const int far_tile = wrap ? pix_tile + pix_stride : pix_tile, far = wrap ? c + 2 - n_chunks : c + 2;
#pragma unroll
            for (int u = 0; u < 2; ++u) fc[u] = read_x(buf, 0, u, 2);
#pragma unroll
            for (int u = 0; u < 2; ++u) fa[u] = read_x(buf, 0, u, 0);
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                load_w(s + 2 < STEPS ? STEPS * c + s + 2 : (last ? 0 : STEPS * (c + 1)) + s + 2 - STEPS, w[(s + 2) & 3]);
                step(buf, s, w[s], [&](int t) {
                    if (t) return;
                    publish_slot(xs[s], s, buf ^ 1);
                    issue_x(far_tile, far, s, xs[s]);
                });
            }
            publish_mark(buf ^ 1);
            buf ^= 1;
            __syncthreads();
        }
        if (active) finish(pix_tile, marked);
    }
}

// For launches of a few 32 x 32 tiles per compute unit.  A workgroup owns one, and its four waves take the units of 32 input channels in
// turn.  A wave shares nothing while it works: it stages its own activations through its own part of LDS (as they
// are, in rows of 32 channels, the 16-byte slot s of pixel r at s ^ (r / 2 % 8), so that neither side meets a bank twice),
// splits them in registers and multiplies; the loads of its next unit are in flight meanwhile, and there is no barrier
// until the waves' results meet in LDS, where they are added in 64 bits.  Bound by the loads: 91 MB pass the L1 caches
// for 1100 pixels, 512 x 512.  (Tiles of 32 x 64 and 64 x 32 halve that, but leave units idle: the same time there, up to a fifth more in
// launches of fewer tiles; eight waves: a workgroup per unit instead of three, 11.9 us against 10.5.)
constexpr int NS = 4;
__global__ __launch_bounds__(64 * NS, 2) void conv1x1_wide_split_kernel(
    const float* __restrict__ x, float* __restrict__ y, const uint16_t* __restrict__ wt, uint32_t wt_bytes,
    const float* __restrict__ bias, const uint32_t* __restrict__ records, const uint32_t* __restrict__ woff,
    const float* __restrict__ wts, long long M, int K, int N, int n_bundles, int n_chunks, int n_pairs, int n_pix_tiles,
    int pix_fast, float tiny_sum, int act)
{
    __shared__ __attribute__((aligned(16))) char lds[NS][4096];          // 32 pixels x 32 channels, then 32 x 32 results
    __shared__ uint8_t tiny_row[NS][32];           // 1: the wave met a non-zero activation below 2^-100 in the pixel

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;                // the tiles that share the larger operand on one XCD
    const int n_fast = pix_fast ? n_pix_tiles : n_pairs;
    const int slow = (jj / n_fast) * 8 + xcd, fast = jj % n_fast;
    const int pix_tile = pix_fast ? fast : slow, pair = pix_fast ? slow : fast;      // 32 channels, two bundles
    if (pix_tile >= n_pix_tiles || pair >= n_pairs) return;
    const long long pix0 = (long long)pix_tile * 32;
    const int rows = (int)(M - pix0 < 32 ? M - pix0 : 32);
    const int n_units = (K + 31) / 32;

    // ---- activations: slot i of a lane = row i * 8 + lane / 8, channels 4 * (lane % 8) of the unit.  Weights: three fragments (a, b, c)
    // per step of 16 channels.  Past the last unit every lane's offset lies outside the buffers.
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(x + pix0 * K, (uint32_t)rows * (uint32_t)K * 4u);
    const int slot = lane & 7;
    const uint32_t xoff = ((uint32_t)(lane >> 3) * (uint32_t)K + (uint32_t)slot * 4u) * 4u;
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(wt, wt_bytes);
    const uint32_t w0 = (uint32_t)pair * (uint32_t)(STEPS * n_chunks) * 3072u;
    struct Set {
        v4f x[4];
        v8b w[2][3];
    };
    auto issue = [&](int u, Set& s) {
        const bool real = u < n_units;
        const int uu = real ? u : 0;
        const uint32_t past = real && uu * 32 + slot * 4 < K ? 0u : 0x80000000u;
#pragma unroll
        for (int i = 0; i < 4; ++i) s.x[i] = __builtin_bit_cast(v4f, buf_load(xres, (xoff + (uint32_t)i * (uint32_t)K * 32u) | past, (uint32_t)uu * 128u));
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int p = 0; p < 3; ++p)
                s.w[h][p] = __builtin_bit_cast(v8b, buf_load(wres, real ? (uint32_t)lane * 16u + p * 1024u : 0xFFFFFFF0u, real ? w0 + (uint32_t)(uu * 2 + h) * 3072u : 0u));
    };

    char* const wr = lds[wave] + (lane >> 3) * 128;
    const char* const rd = lds[wave] + (lane & 31) * 128;
    v16f main, cross;
#pragma unroll
    for (int i = 0; i < 16; ++i) main[i] = cross[i] = 0.f;
    uint32_t least = 0xFFFFFFFFu;
    auto multiply = [&](const Set& s) {
        wave_lds_order();
#pragma unroll
        for (int i = 0; i < 4; ++i) *(v4f*)(wr + i * 1024 + ((slot ^ (i * 4 + (lane >> 4))) & 7) * 16) = s.x[i];
        wave_lds_order();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int at = h * 4 + (lane >> 5) * 2, f = (lane & 31) >> 1;
            const v4f lo = *(const v4f*)(rd + ((at ^ f) & 7) * 16), hi = *(const v4f*)(rd + (((at + 1) ^ f) & 7) * 16);
            least = least_magnitude(hi, least_magnitude(lo, least));
            uint32_t p[3][4];
            split2(lo.x, lo.y, p[0][0], p[1][0], p[2][0]);
            split2(lo.z, lo.w, p[0][1], p[1][1], p[2][1]);
            split2(hi.x, hi.y, p[0][2], p[1][2], p[2][2]);
            split2(hi.z, hi.w, p[0][3], p[1][3], p[2][3]);
            v8b q[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const v4u words = {p[k][0], p[k][1], p[k][2], p[k][3]};
                q[k] = __builtin_bit_cast(v8b, words);
            }
            auto mul = [&](int wp, int xp, v16f& sum) { sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s.w[h][wp], q[xp], sum, 0, 0, 0); };
            mul(0, 2, cross);
            mul(0, 0, main);
            mul(2, 0, cross);
            mul(1, 1, cross);
            mul(1, 0, cross);
            mul(0, 1, cross);
        }
    };

    Set s0, s1;
    issue(wave, s0);
    for (int u = wave; u < n_units; u += 2 * NS) {
        issue(u + NS, s1);
        multiply(s0);
        issue(u + 2 * NS, s0);
        if (u + NS < n_units) multiply(s1);
    }

    // ---- the waves' results, [group of 4 + 4 channels][lane]; wave g then adds up group g
    __syncthreads();
    const unsigned long long met = __builtin_amdgcn_ballot_w64(least < kTiny);           // (two lanes per pixel)
    if (lane < 32) tiny_row[wave][lane] = ((met | met >> 32) >> lane & 1u) != 0;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        v4f o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = main[4 * g + i] + cross[4 * g + i];
        *(v4f*)(lds[wave] + g * 1024 + lane * 16) = o;
    }
    __syncthreads();
    const int ch = pair * 32 + wave * 8 + (lane >> 5) * 4, row = lane & 31;
    double sum[4] = {0., 0., 0., 0.};
    bool marked = false;
#pragma unroll
    for (int n = 0; n < NS; ++n) {
        const v4f v = *(const v4f*)(lds[n] + wave * 1024 + lane * 16);
        marked |= tiny_row[n][row] != 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] += (double)v[i];
    }
    const v4f bv = *(const v4f*)(bias + (ch < n_bundles * 16 ? ch : 0));
    v4f o;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float s = (float)sum[i];
        o[i] = (float)(sum[i] + (double)bv[i]);
        bad |= o[i] - o[i] != 0.f || magnitude(s) < kTiny || (marked && __builtin_fabsf(s) < tiny_sum);
    }
    const uint32_t redo = bad && row < rows && ch < N ? 1u : 0u;
    if (act == SBN_ACT_RELU) o = relu4(o);
    const __amdgpu_buffer_rsrc_t yres = make_rsrc(y + pix0 * N, (uint32_t)rows * (uint32_t)N * 4u);
    const uint32_t off = ch < N ? ((uint32_t)row * (uint32_t)N + (uint32_t)ch) * 4u : 0xFFFFFFF0u;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o), yres, (int)off, 0, 0);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(redo != 0) != 0, 0)) {
        const Exact exact = {x, y, records, woff, wts, bias, K, N, n_chunks, act};
        auto pixel = [&](int ln) { return pix0 + (ln & 31); };
        auto channel = [&](int ln) { return pair * 32 + wave * 8 + (ln >> 5) * 4; };
        do_again(redo, 1, [&](int, int ln) { exact.by_wave(pixel(ln), channel(ln), lane); }, [&](int) { exact.by_lane(pixel(lane), channel(lane)); });
    }
}

// sums below this may have lost more than 2^-24 of themselves to activations below 2^-100 (c_in terms, each off by 2^-125 of a weight)
float tiny_sum_of(const sbn_packed* p) { return std::max((float)p->c_in * p->dev.w_top * 0x1p-101f, 0x1p-100f); }

int launch_split(const sbn_packed* p, const float* x, float* y, long long M, hipStream_t st)
{
    const sbn::DeviceLayout& L = p->dev;
    const long long n_pix_tiles = (M + 31) / 32;
    const int n_pairs = (L.n_bundles + 1) / 2, pix_fast = n_pairs >= 8 && n_pairs >= n_pix_tiles;      // (as in the few-pixel kernel)
    const long long slow = pix_fast ? n_pairs : n_pix_tiles, fast = pix_fast ? n_pix_tiles : n_pairs;
    const long long grid = (slow + 7) / 8 * 8 * fast;
    if (grid > 0x7FFFFFFFll) return sbn::fail(SBN_EINVAL, "too many pixels for one launch (%lld)", M);
    hipLaunchKernelGGL(conv1x1_wide_split_kernel, dim3((unsigned)grid), dim3(64 * NS), 0, st, x, y, L.d_wt,
                       (uint32_t)(L.wt.size() * sizeof(uint16_t)), L.d_bias, L.d_records, L.d_woff, L.d_wts, M, p->c_in, p->c_out,
                       L.n_bundles, L.n_chunks, n_pairs, (int)n_pix_tiles, pix_fast, tiny_sum_of(p), p->act);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sbn::fail(SBN_EHIP, "conv1x1 launch: %s", hipGetErrorString(e));
    return SBN_OK;
}

template <int PX, int NWV, bool PIPE>
int launch(const sbn_packed* p, const float* x, float* y, long long M, hipStream_t st)
{
    const sbn::DeviceLayout& L = p->dev;
    constexpr int T = 32 * PX;
    const long long n_pix_tiles = (M + T - 1) / T;
    const int per_tile = 2 * NWV, n_col_tiles = (L.n_bundles + per_tile - 1) / per_tile;
    // PIPE: one workgroup per compute unit, which walks its pixel tiles as one stream of chunks; otherwise a
    // workgroup per tile.  The column tiles of a pixel tile go to one of the eight XCDs.
    const long long room = PIPE ? std::max(1, L.cus / 8 / n_col_tiles) : (n_pix_tiles + 7) / 8;
    const long long pix_slots = 8 * std::min(room, (n_pix_tiles + 7) / 8);
    const long long grid = pix_slots * n_col_tiles;
    if (grid > 0x7FFFFFFFll || n_pix_tiles + pix_slots > 0x7FFFFFFFll)
        return sbn::fail(SBN_EINVAL, "too many pixels for one launch (%lld)", M);
    hipLaunchKernelGGL((conv1x1_wide_kernel<PX, NWV, PIPE>), dim3((unsigned)grid), dim3(64 * NWV), 0, st, x, y, L.d_wt,
                       (uint32_t)(L.wt.size() * sizeof(uint16_t)), L.d_bias, L.d_records, L.d_woff, L.d_wts, M, p->c_in, p->c_out,
                       L.n_bundles, L.n_chunks, n_col_tiles, (int)n_pix_tiles, (int)pix_slots, tiny_sum_of(p), p->act);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sbn::fail(SBN_EHIP, "conv1x1 launch: %s", hipGetErrorString(e));
    return SBN_OK;
}

}  // namespace

namespace sbn {

// Up to four tiles of 32 x 32 per compute unit the launch waits for its loads, which the kernel of such tiles has more of in
// flight; no lower line: the few-pixel kernel is asked first.  Of 66 random layers of 200 to 9000 pixels and 96 to 1024 channels,
// sparsity 0 to 40 %, every one gained, 1.29 times on average (30 %, us: 1100 pixels, 512 x 512 12.0 / 10.5; 784, 1024 x 1024 23.6 / 20.3;
// 3136, 256 x 256 10.5 / 8.4; 275, 1024 x 1024 13.4 / 11.2).  In 1100 to 1500 tiles it loses as much.
static long long split_tiles(const sbn_packed* p, long long M) { return (M + 31) / 32 * ((p->dev.n_bundles + 1) / 2); }
static bool split_pays(const sbn_packed* p, long long M) { return split_tiles(p, M) <= 4ll * p->dev.cus; }

// The same tiles for layers that keep too little for the other forms on triples, from 1.25 per compute unit on (below, the few-pixel kernel and the
// 32-bit forms have their round to themselves).  With more than 64 output channels, and with little kept at all, the 32-bit
// forms gain on launches of few pixels, whose time is that of the weights; up to 64 output channels of at least 768 gain from 0.6 tiles on (18 layers, 1.46 times, none slower:
// 4735 pixels, 1024 x 64, 60 % 23.1 / 12.0; from 512 channels on 11 of 48 lose).  7006 random layers, 400 to 300000 pixels, 16 to 1024 channels each way, 30 to 95 % (us, before / so):
//   up to 64 output channels, 122 of them taken: 1.49 times faster on average, none slower by 3 %
//     12544, 1024 x 64, 70 %  53.1 / 20.7    8200, 1024 x 56, 90 %  38.1 / 15.7    11720, 256 x 64, 30 %  11.8 / 7.3    15680, 528 x 64, 60 %  23.6 / 14.5
//   more, 112 taken: 1.29 times, two slower, at most by 4 %
//     7186, 1024 x 128, 50 %  36.4 / 20.8    7892, 928 x 128, 70 %  35.8 / 19.8    10192, 512 x 96, 60 %  21.1 / 13.1
//   not taken: 743, 1024 x 1024, 80 %  15.5 / 17.4    528, 512 x 1024, 80 %  8.5 / 10.1    6272, 192 x 128, 70 %  6.8 / 7.9    784, 272 x 544, 95 %  5.4 / 7.4
bool conv1x1_split_chosen(const sbn_packed* p, long long M)
{
    const long long tiles = split_tiles(p, M), cus = p->dev.cus;
    if (!p->dev.d_wt || !conv1x1_split_pays(p) || tiles > 4 * cus) return false;
    if (p->c_out <= 64 && p->c_in >= 768 && 5 * tiles > 3 * cus) return true;
    if (4 * tiles <= 5 * cus) return false;
    const double share = 16.0 * (double)p->dev.n_present / ((double)p->c_in * p->c_out);
    return p->c_out <= 64 ? share >= 0.15 || tiles > 2 * cus : M >= 4ll * p->c_out;
}

// Launches of a few more 64 x 128 tiles than compute units, where some units have two and most one, need more of a margin
// (2254 pixels, 55 % kept: 512 x 1024 21.1 us against 19.5 of the 32-bit form, 1024 x 1024 35.5 against 34.3; 1 568 pixels 14 against 18).
bool conv1x1_wide_chosen(const sbn_packed* p, long long M)
{
    const long long tiles = (M + 63) / 64 * ((p->c_out + 127) / 128), cus = p->dev.cus;
    return p->dev.d_wt && conv1x1_wide_margin(p) >= (tiles > cus && 3 * tiles < 4 * cus && !split_pays(p, M) ? 1.45 : 1.0);
}
// Fewer pixels than four times the output channels read mostly weights, 6 bytes for each of the layer's against 4 for each kept: a tie at a margin near 1
// when they lie in the L2 (1372 pixels, 512 x 512, 50 %, 11.3 against 11.5 us), a loss when they do not (13 layers in turn on seven images 129 against 125).
bool conv1x1_wide_few(const sbn_packed* p, long long M)
{
    return conv1x1_wide_chosen(p, M) && split_pays(p, M) && (M >= 4ll * p->c_out || conv1x1_wide_margin(p) >= 1.25);
}

// form 0: 128 x 256 tiles where they fill three quarters of one round of a tile per compute unit, or four fifths of several,
// else 64 x 128 tiles (512 x 512: 62720 pixels, 3.8 rounds, 163 us against 186; 37632, 2.3 of 3, 116 against 105; 25088, 1.5 of 2, 80
// against 74; 9000, 0.55 of one, 40 against 34; 1024 x 1024, 6272 pixels, 0.77 of one, 73 against 86).  A last round that would be
// a third full or less, after three or more, leaves as a launch of its own, which takes the form that suits its pixels (100352 pixels,
// 6.1 rounds, 270 -> 263 us; 50176, 3.06 rounds, 152 -> 138; 75264, 0.6 of the fifth, 200 -> 202: not taken).  Layers of few chunks
// spend too much of a tile on its ends (128 x 128, 200704 pixels: 83 against 69; 256 x 256, 50176: 52 against 45).
int launch_conv1x1_wide(const sbn_packed* p, const float* x, float* y, long long M, int form, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (!p->dev.d_wt) return fail(SBN_EINVAL, "internal error: the layer has no bfloat16 triples");
    if (!form && split_pays(p, M)) form = 2032;
    if (!form) {
        const long long col_tiles = (p->c_out + 255) / 256, tiles = (M + 127) / 128 * col_tiles, cus = p->dev.cus;
        const long long rounds = (tiles + cus - 1) / cus;
        const bool fits = col_tiles * 256 * 7 <= p->c_out * 8;                        // at most an eighth of the channels past c_out
        const bool filled = rounds == 1 ? 4 * tiles >= 3 * cus : 5 * tiles >= 4 * rounds * cus;
        // whole rounds, and the pixels of a last round that would fill a third of the chip or less by themselves
        const long long slots = 8 * std::max<long long>(1, cus / 8 / col_tiles);      // pixel tiles of a round (as in launch)
        const long long whole = M / 128 / slots * slots * 128, rest = M - whole;
        if (fits && p->c_in >= 384 && whole >= 3 * 128 * slots && rest > 0 && 3 * rest <= 128 * slots) {
            if (int rc = launch<4, 8, true>(p, x, y, whole, st)) return rc;
            return launch_conv1x1(p, x + whole * p->c_in, y + whole * p->c_out, rest, stream);
        }
        form = fits && filled && p->c_in >= 384 ? 2256 : 2064;
    }
    if (form == 2032) return launch_split(p, x, y, M, st);
    return form == 2256 ? launch<4, 8, true>(p, x, y, M, st) : launch<2, 4, false>(p, x, y, M, st);
}

}  // namespace sbn
