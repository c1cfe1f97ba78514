// Kernel-level group-sparse 3x3 convolution, stride 1, on triples of bfloat16, for gfx950.
//
// The arithmetic is that of sbn_conv1x1_wide.hip (operands a + b + c exactly, six v_mfma_f32_32x32x16_bf16 per
// product, sums in 32-bit floats, 32-bit multiply-adds for what bfloat16 cannot hold): one step per 16
// channels and tap, over blocks filled up with the removed kernels' zeros.
//
// Mapping.  Output pixels are numbered through the images (image, row, column); a workgroup owns
// T = 64 * U consecutive ones x 64 output channels, so no lane multiplies padding whatever the extents.  With
// stride 1 the tap (ky, kx) of pixel p is pixel p + (ky - 1) * W + kx - 1 of the same numbering, so the
// tile's input is one run of T + 2 * W + 2 pixels.  Per 32 channels it goes global -> registers -> triples ->
// LDS, once for all nine taps; a lane whose tap lies outside the image reads a row of zeros instead (nine
// bits per pixel, worked out once).
//
// Three forms (launch_conv3x3_wide has the rule): U = 2, a wave 64 pixels x 32 channels; U = 1, a wave 32 x 32, for
// launches of few tiles; and the same with S = 2 slices of waves that share the input channels.
//
// Relative error (2-norm, units of 1e-8), 14 x 14 x 256 at 70 % and 50 % sparsity, 7 x 7 x 512 at 70 %, 57 x 57 x 64 at 50 %: 9.1, 9.9,
// 9.3, 6.2; the 32-bit form shows 12 to 25.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sbn_internal.h"
#include "sbn_wide.h"

namespace {

using namespace sbn_wide;

constexpr int KC = 32;                    // channels staged at a time
constexpr int STEPS = 18;                 // nine taps of two halves of 16 channels

// Four output channels ch .. ch + 3 (one filter group) of pixel pix by 32-bit multiply-adds over the kept kernels: by one
// lane, a row of taps' loads at a time, or by a wave, a lane per piece of eight sub-chunks.
struct Exact {
    const float* __restrict__ x;
    float* __restrict__ y;
    const uint32_t* __restrict__ records;
    const uint32_t* __restrict__ woff;
    const float* __restrict__ wts;
    const float* __restrict__ bias;
    int H, W, K, N, n_sub, act;

    __device__ __forceinline__ void store(v4f acc, long long pix, int ch) const
    {
        acc += *(const v4f*)(bias + ch);
        if (act == SBN_ACT_RELU) acc = relu4_of_any(acc);
        *(v4f*)(y + pix * N + ch) = acc;
    }
    // one entry: w = its group's [tap][co][ci], xp = its piece of the centre pixel
    __device__ __forceinline__ void entry(v4f& acc, const v4f* w, const float* xp, int ox, int oy) const
    {
#pragma unroll 1
        for (int dy = -1; dy <= 1; ++dy, w += 48) {
            if (oy + dy < 0 || oy + dy >= H) continue;
            v4f xv[3], wv[3][4];
            bool in[3];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                in[u] = ox + u - 1 >= 0 && ox + u - 1 < W;
                xv[u] = *(const v4f*)(xp + ((long long)dy * W + (in[u] ? u - 1 : 0)) * K);
#pragma unroll
                for (int co = 0; co < 4; ++co) wv[u][co] = w[u * 16 + co];
            }
#pragma unroll
            for (int u = 0; u < 3; ++u) add_piece(acc, wv[u], xv[u], in[u]);
        }
    }
    __device__ __forceinline__ void by_lane(int pix, int ch) const
    {
        const int b = ch >> 4, g = (ch >> 2) & 3, ox = pix % W, oy = pix / W % H;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < n_sub; ++c) {
            const uint32_t* r = records + ((size_t)b * n_sub + c) * 8;
            const v4f* w = (const v4f*)(wts + (size_t)woff[(size_t)b * (n_sub + 1) + c] * 576 + g * 16);
            for (int q = 0; q < 8 && r[q] != 0; ++q, w += 144)
                if (r[q] >> g & 1u) entry(acc, w, x + (long long)pix * K + c * KC + (int)(r[q] >> 12) * 4, ox, oy);
        }
        store(acc, pix, ch);
    }
    __device__ __forceinline__ void by_wave(int pix, int ch, int lane) const
    {
        const int b = ch >> 4, g = (ch >> 2) & 3, ox = pix % W, oy = pix / W % H;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int c = lane >> 3; c < n_sub; c += 8) {
            const uint32_t r = records[((size_t)b * n_sub + c) * 8 + (lane & 7)];
            if (r >> g & 1u)
                entry(acc, (const v4f*)(wts + ((size_t)woff[(size_t)b * (n_sub + 1) + c] + (lane & 7)) * 576 + g * 16),
                      x + (long long)pix * K + c * KC + (int)(r >> 12) * 4, ox, oy);
        }
        acc = sum_over_wave(acc);
        if (lane == 0) store(acc, pix, ch);
    }
};

// U: 32-pixel tiles of a wave.  NL: staged 16-byte slots per lane; NL * 32 >= T + 2 * W + 2 pixels.
// S: slices of four waves; slice s multiplies the sub-chunks s, s + S, ... out of its own image, and the sums meet at the end.
template <int U, int NL, int S>
__global__ __launch_bounds__(256 * S, 2) void conv3x3_wide_kernel(
    const float* __restrict__ x, float* __restrict__ y, const uint16_t* __restrict__ wt, uint32_t wt_bytes,
    const float* __restrict__ bias, const uint32_t* __restrict__ records, const uint32_t* __restrict__ woff,
    const float* __restrict__ wts, int M, int H, int W, int K, int N, int n_bundles, int n_sub, int n_col_tiles, int n_pix_tiles,
    float tiny_sum, int act)
{
    constexpr int T = 64 * U;
    // LDS image, a, b and c alike: per 8 channels a plane of one 16-byte row per pixel, a row of zeros at its end, and 64
    // bytes between the planes' banks, so that the 4 rows x 4 planes that half a wave stages at a time do not meet in a bank.
    constexpr int ROWS = NL * 32, PLANE = (ROWS + 4) * 16, PART = 4 * PLANE;
    static_assert(3 * PART >= 4 * U * 4096 || S == 1, "the slices' sums fit one image");
    __shared__ __attribute__((aligned(16))) char lds_all[S][3 * PART];
    __shared__ uint8_t tiny_row[ROWS];             // 1: the staged pixel holds a non-zero activation below 2^-100

    const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;                // column tiles of one pixel tile on one XCD
    const int pix_tile = (jj / n_col_tiles) * 8 + xcd, col_tile = jj % n_col_tiles;
    if (pix_tile >= n_pix_tiles) return;
    const int tid = threadIdx.x & 255, lane = tid & 63;                  // thread of the slice
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slice = S == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    char* const lds = lds_all[slice];
    const int first = (wave & 1) * 32 * U;                               // the wave's first pixel of the tile
    const int pair = col_tile * 2 + (wave >> 1);                         // 32 channels, two bundles
    const bool active = pair * 2 < n_bundles;
    const int p0 = pix_tile * T, q0 = p0 - W - 1;                        // first output pixel, first staged one
    const int rows_valid = M - p0 < T ? M - p0 : T;

    // ---- this lane's pixels: LDS offset of the top left tap, and which taps lie inside the image
    int at[U];
    uint32_t inside[U];
#pragma unroll
    for (int t = 0; t < U; ++t) {
        const int l = first + t * 32 + (lane & 31), p = p0 + l;
        const int ox = p % W, oy = p / W % H;
        uint32_t m = 0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int iy = oy + k / 3 - 1, ix = ox + k % 3 - 1;
            if (iy >= 0 && iy < H && ix >= 0 && ix < W) m |= 1u << k;
        }
        inside[t] = p < M ? m : 0u;
        at[t] = (lane >> 5) * PLANE + l * 16;
    }
    const int zero_at = (lane >> 5) * PLANE + ROWS * 16;
    if (tid < 48) *(uint32_t*)(lds + (tid >> 2) * PLANE + ROWS * 16 + (tid & 3) * 4) = 0u;
    for (int i = threadIdx.x; i < ROWS; i += 256 * S) tiny_row[i] = 0;

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
    char* const wr = lds + (quad >> 1) * PLANE + (tid >> 3) * 16 + (quad & 1) * 8;

    // ---- weights: three fragments (a, b, c) per step, step = 18 * sub-chunk + 2 * tap + half
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(wt, wt_bytes);
    const int n_steps = n_sub * STEPS;
    const uint32_t w0 = (uint32_t)(active ? pair : 0) * (uint32_t)n_steps * 3072u;
    auto load_w = [&](int step, v8b (&w)[3]) {
        step = step < n_steps ? step : 0;                                // (past the end: multiplied with zeros)
#pragma unroll
        for (int s = 0; s < 3; ++s) w[s] = __builtin_bit_cast(v8b, buf_load(wres, (uint32_t)lane * 16u + s * 1024u, w0 + (uint32_t)step * 3072u));
    };

    // `main` runs over one row of taps only (six steps) and is then added to `total`: a sum of 9 * c_in / 16 steps would be
    // rounded more often than the 32-bit form's partial sums.
    v16f total[U], main[U], cross[U];
#pragma unroll
    for (int t = 0; t < U; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) total[t][i] = main[t][i] = cross[t][i] = 0.f;

    v8b w[3][3], fa[U], fb[U], fc[U];
    issue_x(slice);
    load_w(slice * STEPS, w[0]);
    load_w(slice * STEPS + 1, w[1]);
    // (every slice goes through the same number of barriers; past the last sub-chunk it stages zeros)
    for (int c = slice; c - slice < n_sub; c += S) {
        __syncthreads();                           // everyone has finished with the last sub-chunk's image
        uint32_t least = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            least = least_magnitude(stage[i], least);
            split4_to(wr + i * 512, PART, stage[i]);
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(least < kTiny) != 0, 0)) {
#pragma unroll
            for (int i = 0; i < NL; ++i)
                if (least_magnitude(stage[i], 0xFFFFFFFFu) < kTiny) tiny_row[i * 32 + (tid >> 3)] = 1;
        }
        __syncthreads();
        // (opaque: the addresses of a sub-chunk's reads are cheaper to work out again than to keep in registers)
#pragma unroll
        for (int t = 0; t < U; ++t) asm volatile("" : "+v"(at[t]), "+v"(inside[t]));
        // the addresses of tap k, one per tile, for both halves and all parts
        int rd[U];
        auto aim = [&](int k) {
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int in = (int)(inside[t] << (31 - k)) >> 31;       // all ones if the tap is inside
                rd[t] = ((at[t] + (k / 3 * W + k % 3) * 16) & in) | (zero_at & ~in);
            }
        };
        auto read = [&](int half, int part, v8b (&to)[U]) {
#pragma unroll
            for (int t = 0; t < U; ++t) to[t] = *(const v8b*)(lds + rd[t] + half * (2 * PLANE) + part * PART);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto mul = [&](const v8b& wp, const v8b (&xp)[U], v16f (&sum)[U]) {
#pragma unroll
            for (int t = 0; t < U; ++t) sum[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wp, xp[t], sum[t], 0, 0, 0);
        };
        aim(0);
        read(0, 2, fc);
        read(0, 0, fa);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const v8b(&wi)[3] = w[i % 3];
            load_w(i + 2 < STEPS ? c * STEPS + i + 2 : (c + S) * STEPS + i + 2 - STEPS, w[(i + 2) % 3]);
            if (i == 2) issue_x(c + S);
            __builtin_amdgcn_sched_barrier(0);
            read(i % 2, 1, fb);
            mul(wi[0], fc, cross);
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < STEPS) {
                if (i % 2) aim((i + 1) / 2);       // (fb of this step has been asked for)
                read((i + 1) % 2, 2, fc);
            }
            mul(wi[2], fa, cross);
            mul(wi[0], fa, main);
            mul(wi[1], fa, cross);
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < STEPS) read((i + 1) % 2, 0, fa);
            mul(wi[1], fb, cross);
            mul(wi[0], fb, cross);
            __builtin_amdgcn_sched_barrier(0);
            if (i % 6 == 5) {
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    total[t] += main[t];
#pragma unroll
                    for (int k = 0; k < 16; ++k) main[t][k] = 0.f;
                }
            }
        }
    }

    // ---- total + cross of all slices
#pragma unroll
    for (int t = 0; t < U; ++t) total[t] += cross[t];
    if constexpr (S > 1) {
        __syncthreads();                           // images are dead
        if (slice > 0) {
#pragma unroll
            for (int t = 0; t < U; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *(v4f*)(lds + ((wave * U + t) * 4 + g) * 1024 + lane * 16) = (v4f){total[t][4 * g], total[t][4 * g + 1], total[t][4 * g + 2], total[t][4 * g + 3]};
        }
        __syncthreads();
        if (slice > 0) return;
#pragma unroll
        for (int s = 1; s < S; ++s)
#pragma unroll
            for (int t = 0; t < U; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4f o = *(const v4f*)(lds_all[s] + ((wave * U + t) * 4 + g) * 1024 + lane * 16);
#pragma unroll
                    for (int i = 0; i < 4; ++i) total[t][4 * g + i] += o[i];
                }
    }
    if (!active) return;

    // ---- bias, activation, store.  (tiny_row: the last writes lie before the last sub-chunk's second barrier)
    const __amdgpu_buffer_rsrc_t yres = make_rsrc(y + (long long)p0 * N, (uint32_t)rows_valid * (uint32_t)N * 4u);
    const __amdgpu_buffer_rsrc_t bres = make_rsrc(bias, (uint32_t)n_bundles * 64u);
    const int ch_lane = pair * 32 + (lane >> 5) * 4;                     // + 8 * g
    uint32_t marked = 0;                           // bit t: a tap of the pixel of tile t reads tiny values
#pragma unroll
    for (int t = 0; t < U; ++t)
#pragma unroll
        for (int k = 0; k < 9; ++k)
            if ((inside[t] >> k & 1u) && tiny_row[first + t * 32 + (lane & 31) + k / 3 * W + k % 3]) marked |= 1u << t;
    uint32_t redo = 0;                             // bit 4 * t + g: to be done again
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const v4f bg = __builtin_bit_cast(v4f, buf_load(bres, (uint32_t)(ch_lane + 8 * g) * 4u, 0));
#pragma unroll
        for (int t = 0; t < U; ++t) {
            bool bad = false;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float s = total[t][4 * g + i];
                const float o = s + bg[i];
                bad |= o - o != 0.f || magnitude(s) < kTiny || ((marked >> t & 1u) && __builtin_fabsf(s) < tiny_sum);
                total[t][4 * g + i] = o;
            }
            if (bad && first + t * 32 + (lane & 31) < rows_valid && ch_lane + 8 * g < N) redo |= 1u << (4 * t + g);
        }
    }
#pragma unroll
    for (int t = 0; t < U; ++t) store_tile<0>(total[t], yres, first + t * 32, pair * 32, N, act == SBN_ACT_RELU, lane);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(redo != 0) != 0, 0)) {
        const Exact exact = {x, y, records, woff, wts, bias, H, W, K, N, n_sub, act};
        auto pixel = [&](int k, int ln) { return p0 + first + (k >> 2) * 32 + (ln & 31); };
        auto channel = [&](int k, int ln) { return pair * 32 + (ln >> 5) * 4 + 8 * (k & 3); };
        do_again(redo, 4 * U, [&](int k, int ln) { exact.by_wave(pixel(k, ln), channel(k, ln), lane); },
                 [&](int k) { exact.by_lane(pixel(k, lane), channel(k, lane)); });
    }
}

template <int U, int NL, int S>
int launch(const sbn_packed* p, const float* x, float* y, int n, int h, int w, hipStream_t st)
{
    const sbn::DeviceLayout& L = p->dev;
    const long long M = (long long)n * h * w;
    constexpr int T = 64 * U;
    const long long n_pix_tiles = (M + T - 1) / T;
    const int n_col_tiles = (L.n_bundles + 3) / 4;
    const long long grid = ((n_pix_tiles + 7) / 8) * 8 * n_col_tiles;
    if (T + 2 * w + 2 > NL * 32) return sbn::fail(SBN_EINVAL, "internal error: the tile's rows do not fit the staged image");
    if (grid > 0x7FFFFFFFll) return sbn::fail(SBN_EINVAL, "too many output tiles for one launch (%lld)", n_pix_tiles);
    // as in the 1x1 kernel, 9 * c_in terms
    const float tiny_sum = std::max(9.0f * (float)p->c_in * L.w_top * 0x1p-101f, 0x1p-100f);
    hipLaunchKernelGGL((conv3x3_wide_kernel<U, NL, S>), dim3((unsigned)grid), dim3(256 * S), 0, st, x, y, L.d_wt,
                       (uint32_t)(L.wt.size() * sizeof(uint16_t)), L.d_bias, L.d_records32, L.d_woff32, L.d_wts, (int)M, h, w, p->c_in,
                       p->c_out, L.n_bundles, L.n_chunks32, n_col_tiles, (int)n_pix_tiles, tiny_sum, p->act);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sbn::fail(SBN_EHIP, "conv3x3 launch: %s", hipGetErrorString(e));
    return SBN_OK;
}

// the smallest staged image that holds a tile and its halo
template <int U, int S>
int launch_fit(const sbn_packed* p, const float* x, float* y, int n, int h, int w, hipStream_t st)
{
    const int rows = 64 * U + 2 * w + 2;
    if (rows <= 160) return launch<U, 5, S>(p, x, y, n, h, w, st);
    if (rows <= 256) return launch<U, 8, S>(p, x, y, n, h, w, st);
    return launch<U, 12, S>(p, x, y, n, h, w, st);
}

}  // namespace

namespace sbn {

static long long tiles_128(const sbn_packed* p, int n, int h, int w) { return ((long long)n * h * w + 127) / 128 * ((p->dev.n_bundles + 3) / 4); }

// Launches of at most one 128 x 64 tile per compute unit wait more than they multiply, in either form; in larger ones
// layers of few channels have more of a tile's ends to pay for.  Images of fewer than four rows or columns reach few of
// the taps, which the 32-bit form does not multiply.
bool conv3x3_wide_chosen(const sbn_packed* p, int n, int h, int w)
{
    if (!conv3x3_wide_takes(p, n, h, w) || !conv3x3_wide_pays(p)) return false;
    return tiles_128(p, n, h, w) <= p->dev.cus || conv3x3_share_kept(p) >= 0.34 + 6.0 / p->c_in;
}

// Width: the largest tile's rows, 128 + 2 * w + 2, fit 384 staged ones.
bool conv3x3_wide_takes(const sbn_packed* p, int n, int h, int w)
{
    return p->dev.d_wt && p->stride == 1 && w <= 127 && w >= 4 && h >= 4 && (long long)n * h * w <= 0x70000000ll;
}

// form 0: 128 x 64 tiles from one per compute unit on (32 x 28 x 28 x 128: 47 us, 64 x 64 tiles 49; 0.77 per compute unit,
// 32 x 14 x 14 x 256: 49 against 47), two slices up to one 64 x 64 tile per compute unit (32 x 7 x 7 x 512: 47 us, one slice 57; 1.5
// per compute unit, 12 x 20 x 20, 96 x 320: 28 against 22).
int launch_conv3x3_wide(const sbn_packed* p, const float* x, float* y, int n, int h, int w, int form, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (!form) {
        const long long tiles_64 = ((long long)n * h * w + 63) / 64 * ((p->dev.n_bundles + 3) / 4), cus = p->dev.cus;
        form = tiles_128(p, n, h, w) >= cus ? 2128 : tiles_64 <= cus ? 2065 : 2064;
    }
    if (form == 2064) return launch_fit<1, 1>(p, x, y, n, h, w, st);
    if (form == 2065) return launch_fit<1, 2>(p, x, y, n, h, w, st);
    return launch_fit<2, 1>(p, x, y, n, h, w, st);
}

}  // namespace sbn
