// Group-sparse 1x1 and 3x3 convolution of few output pixels, for gfx950.
//
// A launch of few pixels is a chain of waits: descriptors, loads, LDS, barriers, each paid in full because nothing
// else runs meanwhile.  Here there are as few links as possible.  A wave multiplies 16 * PT pixels x 16 * CT output
// channels with v_mfma_f32_16x16x4_f32, whose operands are laid out so that a plain 16-byte load per lane is one:
// lane l holds pixel (or filter) l % 16, channels 4 * (l / 16) .. + 3 of 16.  Both operands go from memory
// to the registers that multiply them, without LDS, barriers or branches, and the NW waves of a workgroup take the
// units of 32 input channels (of one tap) in turn, so that most of a wave's loads are in flight at once.  The NW partial
// results meet in LDS and are added in wave order.
//
// Removed blocks are zeros that are multiplied, at the same rate as the 4x4x1 multiplies of the other 32-bit forms:
// for few pixels the matrix unit is not what bounds the time.  Pieces that no group of the bundle keeps are not
// loaded.  Results that are not finite (an infinite or NaN activation, times the zeros, reaches every output of its pixel)
// are done again over the kept blocks only.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sbn_internal.h"
#include "sbn_wide.h"

namespace {

using namespace sbn_wide;
using sbn::kNoEntry;

struct Args {
    const float* x;
    float* y;
    const float* wts;
    const uint32_t* where;            // [bundle][piece of 4 channels, up to a multiple of 8]: byte offset of its entry in wts
    const float* bias;
    const uint32_t* records;          // per 32 channels, for results that are done again
    const uint32_t* woff;
    long long M;                      // output pixels
    uint32_t wts_bytes;
    int K, N, n_bundles, n_sub, act;
    int H, W, OH, OW, stride;         // 3x3
    int n_pix_tiles, pix_fast;
};

// Four output channels ch .. ch + 3 (one filter group) of output pixel pix over the kept blocks: by one lane, or by a wave, a lane
// per piece of eight sub-chunks of 32 channels.
template <int TAPS>
struct Exact {
    const Args& a;

    __device__ __forceinline__ void store(v4f acc, long long pix, int ch) const
    {
        acc += *(const v4f*)(a.bias + ch);
        if (a.act == SBN_ACT_RELU) acc = relu4_of_any(acc);
        *(v4f*)(a.y + pix * a.N + ch) = acc;
    }
    // w: its group's [co][ci] of the entry's first tap; ch: first channel of the piece
    __device__ __forceinline__ void entry(v4f& acc, const v4f* w, long long pix, int ch) const
    {
        long long at = pix;
        int oy = 0, ox = 0;
        if constexpr (TAPS == 9) {
            ox = (int)(pix % a.OW) * a.stride;
            oy = (int)(pix / a.OW % a.OH) * a.stride;
            at = (pix / ((long long)a.OW * a.OH) * a.H + oy) * a.W + ox;
        }
#pragma unroll 1
        for (int t = 0; t < TAPS; ++t, w += 16) {
            const int dy = TAPS == 9 ? t / 3 - 1 : 0, dx = TAPS == 9 ? t % 3 - 1 : 0;
            if (TAPS == 9 && (oy + dy < 0 || oy + dy >= a.H || ox + dx < 0 || ox + dx >= a.W)) continue;
            const float* xp = a.x + (at + (long long)dy * a.W + dx) * a.K + ch;
            v4f xv;
#pragma unroll
            for (int i = 0; i < 4; ++i) xv[i] = ch + i < a.K ? xp[ch + i < a.K ? i : 0] : 0.f;
            const v4f wv[4] = {w[0], w[1], w[2], w[3]};
            add_piece(acc, wv, xv, true);
        }
    }
    __device__ __forceinline__ void by_lane(long long pix, int ch) const
    {
        const int b = ch >> 4, g = (ch >> 2) & 3;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < a.n_sub; ++c) {
            const uint32_t* r = a.records + ((size_t)b * a.n_sub + c) * 8;
            const v4f* w = (const v4f*)(a.wts + (size_t)a.woff[(size_t)b * (a.n_sub + 1) + c] * (TAPS * 64) + g * 16);
            for (int q = 0; q < 8 && r[q] != 0; ++q, w += TAPS * 16)
                if (r[q] >> g & 1u) entry(acc, w, pix, c * 32 + (int)(r[q] >> 12) * 4);
        }
        store(acc, pix, ch);
    }
    __device__ __forceinline__ void by_wave(long long pix, int ch, int lane) const
    {
        const int b = ch >> 4, g = (ch >> 2) & 3;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int c = lane >> 3; c < a.n_sub; c += 8) {
            const uint32_t r = a.records[((size_t)b * a.n_sub + c) * 8 + (lane & 7)];
            if (r >> g & 1u)
                entry(acc, (const v4f*)(a.wts + ((size_t)a.woff[(size_t)b * (a.n_sub + 1) + c] + (lane & 7)) * (TAPS * 64) + g * 16), pix,
                      c * 32 + (int)(r >> 12) * 4);
        }
        acc = sum_over_wave(acc);
        if (lane == 0) store(acc, pix, ch);
    }
};

__device__ __forceinline__ float relu(float v)                           // (as relu4)
{
    const int b = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, b > 0 ? b : 0);
}

template <int TAPS, int NW>
__global__ __launch_bounds__(64 * NW) void conv_few_kernel(Args a)
{
    // A wave's activations, [pixel][32 channels], the 16-byte slot s of pixel r at s ^ (r / 2 % 8): the 16 rows that a read serves at a time
    // and the two that a write does cover all banks.
    __shared__ __attribute__((aligned(16))) char xs[NW][2048];
    // The waves' sums in 64 bits, [pixel][channel], rows 144 bytes apart (no bank is met twice by the 16 rows that are written at a time).
    __shared__ __attribute__((aligned(16))) char red[NW][16 * 144];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, quad = lane >> 4;

    // Workgroup ids go round the eight XCDs: the tiles that share the larger operand run on one of them.
    const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;
    const int n_fast = a.pix_fast ? a.n_pix_tiles : a.n_bundles;
    const int slow = (jj / n_fast) * 8 + xcd, fast = jj % n_fast;
    const int pix_tile = a.pix_fast ? fast : slow, bundle = a.pix_fast ? slow : fast;
    if (pix_tile >= a.n_pix_tiles || bundle >= a.n_bundles) return;

    // ---- activations: a lane fetches slot lane % 8 of the rows lane / 8 and lane / 8 + 8.  1x1: the tile's rows are a buffer.  3x3: the
    // buffer starts a row and a pixel before the first image of the tile, so that the tap's shift is a scalar offset; a lane
    // whose tap lies outside the image gets an offset outside the buffer and reads zeros, as do pixels past the last
    // one and channels past c_in.
    const long long pix0 = (long long)pix_tile * 16;
    const int rows = (int)(a.M - pix0 < 16 ? a.M - pix0 : 16);
    const int slot = lane & 7;
    uint32_t xoff[2], inside[2];
    __amdgpu_buffer_rsrc_t xres;
    if constexpr (TAPS == 1) {
        xres = make_rsrc(a.x + pix0 * a.K, (uint32_t)rows * (uint32_t)a.K * 4u);
#pragma unroll
        for (int t = 0; t < 2; ++t) xoff[t] = ((uint32_t)(t * 8 + (lane >> 3)) * (uint32_t)a.K + (uint32_t)slot * 4u) * 4u;
    } else {
        const int per = a.OH * a.OW;
        const long long b0 = pix0 / per;
        const int first = (int)(pix0 - b0 * per);
        xres = make_rsrc(a.x + (b0 * a.H * a.W - a.W - 1) * a.K, 0x7FFFFFF0u);       // (only taps inside an image are read)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int r = t * 8 + (lane >> 3), p = first + r, b = p / per, q = p - b * per;
            const int oy = q / a.OW * a.stride, ox = q % a.OW * a.stride;
            xoff[t] = ((uint32_t)((b * a.H + oy) * a.W + ox) * (uint32_t)a.K + (uint32_t)slot * 4u) * 4u;
            uint32_t m = 0;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const int iy = oy + k / 3 - 1, ix = ox + k % 3 - 1;
                if (iy >= 0 && iy < a.H && ix >= 0 && ix < a.W) m |= 1u << k;
            }
            inside[t] = r < rows ? m : 0u;
        }
    }

    // ---- unit u: sub-chunk u / TAPS of 32 channels, tap u % TAPS (the taps of a sub-chunk read the same lines).  Past the last one
    // every lane's offset lies outside the buffers.
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(a.wts, a.wts_bytes);
    const int n_units = TAPS * a.n_sub;
    struct Set {
        v4f x[2], w[2];
    };
    struct Where {
        uint32_t at[8];
    };
    auto find = [&](int u, Where& e) {
        const uint32_t* p = a.where + ((size_t)bundle * a.n_sub + (u < n_units ? u : n_units - 1) / TAPS) * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) e.at[i] = p[i];
    };
    auto issue = [&](int u, const Where& e, Set& s) {
        const bool real = u < n_units;
        const int uu = real ? u : 0;
        const int c = uu / TAPS, tap = uu % TAPS;
        const uint32_t shift = TAPS == 9 ? (uint32_t)(tap / 3 * a.W + tap % 3) * (uint32_t)a.K * 4u : 0u;
        const uint32_t past = c * 32 + slot * 4 < a.K && real ? 0u : 0x80000000u;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t out = TAPS == 9 && !(inside[t] >> tap & 1u) ? 0x80000000u : past;
            s.x[t] = __builtin_bit_cast(v4f, buf_load(xres, xoff[t] + out, shift + (uint32_t)c * 128u));
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t p0 = e.at[h * 4], p1 = e.at[h * 4 + 1], p2 = e.at[h * 4 + 2], p3 = e.at[h * 4 + 3];
            const uint32_t at = quad < 2 ? (quad == 0 ? p0 : p1) : (quad == 2 ? p2 : p3);
            s.w[h] = __builtin_bit_cast(v4f, buf_load(wres, real ? at + (uint32_t)l16 * 16u : kNoEntry, (uint32_t)tap * 256u));
        }
    };

    v4f acc[4];                                    // partial sums of 32 bits
    char* const wr = xs[wave] + (lane >> 3) * 128;
    const char* const rd = xs[wave] + l16 * 128;
    auto multiply = [&](int u, Set& s) {
        if ((a.K & 3) && (u / TAPS + 1) * 32 > a.K) {                    // the last piece's channels past c_in are the next pixel's
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (u / TAPS * 32 + slot * 4 + i >= a.K) s.x[t][i] = 0.f;
        }
        // (a wave's LDS instructions are executed in order: no barrier, the compiler is kept from moving them)
        wave_lds_order();
#pragma unroll
        for (int t = 0; t < 2; ++t) *(v4f*)(wr + t * 1024 + ((slot ^ (t * 4 + (lane >> 4))) & 7) * 16) = s.x[t];
        wave_lds_order();
        v4f xv[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) xv[h] = *(const v4f*)(rd + (((h * 4 + quad) ^ (l16 >> 1)) & 7) * 16);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.w[h][j], xv[h][j], acc[j], 0, 0, 0);
    };

    // ---- the wave's units, two at a time; the loads of the next one and the places of the one after it are in flight meanwhile
    Set s0, s1;
    Where e0, e1;
    find(wave, e0);
    find(wave + NW, e1);
    // (asked for early) thread t adds up pixel t / 16, channel t % 16
    const float bias = a.bias[bundle * 16 + l16];
    issue(wave, e0, s0);
    find(wave + 2 * NW, e0);
    // 32-bit sums run over at most two units, 16 products each; everything after that is added in 64 bits and rounded once
    double sum[4] = {0., 0., 0., 0.};
    for (int u = wave; u < n_units; u += 2 * NW) {
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[n] = (v4f){0.f, 0.f, 0.f, 0.f};
        issue(u + NW, e1, s1);
        find(u + 3 * NW, e1);
        multiply(u, s0);
        issue(u + 2 * NW, e0, s0);
        find(u + 4 * NW, e0);
        if (u + NW < n_units) multiply(u + NW, s1);
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] += (double)acc[n][i];
    }

    // ---- the waves' sums, bias, activation, store
    typedef double v2d __attribute__((ext_vector_type(2)));
    *(v2d*)(red[wave] + l16 * 144 + quad * 32) = (v2d){sum[0], sum[1]};
    *(v2d*)(red[wave] + l16 * 144 + quad * 32 + 16) = (v2d){sum[2], sum[3]};
    __syncthreads();
    const __amdgpu_buffer_rsrc_t yres = make_rsrc(a.y + pix0 * a.N, (uint32_t)rows * (uint32_t)a.N * 4u);
    constexpr int PER = NW >= 4 ? 1 : 4 / NW;      // quarters (four pixels) of the tile per wave
    const int ch = bundle * 16 + l16;
    uint32_t redo = 0;                             // bit k: this lane's and the next three channels are to be done again
    if (wave >= 4) return;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int row = (k * NW + wave) * 4 + quad;
        double s = (double)bias;
#pragma unroll
        for (int n = 0; n < NW; ++n) s += *(const double*)(red[n] + row * 144 + l16 * 8);
        float o = (float)s;
        const unsigned long long bad = __builtin_amdgcn_ballot_w64(!(o - o == 0.f) && row < rows && ch < a.N);
        if ((bad >> (lane & 60) & 15u) != 0 && (lane & 3) == 0) redo |= 1u << k;
        if (a.act == SBN_ACT_RELU) o = relu(o);
        const uint32_t off = ch < a.N ? ((uint32_t)row * (uint32_t)a.N + (uint32_t)ch) * 4u : 0xFFFFFFF0u;
        __builtin_amdgcn_raw_buffer_store_b32(as_uint(o), yres, (int)off, 0, 0);
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(redo != 0) != 0, 0)) {
        const Exact<TAPS> exact = {a};
        auto pixel = [&](int k, int ln) { return pix0 + (k * NW + wave) * 4 + (ln >> 4); };
        auto channel = [&](int, int ln) { return bundle * 16 + (ln & 15); };
        do_again(redo, PER, [&](int k, int ln) { exact.by_wave(pixel(k, ln), channel(k, ln), lane); },
                 [&](int k) { exact.by_lane(pixel(k, lane), channel(k, lane)); });
    }
}

template <int TAPS, int NW>
int launch(const sbn_packed* p, const float* x, float* y, int n, int h, int w, hipStream_t st)
{
    const sbn::DeviceLayout& L = p->dev;
    Args a;
    a.x = x, a.y = y, a.wts = L.d_wts, a.where = L.d_where, a.bias = L.d_bias, a.records = L.d_records32, a.woff = L.d_woff32;
    a.H = h, a.W = w, a.stride = p->stride;
    a.OH = (h - 1) / p->stride + 1, a.OW = (w - 1) / p->stride + 1;
    a.M = (long long)n * a.OH * a.OW;
    a.wts_bytes = (uint32_t)(L.wts.size() * sizeof(float)) + TAPS * 256u;      // (the array has slack behind it)
    a.K = p->c_in, a.N = p->c_out, a.n_bundles = L.n_bundles, a.n_sub = L.n_chunks32, a.act = p->act;
    const long long pix_tiles = (a.M + 15) / 16;
    // The weights are the larger operand of layers of more bundles than pixel tiles (49 pixels, 1024 x 1024: 4.6 us, the other way
    // 8.2), but need enough bundles for eight XCDs (12544 pixels, 32 x 64: 8.3, the other way 5.3).
    a.pix_fast = L.n_bundles >= 16 && L.n_bundles >= pix_tiles;
    const long long slow = a.pix_fast ? L.n_bundles : pix_tiles, fast = a.pix_fast ? pix_tiles : L.n_bundles;
    const long long grid = (slow + 7) / 8 * 8 * fast;
    if (grid > 0x7FFFFFFFll) return sbn::fail(SBN_EINVAL, "too many output pixels for one launch (%lld)", a.M);
    a.n_pix_tiles = (int)pix_tiles;
    hipLaunchKernelGGL((conv_few_kernel<TAPS, NW>), dim3((unsigned)grid), dim3(64 * NW), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sbn::fail(SBN_EHIP, "few-pixel launch: %s", hipGetErrorString(e));
    return SBN_OK;
}

}  // namespace

namespace sbn {

// What the kernel's 32-bit offsets reach: the weights, and in 3x3 layers the images that a tile of 16 pixels spans.
bool few_takes(const sbn_packed* p, int n, int h, int w)
{
    if (p->dev.wts.size() * sizeof(float) >= 0xFFF00000ull) return false;
    if (p->kind == SBN_CONV1X1) return (long long)n * h * w <= 0x7FFFFFFFll;
    const long long oh = (h - 1) / p->stride + 1, ow = (w - 1) / p->stride + 1, images = 15 / (oh * ow) + 2;
    return (images * h + 2) * w + 3 <= 0x7FFFFF00ll / 4 / p->c_in;
}

// Waves per workgroup, 0: the launch is not one of few pixels.  All 250 to 600 random layers per kind that the lines were drawn from: 1 to
// 5000 pixels, 16 to 1024 channels (3x3: to 512), sparsity 0 to 90 %, four sets of buffers in turn, launches back to back; us
// of the form that is chosen otherwise against this one:
//   1x1, 30 %   196 pixels, 64 x 128  4.3 / 2.7    784, 128 x 256  5.9 / 3.5    196, 512 x 512    5.8 / 4.3
//               49, 1024 x 1024       8.1 / 4.6    1, 1024 x 1000  8.0 / 4.3    1100, 512 x 512   12.2 / 12.2  (2208 tiles: not taken)
//   3x3, 50 %   3 x 9 x 9, 256 x 200 23.5 / 9.0    1 x 28 x 28, 128 x 128  14.3 / 8.9   1 x 7 x 7, 512 x 512  41.5 / 13.7
//               3 x 45 x 45, 64 x 128, stride 2  14.4 / 9.3                     8 x 14 x 14, 256 x 256  24.7 / 34.3 (1568 tiles: not taken)
// (mean gain over the layers taken: 1x1 1.45, 3x3 1.8, 3x3 of stride 2, which the other kernel takes singly buffered, 2.5 times; 2 of 820 lose more than 3 %, at most 7 %).  Both limits shrink with what the
// layer keeps, which the other forms' time follows and this one's does not.  As many waves as leave the chip about one round of
// workgroups (tiles per compute unit up to 1: eight, up to 6: four).  Relative error (2-norm, units of 1e-8): 3 to 5.5, the forms replaced 4 to 22.
static int few_waves(const sbn_packed* p, long long m)
{
    const int taps = p->kh * p->kw, cus = p->dev.cus;
    const long long tiles = (m + 15) / 16 * p->dev.n_bundles, units = (long long)taps * p->dev.n_chunks32;
    const double kept = 16.0 * (double)p->dev.n_present / ((double)p->c_in * p->c_out);
    const double left = taps == 1 ? 0.4 + 0.6 * kept : 0.2 + 0.8 * kept;
    if ((double)tiles > (taps == 1 ? 6.0 : p->stride == 1 ? 4.7 : 7.8) * cus * left || (double)(tiles * units) > (taps == 1 ? 120.0 : 470.0) * cus * left) return 0;
    if (taps == 9 && units >= 64 && 4 * tiles <= cus) return 16;
    return tiles <= cus ? 8 : 4;
}

bool few_chosen(const sbn_packed* p, int n, int h, int w)
{
    return few_waves(p, (long long)n * ((h - 1) / p->stride + 1) * ((w - 1) / p->stride + 1)) != 0 && few_takes(p, n, h, w);
}

int launch_few(const sbn_packed* p, const float* x, float* y, int n, int h, int w, int form, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    const int waves = form ? form - 3000 : few_waves(p, (long long)n * ((h - 1) / p->stride + 1) * ((w - 1) / p->stride + 1));
    if (p->kind == SBN_CONV1X1) return waves == 8 ? launch<1, 8>(p, x, y, n, h, w, st) : launch<1, 4>(p, x, y, n, h, w, st);
    return waves == 16 ? launch<9, 16>(p, x, y, n, h, w, st) : waves == 8 ? launch<9, 8>(p, x, y, n, h, w, st) : launch<9, 4>(p, x, y, n, h, w, st);
}

}  // namespace sbn
