// Small dense helper kernels: device copy (counter calibration / HBM rate),
// dense depthwise 3x3 + bias + activation and global average pool, which sit
// between the sparse pointwise layers when a whole network is chained.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sbn_internal.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void copy_kernel(const v4f* __restrict__ src, v4f* __restrict__ dst, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

// Dense depthwise 3x3, pad 1.  One thread: 4 channels of R vertically adjacent output pixels;
// the input rows slide through registers so that every loaded row serves up to three outputs,
// and the nine weight vectors are loaded once per thread.  Consecutive threads take consecutive
// channel quads, then consecutive columns: all loads and stores are 16-byte and coalesced.
// x [n][h][w][c], wt [9][c], y [n][oh][ow][c].
//
// Bound by memory only if the vector unit has nothing but the multiply-adds to do.  So a block covers
// part of ONE strip of rows: image, strip and rows are scalars, a row of the input is a buffer whose base is a
// scalar and which is empty when the row lies outside the image, a lane's three column offsets are worked out once
// and lead outside the buffer where the column does.  (With a pixel per thread decoded by three 64-bit
// divisions and a select per load, the 14 x 14 x 512 layer at batch 64 took 17.2 us, 3.0 TB/s;
// so 15.6.)
template <int STRIDE, int R>
__global__ __launch_bounds__(256) void dw3x3_kernel(const float* __restrict__ x, float* __restrict__ y,
                                                   const float* __restrict__ wt, const float* __restrict__ bias,
                                                   int h, int w, int c, int oh, int ow, int act, unsigned strips,
                                                   unsigned blocks_per_strip, unsigned blocks_per_image, unsigned eights)
{
    // Workgroup ids go round the eight XCDs.  Of every eight images each XCD gets one whole, so that the rows and columns
    // that its blocks share are read from its L2; images past the last eight (block `eights` on) are spread block by
    // block.  (MobileNet-v1, 70 %, us, in plain order, with one run of images per XCD, and so: 64 images of 224 x 224 721, 708, 703;
    // 32 of 224 x 224 453, 457, 446; 64 of 128 x 128 349, 373, 332 -- the runs then begin at a power of two from each other.)
    unsigned id = blockIdx.x;
    if (id < eights) id = ((id >> 3) / blocks_per_image * 8u + (id & 7u)) * blocks_per_image + (id >> 3) % blocks_per_image;
    const unsigned row_block = id / blocks_per_strip, ib = id % blocks_per_strip;
    const unsigned c4n = (unsigned)c >> 2;
    const unsigned i0 = ib * blockDim.x, i = i0 + threadIdx.x;            // position in the row of ow * c / 4 quads
    const int ox0 = (int)(i0 / c4n), ox = (int)(i / c4n);
    const unsigned c4 = i % c4n * 4u;
    const int oy0 = (int)(row_block % strips) * R;
    const long long b = row_block / strips;
    const bool live = ox < ow;

    auto rsrc = [](const float* base, bool valid) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, valid ? 0x7FFFFFFF : 0, 0x00020000);
    };
    auto load = [](__amdgpu_buffer_rsrc_t r, unsigned off) {
        return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
    };
    v4f wv[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) wv[k] = load(rsrc(wt + (long long)k * c, true), c4 * 4u);
    const v4f bv = load(rsrc(bias, true), c4 * 4u);
    v4f acc[R];
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i] = bv;

    // offsets from the column left of the block's first output column (a block spans few columns: 31 bits do)
    unsigned off[3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
        const int ix = ox * STRIDE - 1 + kx;
        off[kx] = live && ix >= 0 && ix < w ? ((unsigned)((ox - ox0) * STRIDE + kx) * (unsigned)c + c4) * 4u : 0x80000000u;
    }
    constexpr int ROWS = (R - 1) * STRIDE + 3;              // input rows touched by the strip
    const int iy0 = oy0 * STRIDE - 1;
#pragma unroll
    for (int ir = 0; ir < ROWS; ++ir) {
        const int iy = iy0 + ir;
        const __amdgpu_buffer_rsrc_t xr = rsrc(x + ((b * h + iy) * w + (long long)ox0 * STRIDE - 1) * c, iy >= 0 && iy < h);
        v4f row[3];
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) row[kx] = load(xr, off[kx]);
        // input row ir is tap row ky of output i when ir == i*STRIDE + ky
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int ky = ir - i * STRIDE;
            if (ky >= 0 && ky < 3) {
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) acc[i] += row[kx] * wv[ky * 3 + kx];
            }
        }
    }
    if (!live) return;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int oy = oy0 + i;
        if (oy >= oh) break;
        v4f o = acc[i];
        if (act == SBN_ACT_RELU) {
            o.x = fmaxf(o.x, 0.f);
            o.y = fmaxf(o.y, 0.f);
            o.z = fmaxf(o.z, 0.f);
            o.w = fmaxf(o.w, 0.f);
        }
        *(v4f*)(y + ((b * oh + oy) * ow + ox) * c + c4) = o;
    }
}

// The same for rows of few channel quads, of which half a wave or less would find work in one strip: threads take quads,
// columns, strips and images in one row of numbers.
template <int STRIDE, int R>
__global__ __launch_bounds__(256) void dw3x3_narrow_kernel(const float* __restrict__ x, float* __restrict__ y,
                                                          const float* __restrict__ wt, const float* __restrict__ bias,
                                                          int h, int w, int c, int oh, int ow, int act, long long total)
{
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= total) return;
    const int c4n = c >> 2;
    const int c4 = (int)(t % c4n) * 4;
    long long r = t / c4n;
    const int ox = (int)(r % ow);
    r /= ow;
    const int strips = (oh + R - 1) / R;
    const int oy0 = (int)(r % strips) * R;
    const long long b = r / strips;

    v4f wv[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) wv[k] = *(const v4f*)(wt + k * c + c4);
    const v4f bv = *(const v4f*)(bias + c4);
    v4f acc[R];
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i] = bv;

    constexpr int ROWS = (R - 1) * STRIDE + 3;              // input rows touched by the strip
    const int iy0 = oy0 * STRIDE - 1, ix0 = ox * STRIDE - 1;
    const float* xb = x + b * h * w * c + c4;
#pragma unroll
    for (int ir = 0; ir < ROWS; ++ir) {
        const int iy = iy0 + ir;
        v4f row[3];
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const int ix = ix0 + kx;
            const bool ok = iy >= 0 && iy < h && ix >= 0 && ix < w;
            const v4f v = *(const v4f*)(xb + ((long long)(ok ? iy : 0) * w + (ok ? ix : 0)) * c);
            row[kx] = ok ? v : (v4f){0.f, 0.f, 0.f, 0.f};
        }
        // input row ir is tap row ky of output i when ir == i*STRIDE + ky
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int ky = ir - i * STRIDE;
            if (ky >= 0 && ky < 3) {
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) acc[i] += row[kx] * wv[ky * 3 + kx];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int oy = oy0 + i;
        if (oy >= oh) break;
        v4f o = acc[i];
        if (act == SBN_ACT_RELU) {
            o.x = fmaxf(o.x, 0.f);
            o.y = fmaxf(o.y, 0.f);
            o.z = fmaxf(o.z, 0.f);
            o.w = fmaxf(o.w, 0.f);
        }
        *(v4f*)(y + ((b * oh + oy) * (long long)ow + ox) * c + c4) = o;
    }
}

// Dense 3x3 convolution of a few input channels (network stem), pad 1.  One thread: 4 output
// channels of one output pixel; the (c_out x 9 x c_in) weights sit in LDS as [tap][ci][c_out].
// x [n][h][w][c_in], y [n][oh][ow][c_out].
__global__ __launch_bounds__(256) void stem3x3_kernel(const float* __restrict__ x, float* __restrict__ y,
                                                     const float* __restrict__ wt, const float* __restrict__ bias,
                                                     int h, int w, int c_in, int c_out, int oh, int ow, int stride,
                                                     int act, long long total)
{
    __shared__ __attribute__((aligned(16))) float ws[9 * 4 * 64];
    for (int i = threadIdx.x; i < 9 * c_in * c_out; i += 256) ws[i] = wt[i];
    __syncthreads();
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= total) return;
    const int c4n = c_out >> 2;
    const int co = (int)(t % c4n) * 4;
    long long pix = t / c4n;
    const int ox = (int)(pix % ow);
    pix /= ow;
    const int oy = (int)(pix % oh);
    const long long b = pix / oh;
    v4f acc = *(const v4f*)(bias + co);
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
        const int iy = oy * stride + ky - 1;
        if (iy < 0 || iy >= h) continue;
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const int ix = ox * stride + kx - 1;
            if (ix < 0 || ix >= w) continue;
            const float* xp = x + ((b * h + iy) * w + ix) * c_in;
            for (int ci = 0; ci < c_in; ++ci)
                acc += xp[ci] * *(const v4f*)(ws + ((ky * 3 + kx) * c_in + ci) * c_out + co);
        }
    }
    if (act == SBN_ACT_RELU) {
        acc.x = fmaxf(acc.x, 0.f);
        acc.y = fmaxf(acc.y, 0.f);
        acc.z = fmaxf(acc.z, 0.f);
        acc.w = fmaxf(acc.w, 0.f);
    }
    *(v4f*)(y + ((b * oh + oy) * (long long)ow + ox) * c_out + co) = acc;
}

// The usual stem (3 -> 32 channels): one lane computes all 32 output channels of one output pixel
// on the matrix pipe.  The 27 inputs of the window sit in registers; the 27 x 32 weights fill 14
// registers of the wave ([k][c_out] in memory order: lane l of register r holds element 64 r + l),
// and one v_mfma_f32_4x4x1 per (input k, group of 4 output channels) broadcasts the four weights
// from lanes 4b..4b+3 of their register to all 16 blocks: 216 MFMAs per 64 pixels instead of 864
// multiply-adds per lane, which leaves the kernel bound by its memory traffic.
template <int ABID>
__device__ __forceinline__ v4f stem_mfma(float w, float x, v4f c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(w, x, c, 4, ABID, 0);
}

template <int CIN, int COUT, int P>
__device__ __forceinline__ void stem_pairs(const float (&wreg)[(9 * CIN * COUT + 63) / 64], const float (&xin)[9 * CIN],
                                           v4f (&acc)[COUT / 4])
{
    // pair P = k * (COUT/4) + g lives in block P % 16 of register P / 16
    if constexpr (P < 9 * CIN * (COUT / 4)) {
        constexpr int G = P % (COUT / 4), KI = P / (COUT / 4);
        acc[G] = stem_mfma<P % 16>(wreg[P / 16], xin[KI], acc[G]);
        stem_pairs<CIN, COUT, P + 1>(wreg, xin, acc);
    }
}

template <int CIN, int COUT>
__global__ __launch_bounds__(256) void stem3x3_fixed_kernel(const float* __restrict__ x, float* __restrict__ y,
                                                           const float* __restrict__ wt,
                                                           const float* __restrict__ bias, int h, int w, int oh,
                                                           int ow, int stride, int act, long long total)
{
    constexpr int LS = COUT + 4;                           // LDS row stride (floats)
    constexpr int NWR = (9 * CIN * COUT + 63) / 64;        // weight registers
    __shared__ __attribute__((aligned(16))) float tile[256 * LS];
    const int lane = threadIdx.x & 63;
    const long long t0 = (long long)blockIdx.x * 256;
    const long long t = t0 + threadIdx.x;
    float wreg[NWR];
#pragma unroll
    for (int r = 0; r < NWR; ++r) wreg[r] = r * 64 + lane < 9 * CIN * COUT ? wt[r * 64 + lane] : 0.f;
    // every lane takes part in the MFMAs; lanes past the last pixel compute pixel total-1 again
    const long long tc = t < total ? t : total - 1;
    const int ox = (int)(tc % ow);
    const int oy = (int)((tc / ow) % oh);
    const long long b = tc / ((long long)ow * oh);
    float xin[9 * CIN];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int iy = oy * stride + k / 3 - 1, ix = ox * stride + k % 3 - 1;
        const bool ok = iy >= 0 && iy < h && ix >= 0 && ix < w;
        const float* xp = x + ((b * h + (ok ? iy : 0)) * w + (ok ? ix : 0)) * CIN;
#pragma unroll
        for (int ci = 0; ci < CIN; ++ci) {
            const float v = xp[ci];
            xin[k * CIN + ci] = ok ? v : 0.f;
        }
    }
    v4f acc[COUT / 4];
#pragma unroll
    for (int g = 0; g < COUT / 4; ++g) acc[g] = *(const v4f*)(bias + g * 4);
    stem_pairs<CIN, COUT, 0>(wreg, xin, acc);
#pragma unroll
    for (int g = 0; g < COUT / 4; ++g) {
        v4f o = acc[g];
        if (act == SBN_ACT_RELU) {
            o.x = fmaxf(o.x, 0.f);
            o.y = fmaxf(o.y, 0.f);
            o.z = fmaxf(o.z, 0.f);
            o.w = fmaxf(o.w, 0.f);
        }
        *(v4f*)(tile + threadIdx.x * LS + g * 4) = o;
    }
    // the workgroup's 256 pixels are contiguous in y: store them as full rows
    __syncthreads();
#pragma unroll
    for (int i = 0; i < COUT / 4; ++i) {
        const int slot = i * 256 + threadIdx.x;
        const int pl = slot / (COUT / 4), c0 = (slot % (COUT / 4)) * 4;
        if (t0 + pl < total) *(v4f*)(y + (t0 + pl) * COUT + c0) = *(const v4f*)(tile + pl * LS + c0);
    }
}

// x [n][hw][c] -> y [n][c].  A workgroup takes one image x 64 channels: thread t owns channels
// 4*(t%16)..+3 and every sixteenth pixel starting at t/16 (16-byte loads, all of them independent);
// the sixteen partial sums meet in LDS and are added in 64 bits (relative error, 49 values
// between 0 and 1: 2.9e-8; four partial sums of 32 bits 5.7e-8).  (Bound by one load's way there and back: 49 pixels x 1024
// channels with 256 channels and four partial sums per workgroup 5.4 us for one
// image, 7.9 for 64; so 2.9 and 6.0.)
constexpr int kPoolChannels = 64;
__global__ __launch_bounds__(256) void avgpool_kernel(const float* __restrict__ x, float* __restrict__ y, int hw,
                                                     int c, int c_tiles)
{
    __shared__ __attribute__((aligned(16))) float part[16 * kPoolChannels];
    const long long b = blockIdx.x / c_tiles;
    const int at = (threadIdx.x & 15) * 4, ch = (blockIdx.x % c_tiles) * kPoolChannels + at;
    const int q = threadIdx.x >> 4;
    v4f s = {0.f, 0.f, 0.f, 0.f};
    if (ch < c)
        for (int p = q; p < hw; p += 16) s += *(const v4f*)(x + (b * hw + p) * c + ch);
    *(v4f*)(part + q * kPoolChannels + at) = s;
    __syncthreads();
    if (q == 0 && ch < c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double sum = 0.;
#pragma unroll
            for (int k = 0; k < 16; ++k) sum += (double)part[k * kPoolChannels + at + i];
            s[i] = (float)(sum / (double)hw);
        }
        *(v4f*)(y + b * c + ch) = s;
    }
}

int check_launch(const char* who)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sbn::fail(SBN_EHIP, "%s launch: %s", who, hipGetErrorString(e));
    return SBN_OK;
}

}  // namespace

namespace sbn {

int launch_copy(const void* src, void* dst, size_t bytes, void* stream)
{
    const size_t n16 = bytes / 16;
    if (n16 == 0) return SBN_OK;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;      // grid-stride, 32 workgroups per CU
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, (const v4f*)src,
                       (v4f*)dst, n16);
    return check_launch("copy");
}

int launch_dw3x3(const float* x, float* y, const float* w_dev, const float* b_dev, int n, int h, int w, int c,
                 int stride, int act, void* stream)
{
    const int oh = (h - 1) / stride + 1, ow = (w - 1) / stride + 1;
    const long long quads = (long long)ow * (c / 4);
    if ((long long)n * oh * quads == 0) return SBN_OK;
    // Rows of at most half a wave (4096 x 7 x 7 x 4: 9.5 us, 18.2 with a block per strip; x 16: 9.4 and 11.2; rows of 56
    // quads, x 32: 13.2 and 12.1)
    if (quads <= 32) {
        const long long total = (long long)n * ((oh + 3) / 4) * quads, blocks = (total + 255) / 256;
        if (blocks > 0x7FFFFFFFll) return fail(SBN_EINVAL, "depthwise layer too large for one launch");
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, x, y, w_dev, b_dev, h, w, c, oh, ow, act, total);
        };
        stride == 1 ? go(dw3x3_narrow_kernel<1, 4>) : go(dw3x3_narrow_kernel<2, 4>);
        return check_launch("dw3x3");
    }
    // Strips of four rows load 4.5 (stride 2: 6.75) values per output instead of 9; where they leave fewer than two
    // waves per compute unit, one row each: the chain of loads is shorter.  (49 images, 1.5 waves, 8 x 8 x 512 by stride 2: 5.4 and 5.1 us; 3
    // waves, 16 x 16 x 256 by stride 2: 5.7 and 6.8, 4 x 4 x 1024: 6.1 and 7.2.)
    int device = 0, cus = 0;
    if (hipGetDevice(&device) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0) cus = 256;
    const bool small = (long long)n * ((oh + 3) / 4) * quads < 64ll * 2 * cus;
    const int R = small ? 1 : 4;
    // (blocks of 64 threads where a row is short: at most 63 idle lanes per strip)
    const unsigned threads = quads % 256 == 0 || quads >= 2048 ? 256 : 64;
    const long long strips = (oh + R - 1) / R, per_strip = (quads + threads - 1) / threads, blocks = n * strips * per_strip;
    if (blocks > 0x7FFFFFFFll) return fail(SBN_EINVAL, "depthwise layer too large for one launch");
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), 0, (hipStream_t)stream, x, y, w_dev, b_dev, h, w, c,
                           oh, ow, act, (unsigned)strips, (unsigned)per_strip, (unsigned)(strips * per_strip), (unsigned)(n / 8 * 8 * strips * per_strip));
    };
    if (stride == 1)
        small ? go(dw3x3_kernel<1, 1>) : go(dw3x3_kernel<1, 4>);
    else
        small ? go(dw3x3_kernel<2, 1>) : go(dw3x3_kernel<2, 4>);
    return check_launch("dw3x3");
}

int launch_stem3x3(const float* x, float* y, const float* w_dev, const float* b_dev, int n, int h, int w, int c_in,
                   int c_out, int stride, int act, void* stream)
{
    const int oh = (h - 1) / stride + 1, ow = (w - 1) / stride + 1;
    if (c_in == 3 && c_out == 32) {
        const long long pixels = (long long)n * oh * ow;
        if (pixels == 0) return SBN_OK;
        if ((pixels + 255) / 256 > 0x7FFFFFFFll) return fail(SBN_EINVAL, "stem layer too large for one launch");
        hipLaunchKernelGGL((stem3x3_fixed_kernel<3, 32>), dim3((unsigned)((pixels + 255) / 256)), dim3(256), 0,
                           (hipStream_t)stream, x, y, w_dev, b_dev, h, w, oh, ow, stride, act, pixels);
        return check_launch("stem3x3");
    }
    const long long total = (long long)n * oh * ow * (c_out / 4);
    if (total == 0) return SBN_OK;
    const long long blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFll) return fail(SBN_EINVAL, "stem layer too large for one launch");
    hipLaunchKernelGGL(stem3x3_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, x, y, w_dev, b_dev, h,
                       w, c_in, c_out, oh, ow, stride, act, total);
    return check_launch("stem3x3");
}

int launch_avgpool(const float* x, float* y, int n, int hw, int c, void* stream)
{
    if ((long long)n * c * hw == 0) return SBN_OK;
    if (c % 4) return fail(SBN_ESHAPE, "the average pool needs a multiple of 4 channels (got %d)", c);
    const int c_tiles = (c + kPoolChannels - 1) / kPoolChannels;
    // As many images at a time as one launch takes (1024 channels: 1 048 575).
    const int most = (int)std::max<long long>(1, kMaxGroups256 / c_tiles);
    for (int at = 0; at < n; at += most) {
        const int some = std::min(most, n - at);
        hipLaunchKernelGGL(avgpool_kernel, dim3((unsigned)((long long)some * c_tiles)), dim3(256), 0, (hipStream_t)stream,
                           x + (long long)at * hw * c, y + (long long)at * c, hw, c, c_tiles);
        if (int rc = check_launch("avgpool")) return rc;
        if (n - at <= most) break;                                       // (at + most may not fit an int)
    }
    return SBN_OK;
}

}  // namespace sbn
