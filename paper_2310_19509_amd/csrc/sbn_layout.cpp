// Device layout of a packed layer: regroups the canonical rows (Algorithm 1's
// per-output-group block lists) into bundles of four 4-filter groups whose
// kept 4-channel pieces are walked together, so that one staged activation
// read serves every group of the bundle that keeps the piece.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstring>
#include <memory>

#include "sbn_internal.h"

namespace sbn {

// Nearest 16-bit float (ties to even) of a finite v, |v| < 65520, returned as bits; *back is its value.
static uint16_t to_half(float v, float* back)
{
    uint32_t u;
    std::memcpy(&u, &v, 4);
    const uint32_t sign = u >> 16 & 0x8000u;
    u &= 0x7FFFFFFFu;
    float a;
    std::memcpy(&a, &u, 4);
    if (u < 0x38800000u) {                       // below 2^-14: a multiple of 2^-24; 0.5 has that spacing
        const float r = (a + 0.5f) - 0.5f;
        *back = sign ? -r : r;
        return (uint16_t)(sign | (uint32_t)(r * 16777216.0f));
    }
    u += 0xFFFu + (u >> 13 & 1u);
    u &= ~0x1FFFu;
    std::memcpy(&a, &u, 4);
    *back = sign ? -a : a;
    return (uint16_t)(sign | ((u - 0x38000000u) >> 13));
}

// The weights as pairs of 16-bit floats (DeviceLayout::wh).  Only layers whose outputs sum enough
// products: a pair carries 22 to 23 bits of a 24-bit weight and the product of the two low halves is
// left out, about 9e-8 of the result in all, whatever the length of the sum, while a sum of n
// products in 32-bit floats loses about 1e-8 * sqrt(n) (simulated and measured: 8.2e-8 against 9.2e-8
// with 64 products, 1.09e-7 against 9.8e-8 with 128, 2.0e-7 against 1.1e-7 with 512).
static void build_half_pairs(sbn_packed* p)
{
    DeviceLayout& L = p->dev;
    L.wh.clear();
    L.wh_exp.clear();
    L.n_steps = 0;
    const int taps = p->kh * p->kw;
    const size_t kept = p->kidx.size() * (size_t)p->go * p->gi * taps;
    if (taps == 1 || p->c_in % 4 || kept < (size_t)kHalfMinKept * p->c_out) return;
    const int n_steps = L.n_chunks32 * taps;
    const size_t n_filters = (size_t)L.n_bundles * kBundleChannels, wstride = (size_t)taps * 64;
    if (n_filters * (size_t)n_steps * 128 >= 0xFFFFFFFFull) return;      // 32-bit byte offsets on the device

    // Per filter: the power of two that takes its largest weight to [2^14, 2^15).  An entry holds its
    // weights as [tap][g][ci][co]; per entry, the largest of every filter first.
    auto bits_of = [](float v) {
        uint32_t u;
        std::memcpy(&u, &v, 4);
        return u & 0x7FFFFFFFu;
    };
    std::vector<uint32_t> top(n_filters, 0u), piece(L.n_entries * kBundleChannels, 0u);
    for (int b = 0; b < L.n_bundles; ++b) {
        const uint32_t* wo = &L.woff[(size_t)b * (L.n_chunks + 1)];
        for (size_t e = wo[0]; e < wo[L.n_chunks]; ++e) {
            const float* w = &L.wts[e * wstride];
            uint32_t* m = &piece[e * kBundleChannels];
            for (int i = 0; i < taps * kBundleGroups; ++i, w += 16)
                for (int j = 0; j < 16; ++j) m[i % kBundleGroups * 4 + j % 4] = std::max(m[i % kBundleGroups * 4 + j % 4], bits_of(w[j]));
            for (int f = 0; f < kBundleChannels; ++f) top[(size_t)b * kBundleChannels + f] = std::max(top[(size_t)b * kBundleChannels + f], m[f]);
        }
    }
    // (a filter whose weights span so much that a whole kept piece would lose bits: 32-bit kernels)
    for (int b = 0; b < L.n_bundles; ++b) {
        const uint32_t* wo = &L.woff[(size_t)b * (L.n_chunks + 1)];
        for (size_t e = wo[0]; e < wo[L.n_chunks]; ++e)
            for (int f = 0; f < kBundleChannels; ++f) {
                const uint32_t m = piece[e * kBundleChannels + f];
                if (m != 0 && (m >> 23) + 26 < (top[(size_t)b * kBundleChannels + f] >> 23)) return;
            }
    }
    std::vector<float> scale(n_filters, 1.0f);
    L.wh_exp.assign(n_filters, 0);
    for (size_t f = 0; f < n_filters; ++f) {
        const int e = std::max((int)(top[f] >> 23), 27);
        if (e == 255) {                                                  // infinite or NaN weights stay with the 32-bit kernels
            L.wh_exp.clear();
            return;
        }
        L.wh_exp[f] = e - 141;
        const uint32_t s = (uint32_t)(268 - e) << 23;
        std::memcpy(&scale[f], &s, 4);
    }
    L.n_steps = n_steps;
    L.wh.assign(n_filters * (size_t)n_steps * 64, 0);
    for (int b = 0; b < L.n_bundles; ++b)
        for (int c = 0; c < L.n_chunks32; ++c) {
            const uint32_t* r = &L.records32[((size_t)b * L.n_chunks32 + c) * 8];
            const float* w = &L.wts[(size_t)L.woff32[(size_t)b * (L.n_chunks32 + 1) + c] * wstride];
            for (int q = 0; q < 8 && r[q] != 0; ++q, w += wstride) {
                const int kb4 = (int)(r[q] >> 12);                       // channels 4 * kb4 .. + 3 of the 32
                uint16_t* frag = &L.wh[(((size_t)b * n_steps + (size_t)c * taps) * 2) * 512];
                for (int t = 0; t < taps; ++t, frag += 1024)
                    for (int g = 0; g < kBundleGroups; ++g) {
                        if (!(r[q] >> g & 1u)) continue;                 // removed: stays zero
                        for (int co = 0; co < 4; ++co) {
                            const int f = g * 4 + co;
                            const float sc = scale[(size_t)b * kBundleChannels + f];
                            uint16_t* const to = frag + (size_t)(kb4 / 2 * 16 + f) * 8 + (kb4 % 2) * 4;
                            for (int ci = 0; ci < 4; ++ci) {
                                const float v = w[t * 64 + g * 16 + ci * 4 + co] * sc;
                                float hi, lo;
                                to[ci] = to_half(v, &hi);
                                to[512 + ci] = to_half((v - hi) * 2048.0f, &lo);
                            }
                        }
                    }
            }
        }
}

// Nearest bfloat16 (ties to even) of a finite v that does not overflow, returned as bits; *back is its value.
static inline uint16_t to_bf16(float v, float* back)
{
    uint32_t u;
    std::memcpy(&u, &v, 4);
    u = (u + 0x7FFFu + (u >> 16 & 1u)) & 0xFFFF0000u;
    std::memcpy(back, &u, 4);
    return (uint16_t)(u >> 16);
}

// The weights as exact triples of bfloat16 (DeviceLayout::wt).
static void build_triples(sbn_packed* p)
{
    DeviceLayout& L = p->dev;
    L.wt.clear();
    L.w_top = 0.0f;
    if (p->kh * p->kw != 1 || p->c_in % 4 || p->c_in <= kChunk) return;
    if (!conv1x1_wide_pays(p) && forced_kernel_form(SBN_CONV1X1) < 2000) return;
    const size_t n_pairs = ((size_t)L.n_bundles + 1) / 2, n_steps = (size_t)L.n_chunks * 4;
    if (n_pairs * n_steps * 3072 >= 0xFFFFFFFFull) return;               // 32-bit byte offsets on the device
    // Infinite, NaN and nearly infinite weights (the first bfloat16 would overflow), and weights whose last bits
    // lie below the smallest normal bfloat16, stay with the 32-bit kernels.
    uint32_t top = 0;
    for (const float v : L.wts) {
        uint32_t u;
        std::memcpy(&u, &v, 4);
        u &= 0x7FFFFFFFu;
        if (u >= 0x7F7F8000u || (u != 0 && u < 0x0D800000u)) return;     // (2^-100)
        top = std::max(top, u);
    }
    std::memcpy(&L.w_top, &top, 4);
    L.wt.assign(n_pairs * n_steps * 1536, 0);
    for (int b = 0; b < L.n_bundles; ++b)
        for (int c = 0; c < L.n_chunks; ++c) {
            const uint32_t* r = &L.records[((size_t)b * L.n_chunks + c) * kSlots];
            const float* w = &L.wts[(size_t)L.woff[(size_t)b * (L.n_chunks + 1) + c] * 64];
            for (int q = 0; q < kSlots && r[q] != 0; ++q, w += 64) {
                const int piece = (int)(r[q] >> 12);                     // channels 4 * piece .. + 3 of the 64
                uint16_t* const frag = &L.wt[((size_t)(b / 2) * n_steps + (size_t)c * 4 + piece / 4) * 1536];
                for (int f = 0; f < kBundleChannels; ++f) {              // (removed groups' weights are zeros)
                    uint16_t* const to = frag + (size_t)(piece % 4 / 2 * 32 + b % 2 * kBundleChannels + f) * 8 + piece % 2 * 4;
                    for (int ci = 0; ci < 4; ++ci) {
                        const float v = w[f * 4 + ci];
                        float hi, mid, lo;
                        to[ci] = to_bf16(v, &hi);
                        to[512 + ci] = to_bf16(v - hi, &mid);
                        to[1024 + ci] = to_bf16(v - hi - mid, &lo);
                    }
                }
            }
        }
}

void build_device_layout(sbn_packed* p)
{
    DeviceLayout& L = p->dev;
    const int taps = p->kh * p->kw, go = p->go, gi = p->gi;
    const int n_groups4 = p->c_out / 4;                              // go is 4 or 8
    L.n_bundles = (n_groups4 + kBundleGroups - 1) / kBundleGroups;
    L.n_chunks = (p->c_in + kChunk - 1) / kChunk;
    const size_t wstride = (size_t)taps * kBundleGroups * 16;        // floats per entry
    const size_t blk = (size_t)taps * gi * go;

    L.n_chunks32 = (p->c_in + 31) / 32;
    L.records.assign((size_t)L.n_bundles * L.n_chunks * kSlots, 0u);
    L.woff.assign((size_t)L.n_bundles * (L.n_chunks + 1), 0u);
    L.records32.assign((size_t)L.n_bundles * L.n_chunks32 * 8, 0u);
    L.woff32.assign((size_t)L.n_bundles * (L.n_chunks32 + 1), 0u);
    L.wts.clear();
    size_t n_entries = 0;

    const int sub = go / 4;                                          // 4-filter groups per canonical row
    const size_t n_pos = (size_t)(p->c_in + 3) / 4;
    std::vector<uint32_t> present(n_pos);                            // per piece: which groups keep it
    std::vector<size_t> entry(n_pos);                                // and its entry
    std::vector<int> kept;                                           // the bundle's pieces, ascending
    kept.reserve(n_pos);
    {
        size_t most = 0;                                             // room for all entries at once
        for (int b = 0; b < L.n_bundles; ++b) {
            size_t blocks = 0;
            for (int row = b * kBundleGroups / sub; row < std::min(p->c_out / go, (b + 1) * kBundleGroups / sub); ++row)
                blocks += p->row_ptr[(size_t)row + 1] - p->row_ptr[(size_t)row];
            most += std::min(n_pos, blocks * std::max<size_t>(1, (size_t)gi / 4));
        }
        L.wts.reserve(most * wstride);
    }
    for (int b = 0; b < L.n_bundles; ++b) {
        const int g_lo = b * kBundleGroups, g_hi = std::min(n_groups4, g_lo + kBundleGroups);
        std::fill(present.begin(), present.end(), 0u);
        for (int g4 = g_lo; g4 < g_hi; ++g4) {
            const int row = g4 / sub;
            for (uint32_t e = p->row_ptr[(size_t)row]; e < p->row_ptr[(size_t)row + 1]; ++e)
                for (int c = 0; c < gi; ++c) present[(size_t)(p->kidx[e] + c) / 4] |= 1u << (g4 - g_lo);
        }
        kept.clear();
        for (size_t kb4 = 0; kb4 < n_pos; ++kb4)
            if (present[kb4] != 0) {
                entry[kb4] = n_entries++;
                kept.push_back((int)kb4);
            }
        L.wts.resize(n_entries * wstride, 0.0f);
        for (int g4 = g_lo; g4 < g_hi; ++g4) {
            const int row = g4 / sub, s = g4 % sub, g = g4 - g_lo;
            for (uint32_t e = p->row_ptr[(size_t)row]; e < p->row_ptr[(size_t)row + 1]; ++e)
                for (int c = 0; c < gi; ++c) {
                    const int ch = p->kidx[e] + c;
                    float* const to = &L.wts[entry[(size_t)ch / 4] * wstride + (size_t)g * 16];
                    const float* const from = &p->vals[e * blk + (size_t)c * go + (size_t)s * 4];
                    // 1x1: [g][co][ci] (16-byte loads per lane); 3x3: [tap][g][ci][co] (4-byte loads)
                    if (taps == 1)
                        for (int co = 0; co < 4; ++co) to[co * 4 + ch % 4] = from[co];
                    else
                        for (int t = 0; t < taps; ++t)
                            for (int co = 0; co < 4; ++co)
                                to[(size_t)t * kBundleGroups * 16 + (size_t)(ch % 4) * 4 + co] = from[(size_t)t * gi * go + co];
                }
        }
        // records and chunk offsets
        uint32_t* wo = &L.woff[(size_t)b * (L.n_chunks + 1)];
        std::vector<int> fill((size_t)L.n_chunks, 0);
        for (int c = 0; c <= L.n_chunks; ++c) wo[c] = (uint32_t)n_entries;
        for (const int kb4 : kept) {
            const int c = kb4 / kSlots, q = fill[(size_t)c]++;
            L.records[((size_t)b * L.n_chunks + c) * kSlots + q] = ((uint32_t)(kb4 % kSlots) << 12) | present[(size_t)kb4];
            wo[c] = std::min(wo[c], (uint32_t)entry[(size_t)kb4]);
        }
        // empty chunks start where the next non-empty one does
        for (int c = L.n_chunks - 1; c >= 0; --c) wo[c] = std::min(wo[c], wo[c + 1]);
        // the same entries, one record of 8 descriptors per 32 channels
        uint32_t* wo32 = &L.woff32[(size_t)b * (L.n_chunks32 + 1)];
        std::vector<int> fill32((size_t)L.n_chunks32, 0);
        for (int c = 0; c <= L.n_chunks32; ++c) wo32[c] = (uint32_t)n_entries;
        for (const int kb4 : kept) {
            const int c = kb4 / 8, q = fill32[(size_t)c]++;
            L.records32[((size_t)b * L.n_chunks32 + c) * 8 + q] = ((uint32_t)(kb4 % 8) << 12) | present[(size_t)kb4];
            wo32[c] = std::min(wo32[c], (uint32_t)entry[(size_t)kb4]);
        }
        for (int c = L.n_chunks32 - 1; c >= 0; --c) wo32[c] = std::min(wo32[c], wo32[c + 1]);
    }
    L.n_entries = n_entries;
    // every-piece tables for 1x1 layers of more than one chunk that keep most of their pieces
    L.desc_s.clear();
    L.wts_s.clear();
    const size_t n_pieces = (size_t)(p->c_in + 3) / 4;
    if (taps == 1 && p->c_in > kChunk && p->c_in % 4 == 0 &&
        (double)n_entries >= kStaticWalkMinFill * (double)((size_t)L.n_bundles * n_pieces)) {
        const size_t per_bundle = (size_t)L.n_chunks * kSlots;
        L.desc_s.assign((size_t)L.n_bundles * per_bundle, 0u);
        L.wts_s.assign((size_t)L.n_bundles * per_bundle * 64, 0.0f);
        for (int b = 0; b < L.n_bundles; ++b)
            for (int c = 0; c < L.n_chunks; ++c) {
                const uint32_t* r = &L.records[((size_t)b * L.n_chunks + c) * kSlots];
                const size_t e0 = L.woff[(size_t)b * (L.n_chunks + 1) + c];
                for (int q = 0; q < kSlots && r[q] != 0; ++q) {
                    const size_t piece = (size_t)c * kSlots + (r[q] >> 12);
                    L.desc_s[(size_t)b * per_bundle + piece] = r[q] & 0xFu;
                    std::copy(L.wts.begin() + (e0 + q) * 64, L.wts.begin() + (e0 + q + 1) * 64,
                              L.wts_s.begin() + ((size_t)b * per_bundle + piece) * 64);
                }
            }
    }
    build_half_pairs(p);
    build_triples(p);
    L.bias_padded.assign((size_t)L.n_bundles * kBundleChannels, 0.0f);
    std::copy(p->bias.begin(), p->bias.end(), L.bias_padded.begin());
}

// What the kernels take for granted about the tables: checked once per packed layer, on the
// host, so that no kernel ever walks a malformed record.  Returns NULL or what is wrong.
static const char* check_tables(const std::vector<uint32_t>& rec, const std::vector<uint32_t>& wo, int n_bundles,
                                int n_chunks, int slots, size_t n_entries)
{
    if (rec.size() != (size_t)n_bundles * n_chunks * slots || wo.size() != (size_t)n_bundles * (n_chunks + 1))
        return "table sizes";
    size_t next = 0;                                   // entries are numbered bundle by bundle, chunk by chunk
    for (int b = 0; b < n_bundles; ++b)
        for (int c = 0; c < n_chunks; ++c) {
            const uint32_t* r = &rec[((size_t)b * n_chunks + c) * slots];
            int n = 0;
            while (n < slots && r[n] != 0) ++n;
            for (int q = n; q < slots; ++q)
                if (r[q] != 0) return "descriptor after the terminator";
            for (int q = 0; q < n; ++q) {
                const uint32_t kb4 = r[q] >> 12, m = r[q] & 0xFFFu;
                if (kb4 >= (uint32_t)slots || m == 0 || m > 15u) return "descriptor out of range";
                if (q && kb4 <= (r[q - 1] >> 12)) return "pieces of a record not ascending";
            }
            if (wo[(size_t)b * (n_chunks + 1) + c] != next) return "first-entry index";
            next += (size_t)n;
            if (wo[(size_t)b * (n_chunks + 1) + c + 1] != next) return "first-entry index of the next chunk";
        }
    return next == n_entries ? nullptr : "entry count";
}

const char* check_device_layout(const sbn_packed* p)
{
    const DeviceLayout& L = p->dev;
    if (L.n_bundles != (p->c_out / 4 + kBundleGroups - 1) / kBundleGroups || L.n_chunks != (p->c_in + kChunk - 1) / kChunk ||
        L.n_chunks32 != (p->c_in + 31) / 32)
        return "bundle or chunk count";
    if (const char* e = check_tables(L.records, L.woff, L.n_bundles, L.n_chunks, kSlots, L.n_entries)) return e;
    if (const char* e = check_tables(L.records32, L.woff32, L.n_bundles, L.n_chunks32, 8, L.n_entries)) return e;
    if (L.wts.size() != L.n_entries * (size_t)p->kh * p->kw * kBundleGroups * 16) return "weight array size";
    if (L.bias_padded.size() != (size_t)L.n_bundles * kBundleChannels) return "bias array size";
    if (!L.desc_s.empty()) {
        const size_t per_bundle = (size_t)L.n_chunks * kSlots;
        if (p->kh != 1 || L.desc_s.size() != (size_t)L.n_bundles * per_bundle || L.wts_s.size() != L.desc_s.size() * 64)
            return "every-piece table sizes";
        size_t present = 0;
        for (size_t i = 0; i < L.desc_s.size(); ++i) {
            if (L.desc_s[i] > 15u) return "every-piece mask out of range";
            if ((i % per_bundle) * 4 >= (size_t)p->c_in && L.desc_s[i] != 0) return "every-piece mask past the last channel";
            present += L.desc_s[i] != 0;
        }
        if (present != L.n_entries) return "every-piece entry count";
    } else if (!L.wts_s.empty()) {
        return "every-piece weights without masks";
    }
    if (L.wh.empty() ? !L.wh_exp.empty() || L.n_steps != 0
                     : p->kh != 3 || L.n_steps != 9 * L.n_chunks32 || L.wh.size() != (size_t)L.n_bundles * L.n_steps * 1024 ||
                           L.wh_exp.size() != (size_t)L.n_bundles * kBundleChannels)
        return "16-bit pair table sizes";
    if (!L.wt.empty() && (p->kh != 1 || p->c_in <= kChunk || L.wt.size() != (size_t)((L.n_bundles + 1) / 2) * L.n_chunks * 4 * 1536))
        return "bfloat16 triple table size";
    return nullptr;
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int upload_device_layout(sbn_packed* p)
{
    DeviceLayout& L = p->dev;
    int ndev = 0;
    hipError_t e = hipGetDeviceCount(&ndev);
    if (e != hipSuccess) return fail(SBN_EHIP, "hipGetDeviceCount: %s", hipGetErrorString(e));
    if (p->device >= ndev) return fail(SBN_EINVAL, "device %d does not exist (%d visible)", p->device, ndev);
    int prev = 0;
    (void)hipGetDevice(&prev);
    if ((e = hipSetDevice(p->device)) != hipSuccess) return fail(SBN_EHIP, "hipSetDevice: %s", hipGetErrorString(e));
    int cus = 0;                           // the launchers size their grids by it
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->device) == hipSuccess && cus > 0) L.cus = cus;

    // One allocation.  The kernels fetch the weights of a whole record (up to
    // 16 entries) at once, so the weight array carries 16 entries of slack.
    const size_t wstride = (size_t)p->kh * p->kw * kBundleGroups * 16;
    const size_t b_rec = align256(L.records.size() * sizeof(uint32_t));
    const size_t b_woff = align256(L.woff.size() * sizeof(uint32_t));
    const size_t b_rec32 = align256(L.records32.size() * sizeof(uint32_t));
    const size_t b_woff32 = align256(L.woff32.size() * sizeof(uint32_t));
    const size_t b_wts = align256((L.wts.size() + kSlots * wstride) * sizeof(float));
    const size_t b_bias = align256(L.bias_padded.size() * sizeof(float));
    const size_t b_desc_s = align256(L.desc_s.size() * sizeof(uint32_t));
    const size_t b_wts_s = align256(L.wts_s.size() * sizeof(float));
    const size_t b_wh = align256(L.wh.size() * sizeof(uint16_t));
    const size_t b_wh_exp = align256(L.wh_exp.size() * sizeof(int32_t));
    const size_t b_wt = align256(L.wt.size() * sizeof(uint16_t));
    const size_t total = b_rec + b_woff + b_rec32 + b_woff32 + b_wts + b_bias + b_desc_s + b_wts_s + b_wh + b_wh_exp + b_wt;
    // (written once: not zeroed first, the gaps behind the arrays are; before the device memory, as it may throw)
    std::unique_ptr<char[]> host(new char[total]);
    char* blob = nullptr;
    if ((e = hipMalloc((void**)&blob, total)) != hipSuccess) {
        (void)hipSetDevice(prev);
        return fail(e == hipErrorOutOfMemory ? SBN_ENOMEM : SBN_EHIP, "hipMalloc(%zu): %s", total, hipGetErrorString(e));
    }
    size_t off = 0;
    auto put = [&](const void* data, size_t used, size_t reserved) {
        if (used) std::memcpy(host.get() + off, data, used);
        std::memset(host.get() + off + used, 0, reserved - used);
        char* const at = blob + off;
        off += reserved;
        return reserved ? at : nullptr;
    };
    L.d_records = (uint32_t*)put(L.records.data(), L.records.size() * sizeof(uint32_t), b_rec);
    L.d_woff = (uint32_t*)put(L.woff.data(), L.woff.size() * sizeof(uint32_t), b_woff);
    L.d_records32 = (uint32_t*)put(L.records32.data(), L.records32.size() * sizeof(uint32_t), b_rec32);
    L.d_woff32 = (uint32_t*)put(L.woff32.data(), L.woff32.size() * sizeof(uint32_t), b_woff32);
    L.d_wts = (float*)put(L.wts.data(), L.wts.size() * sizeof(float), b_wts);
    L.d_bias = (float*)put(L.bias_padded.data(), L.bias_padded.size() * sizeof(float), b_bias);
    L.d_desc_s = (uint32_t*)put(L.desc_s.data(), L.desc_s.size() * sizeof(uint32_t), b_desc_s);       // NULL when there are none
    L.d_wts_s = (float*)put(L.wts_s.data(), L.wts_s.size() * sizeof(float), b_wts_s);
    L.d_wh = (uint16_t*)put(L.wh.data(), L.wh.size() * sizeof(uint16_t), b_wh);
    L.d_wh_exp = (int32_t*)put(L.wh_exp.data(), L.wh_exp.size() * sizeof(int32_t), b_wh_exp);
    L.d_wt = (uint16_t*)put(L.wt.data(), L.wt.size() * sizeof(uint16_t), b_wt);
    e = hipMemcpy(blob, host.get(), total, hipMemcpyHostToDevice);
    (void)hipSetDevice(prev);
    if (e != hipSuccess) {
        (void)hipFree(blob);
        return fail(SBN_EHIP, "hipMemcpy of packed layer: %s", hipGetErrorString(e));
    }
    L.d_blob = blob;
    return SBN_OK;
}

void release_device_layout(sbn_packed* p)
{
    if (p->dev.d_blob) {
        (void)hipFree(p->dev.d_blob);
        p->dev.d_blob = nullptr;
    }
}

}  // namespace sbn
