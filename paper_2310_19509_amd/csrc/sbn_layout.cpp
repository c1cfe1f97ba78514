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

// The wide multiplies take the time of all c_in x c_out weights, channels past c_out in a 128-channel tile included;
// the 32-bit forms that of the 4 x 4 blocks that hold a kept weight plus a share that does not shrink with them.  The
// margin is the share of such blocks over the least that pays.  Gain over the 32-bit form that the rule replaces, at a
// share of 1 / 0.7 / 0.6 / 0.5 / 0.4 (layers in turn, so that weights are not in the L2; margin 1 lies in the gap marked |):
//   c_in  128, 25088 pixels x 128     1.12 | 1.00 0.97 0.91
//         256, 50176 x 256            1.46 1.12 | 1.02 0.93 0.83
//         512, 50176 x 512            1.57 1.32 1.20 1.06 | 0.97
//         768, 10000 x 384            1.92 1.48 1.32 1.18 | 1.09
//        1024, 12544 x 1024           1.69 1.34 1.23 1.12 1.00 |
// (Fewer than 96 output channels leave a quarter of a tile or more idle.)
double conv1x1_wide_margin(const sbn_packed* p)
{
    const double padded = (double)((p->c_out + 127) / 128 * 128);
    return p->c_out > 80 ? 256.0 * (double)p->dev.n_present / ((5.0 * p->c_in + 1280.0) * padded) : 0.0;
}
bool conv1x1_wide_pays(const sbn_packed* p) { return conv1x1_wide_margin(p) >= 1.0; }

// Layers that gain from the 32 x 32 tiles alone, at the right number of pixels (conv1x1_split_chosen): those tiles read the activations
// once per 32 output channels and split the input channels, where the 32-bit form that splits them reads them once per 16 and the others
// do not split them.  Up to 64 output channels at almost any share kept, more from 0.3 on, where the most pixels that the form takes (four
// tiles per compute unit) are more than the fewest (four times the output channels): below 512 on 256 compute units.  (At 512 the one launch
// between the two lines, 2048 pixels, is a tie at 70 %: 12.4 us against 12.3 of the 32-bit form with 512 input channels, 60 % 12.4 and 12.8; the tables are
// 1.6 MB, nearly as much as the layer's others, and 0.8 of its 1.4 ms of packing on the host.)
bool conv1x1_split_pays(const sbn_packed* p)
{
    if ((p->c_out + 31) / 32 * 32 * 3 > p->c_out * 4) return false;     // (a quarter of the channels of the tiles idle)
    const double share = 16.0 * (double)p->dev.n_present / ((double)p->c_in * p->c_out);
    if (p->c_out <= 64) return p->c_in >= 192 && share >= (p->c_in >= 512 ? 0.05 : 0.15);
    const long long most = 4ll * p->dev.cus / ((p->dev.n_bundles + 1) / 2) * 32;
    return p->c_out > 80 && p->c_in >= 256 && share >= 0.3 && most > 4ll * p->c_out;
}

// Kernels in 4 x 4 blocks that a layer keeps, over all that the wide multiplies go through (input channels in 32s,
// output channels in 64s).  The multiplies' time does not depend on it, the 32-bit form's does; us, 32-bit form against this one (layers in
// turn, so that weights are not in the L2):
//   share kept                   0.5       0.4       0.3       0.2
//   3 x 23 x 23, 128 x 128       19 / 15   17 / 15   15 / 15   13 / 15
//   32 x 7 x 7, 512 x 512        68 / 47   62 / 47   51 / 46   40 / 46
//   32 x 14 x 14, 256 x 256      65 / 47   58 / 46   46 / 45   36 / 45
//   32 x 28 x 28, 128 x 128      59 / 47   52 / 46   44 / 45   34 / 44
//   32 x 56 x 56, 64 x 64        56 / 51   49 / 49   40 / 48   31 / 47
//   16 x 90 x 90, 512 x 512    3120 / 2542 2663 / 2521 2166 / 2438 1641 / 2403
// (At 0.3, where it is a tie, the 32-bit form's smaller tables decide: with three sets of four such layers in turn 164 us against 174.)
double conv3x3_share_kept(const sbn_packed* p)
{
    return 16.0 * (double)p->dev.n_present / ((double)((p->c_in + 31) / 32 * 32) * ((p->c_out + 63) / 64 * 64));
}
bool conv3x3_wide_pays(const sbn_packed* p) { return p->stride == 1 && p->c_in >= 32 && conv3x3_share_kept(p) >= 0.33; }

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
    const int taps = p->kh * p->kw;
    const bool pays = taps == 1 ? conv1x1_wide_pays(p) || conv1x1_split_pays(p) : conv3x3_wide_pays(p);
    const int forced = forced_kernel_form(p->kind);
    const bool wanted = forced >= 2000 && forced < 3000;                 // (the few-pixel forms, from 3000 on, do not read them)
    if (p->c_in % 4 || (taps == 1 && p->c_in <= kChunk) || p->stride != 1 || (!pays && !wanted)) return;
    const size_t n_pairs = ((size_t)L.n_bundles + 1) / 2, n_steps = taps == 1 ? (size_t)L.n_chunks * 4 : (size_t)L.n_chunks32 * 18;
    if (n_pairs * n_steps * 3072 >= 0xFFFFFFFFull) return;               // 32-bit byte offsets on the device
    // Infinite, NaN and nearly infinite weights (the first bfloat16 would overflow), and weights whose last bits
    // lie below the smallest normal bfloat16, stay with the 32-bit kernels.
    uint32_t top = 0, outside = 0;
    for (const float v : L.wts) {                                        // (no branch: a vector loop)
        uint32_t u;
        std::memcpy(&u, &v, 4);
        u &= 0x7FFFFFFFu;
        outside |= (uint32_t)(u - 1u < 0x0D800000u - 1u);                // (2^-100)
        top = std::max(top, u);
    }
    if (outside || top >= 0x7F7F8000u) return;
    std::memcpy(&L.w_top, &top, 4);
    L.wt.assign(n_pairs * n_steps * 1536, 0);
    const size_t wstride = (size_t)taps * 64;
    for (int b = 0; b < L.n_bundles; ++b)
        for (int c = 0; c < L.n_chunks32; ++c) {
            const uint32_t* r = &L.records32[((size_t)b * L.n_chunks32 + c) * 8];
            const float* w = L.wts.data() + (size_t)L.woff32[(size_t)b * (L.n_chunks32 + 1) + c] * wstride;
            for (int q = 0; q < 8 && r[q] != 0; ++q, w += wstride) {
                const int piece = (int)(r[q] >> 12);                     // channels 4 * piece .. + 3 of the 32
                uint16_t* frag = &L.wt[((size_t)(b / 2) * n_steps + (size_t)c * 2 * taps + piece / 4) * 1536 +
                                       (size_t)(piece % 4 / 2 * 32 + b % 2 * kBundleChannels) * 8 + piece % 2 * 4];
                for (int t = 0; t < taps; ++t, frag += 2 * 1536)
                    for (int f = 0; f < kBundleChannels; ++f) {
                        if (!(r[q] >> (f / 4) & 1u)) continue;           // (a removed group's weights are zeros)
                        for (int ci = 0; ci < 4; ++ci) {
                            const float v = w[t * 64 + f * 4 + ci];
                            float hi, mid, lo;
                            frag[f * 8 + ci] = to_bf16(v, &hi);
                            frag[f * 8 + ci + 512] = to_bf16(v - hi, &mid);
                            frag[f * 8 + ci + 1024] = to_bf16(v - hi - mid, &lo);
                        }
                    }
            }
        }
}

void build_device_layout(sbn_packed* p)
{
    DeviceLayout& L = p->dev;
    const int taps = p->kh * p->kw, go = p->go, gi = p->gi;
    int ndev = 0, cus = 0;                                           // the rules and the launchers count by it
    if (p->device >= 0 && hipGetDeviceCount(&ndev) == hipSuccess && p->device < ndev &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->device) == hipSuccess && cus > 0) L.cus = cus;
    const int n_groups4 = p->c_out / 4;                              // go is 4 or 8
    L.n_bundles = (n_groups4 + kBundleGroups - 1) / kBundleGroups;
    L.n_chunks = (p->c_in + kChunk - 1) / kChunk;
    const size_t wstride = (size_t)taps * kBundleGroups * 16;        // floats per entry
    const size_t blk = (size_t)taps * gi * go;

    L.n_chunks32 = (p->c_in + 31) / 32;
    L.records.assign((size_t)L.n_bundles * L.n_chunks * kSlots, 0u);
    L.woff.assign((size_t)L.n_bundles * (L.n_chunks + 1), 0u);
    L.records32.assign((size_t)L.n_bundles * L.n_chunks32 * 8, 0u);
    L.where.assign((size_t)L.n_bundles * L.n_chunks32 * 8, kNoEntry);
    L.woff32.assign((size_t)L.n_bundles * (L.n_chunks32 + 1), 0u);
    L.wts.clear();
    size_t n_entries = 0;
    L.n_present = 0;

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
                L.n_present += (size_t)__builtin_popcount(present[kb4]);
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
                    for (int t = 0; t < taps; ++t)                   // [tap][g][co][ci]
                        for (int co = 0; co < 4; ++co) to[(size_t)t * kBundleGroups * 16 + co * 4 + ch % 4] = from[(size_t)t * gi * go + co];
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
        for (const int kb4 : kept) {
            const size_t at = entry[(size_t)kb4] * wstride * sizeof(float);
            L.where[(size_t)b * L.n_chunks32 * 8 + (size_t)kb4] = (uint32_t)std::min<size_t>(at, kNoEntry);
        }
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
    if (L.where.size() != (size_t)L.n_bundles * L.n_chunks32 * 8) return "entry offset table size";
    for (const uint32_t at : L.where)
        if (at != kNoEntry && (size_t)at + (size_t)p->kh * p->kw * 256 > L.wts.size() * sizeof(float)) return "entry offset out of range";
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
    if (!L.wt.empty() && ((p->kh == 1 && p->c_in <= kChunk) || p->stride != 1 ||
                          L.wt.size() != (size_t)((L.n_bundles + 1) / 2) * (p->kh == 1 ? L.n_chunks * 4 : L.n_chunks32 * 18) * 1536))
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
    // One allocation.  The kernels fetch the weights of a whole record (up to
    // 16 entries) at once, so the weight array carries 16 entries of slack.
    const size_t wstride = (size_t)p->kh * p->kw * kBundleGroups * 16;
    const size_t b_rec = align256(L.records.size() * sizeof(uint32_t));
    const size_t b_woff = align256(L.woff.size() * sizeof(uint32_t));
    const size_t b_rec32 = align256(L.records32.size() * sizeof(uint32_t));
    const size_t b_woff32 = align256(L.woff32.size() * sizeof(uint32_t));
    const size_t b_where = align256(L.where.size() * sizeof(uint32_t));
    const size_t b_wts = align256((L.wts.size() + kSlots * wstride) * sizeof(float));
    const size_t b_bias = align256(L.bias_padded.size() * sizeof(float));
    const size_t b_desc_s = align256(L.desc_s.size() * sizeof(uint32_t));
    const size_t b_wts_s = align256(L.wts_s.size() * sizeof(float));
    const size_t b_wt = align256(L.wt.size() * sizeof(uint16_t));
    const size_t total = b_rec + b_woff + b_rec32 + b_woff32 + b_where + b_wts + b_bias + b_desc_s + b_wts_s + b_wt;
    // (written once: not zeroed first, the gaps behind the arrays are; before the device is changed, as it may throw)
    std::unique_ptr<char[]> host(new char[total]);
    int prev = 0;
    (void)hipGetDevice(&prev);
    if ((e = hipSetDevice(p->device)) != hipSuccess) return fail(SBN_EHIP, "hipSetDevice: %s", hipGetErrorString(e));
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
    L.d_where = (uint32_t*)put(L.where.data(), L.where.size() * sizeof(uint32_t), b_where);
    L.d_wts = (float*)put(L.wts.data(), L.wts.size() * sizeof(float), b_wts);
    L.d_bias = (float*)put(L.bias_padded.data(), L.bias_padded.size() * sizeof(float), b_bias);
    L.d_desc_s = (uint32_t*)put(L.desc_s.data(), L.desc_s.size() * sizeof(uint32_t), b_desc_s);       // NULL when there are none
    L.d_wts_s = (float*)put(L.wts_s.data(), L.wts_s.size() * sizeof(float), b_wts_s);
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
