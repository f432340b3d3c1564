// Which form of a kernel a call takes, where that depends on the lengths of a whole batch (host code, no HIP in it).
#pragma once
#include <stdint.h>

#include <algorithm>

namespace ifv2 {
namespace rules {

constexpr int kKeys = 64;         // keys of a selection block

// Tiles of one and of two column groups (of `tokens` tokens) in a packed batch, and the half blocks (32 keys) that a tile walks
// on average: a causal walk, or as far as one token's budget goes (neighbouring tokens share most of their blocks).
struct Walks {
    int64_t one = 0, two = 0;
    double half_blocks = 0;
};
inline Walks walks(const int32_t *cu_h, int batch, int tokens, bool sparse, int topk, int dense_below) {
    Walks r;
    for (int s = 0; s < batch; ++s) {
        const int n = cu_h[s + 1] - cu_h[s];
        const int64_t tiles = (n + (int64_t)tokens - 1) / tokens;
        const double far = (n + kKeys / 2.) / kKeys;
        r.one += tiles;
        r.two += (tiles + 1) / 2;
        r.half_blocks += tiles * (sparse && n >= dense_below ? std::min(far, 2. * topk) : far);
    }
    if (r.one > 0) r.half_blocks /= r.one;
    return r;
}

// Generic attention and dQ: column groups per wavefront, and whether a wavefront requests the next half block's rows ahead.
//
// Rows requested ahead shorten a wavefront's walk, but their registers leave a SIMD one wavefront fewer: worth it while the
// 256 CUs go round fewer times than one of a tile's four wavefronts has half blocks.  fp32 attention, 8 heads on 2, d 128, ahead /
// not: 600 tokens 20.0 / 25.1 us, 1000 tokens 35.5 / 49.8, 11 x 700 105 / 90, 80 x 100 51 / 41, 2000 x 4 191 / 137; whole backward
// call, bf16, 8 heads on 2: d 128, 114 x 70 tokens 121 / 110, 500 x 4 53 / 49; d 64, 2000 x 4 223 / 196.
struct GenericForm {
    int groups;
    bool ahead;
};
inline bool rows_ahead(int64_t workgroups, int most, const Walks &x) {
    return workgroups <= std::min(256. / 4 * x.half_blocks, (double)most);
}
inline GenericForm generic_form(bool bf16, int d, int hkv, const Walks &x) {
    // Two column groups: a K or V row read (and a V row spread) serves twice the columns, for half as many wavefronts; worth it
    // for walks of several half blocks.  bf16, 8 heads on 2, d 128, one / two groups: 600 tokens (300 tiles times KV heads) 12.0 /
    // 13.8 us, 1000 tokens (500) 22.3 / 18.4, 4000 tokens 127 / 95, 80 x 100 tokens 36.6 / 38.8, 500 x 4 17.5 / 20.1; d 64: 1000
    // tokens 14.8 / 14.9, 1300 tokens 19.0 / 18.7.  Two groups with rows ahead / without, d 128: 1700 tokens (426 workgroups) 31 /
    // 39, 2000 tokens (500) 38.8 / 47.7, 2500 tokens (626) 59 / 56, 4000 tokens (1000) 118 / 95; d 64: 4000 tokens 65 / 70, 6000
    // tokens (1500) 140 / 126.  fp32 is bound by its products (d 64, 1200 tiles 84 / 88; d 128: the registers do not suffice).
    if (bf16 && x.half_blocks >= 6 && x.one * hkv > (d == 128 ? 380 : 600))
        return {2, rows_ahead(x.two * hkv, d == 128 ? 512 : 1024, x)};
    return {1, rows_ahead(x.one * hkv, 1024, x)};
}
// dQ reads K twice, so two groups pay earlier.  By tiles of one group times KV heads, one / two groups: bf16 d 128: 250 tiles 15.0 /
// 17.2 us, 300 20.0 / 18.8, 994 80 / 55; d 64: 400 17.7 / 16.1; fp32 d 64: 400 38 / 34, 800 74 / 58 (d 128: two groups need 54 registers
// more than there are).  Short walks are too little work per workgroup: whole call, 8 heads on 2, bf16 d 128: 500 x 4 tokens 49 / 63,
// 57 x 140 tokens (walks of 3 half blocks) 133 / 144, 40 x 200 172 / 180, 6 x 300 64 / 63, 8 x 1000 418 / 389; d 64: 800 x 10 tokens
// 97 / 102, 10 x 200 39.6 / 35.6.  Two groups without rows ahead are slower everywhere (d 128, 4000 tokens 394 / 432, 26 x 300 208 / 213).
inline GenericForm generic_dq_form(bool bf16, int d, int hkv, const Walks &x) {
    if ((bf16 || d == 64) && x.half_blocks >= (d == 128 ? 4 : 2) && x.one * hkv > (bf16 ? 280 : 350)) return {2, true};
    return {1, rows_ahead(x.one * hkv, 1024, x)};
}

// Generic dK/dV: tokens per workgroup, and groups of 16 rows of Q and dO per step.
struct DkvForm {
    int chunk, row_groups;
};
inline DkvForm generic_dkv_form(bool bf16, int d, int hkv, int G, const int32_t *cu_h, int batch, bool sparse, int topk, int dense_below) {
    const int step = 16 / G * (bf16 ? 2 : 1);               // tokens
    int64_t nblocks = 0;
    int max_len = 0;
    for (int s = 0; s < batch; ++s) {
        const int len = cu_h[s + 1] - cu_h[s];
        nblocks += (len + kKeys - 1) / kKeys;
        max_len = std::max(max_len, len);
    }
    auto busy = [&](int c) {                                // workgroups whose chunk does not end before their block (causal)
        int64_t n = 0;
        for (int s = 0; s < batch; ++s) {
            const int64_t len = cu_h[s + 1] - cu_h[s], nb = (len + kKeys - 1) / kKeys;
            n += (len + c - 1) / c * (nb + std::max<int64_t>(std::min<int64_t>(c / kKeys, nb), 1)) / 2 * hkv;
        }
        return n;
    };
    int chunk = 256;
    if (d == 128 && (!sparse || max_len < dense_below || (max_len + kKeys - 1) / kKeys <= topk)) {
        // Every block is selected.  As many tokens as leave 256 workgroups with work, not more than a third of the longest sequence
        // (its last chunk is short) where that is several steps.  Whole backward, bf16, 8 heads on 2, chunks of 256 / 128 / 64 / 32:
        // 300 tokens 92 / 56 / 38 / 30 us, 1000 tokens 116 / 80 / 70 / 81, 1985 tokens 166 / 173 / 193 / 200, 2500 tokens 224 / 235 / 269 /
        // 330, 26 x 300 tokens 201 / 186 / 177 / 211.
        // 512 to 768 workgroups of 256 are a little more than the two rounds of 256 that the chip takes at once: 3000 tokens (612)
        // 1.07 / 1 / 1.16 / 1.41, 4000 tokens (1072) 1.02 / 1.06 / 1 / 1.22 of the best.  Steps of less than 8 tokens make twice the
        // steps of a chunk: 16 heads on 2, 2300 tokens 348 / 339 / 321 / 358, fp32, 8 heads on 2, 2300 tokens 1.06 / 1.06 / 1 / 1.10.
        const int most = std::max(max_len / 3, 8 * step);
        while (chunk > 64 && (chunk > most || busy(chunk) < 256)) chunk /= 2;
        if (chunk == 256 && step <= 8 && busy(chunk) <= 768) {
            if (busy(chunk) > 512) chunk = 128;
            else if (step < 8) chunk = 64;
        }
    } else {
        // Lists that leave blocks out, whose workgroups differ more, and the smaller workgroups of d 64 are better shorter: 1985 bf16
        // tokens with 16 blocks each 167 us with 256 tokens, 160 with 64; d 64, 1400 fp32 tokens 221 / 176 / 154 / 165.
        while (chunk > 64 && nblocks * ((max_len + chunk - 1) / chunk) * hkv < 2048) chunk /= 2;
    }
    // Below 256 workgroups chunks of 32; where those are one or two steps (groups of one or two heads), below 160.  64 / 32: 8 heads on
    // 2, bf16: 300 tokens 38 / 30 us, 6 x 300 tokens (180 workgroups) 1.05 / 1; fp32, 900 tokens (240) 1.21 / 1; 4 heads on 4, bf16:
    // 150 tokens 25 / 23 us, 600 tokens (220) 38 / 45, 40 x 100 tokens, d 64 (240) 29 / 32; fp32: 300 tokens (60) 1.04 / 1, 600
    // tokens (220) 1 / 1.06.
    if (chunk == 64 && busy(chunk) < (step >= 16 ? 160 : 256)) chunk = 32;
    // Two groups of 16 rows in one contraction halve the products of bf16 rows, but at d 64 they cost a wavefront per SIMD, which many
    // workgroups with few steps each feel more.  Whole backward, 8 heads on 2, d 64, two groups / one: 500 x 4 tokens 38.9 / 33.6 us,
    // 26 x 300 107 / 97, 114 x 70 99 / 89; 4 x 700 (528 workgroups) 75 / 78, 16 heads on 2 112 / 122; 1300 tokens 8 heads on 1 62 / 68.
    const bool one = !bf16 || (d == 64 && std::min(chunk, max_len) <= 64 && busy(chunk) > 600);
    return {chunk, one ? 1 : 2};
}

}  // namespace rules
}  // namespace ifv2
