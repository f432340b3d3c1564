// Which form of a kernel a call takes, where that depends on the lengths of a whole batch (host code, no HIP in it).
#pragma once
#include <stdint.h>

#include <algorithm>

namespace ifv2 {
namespace rules {

constexpr int kKeys = 64;         // keys of a selection block

// Workgroups of 256 threads that a launch holds in x, which has fewer than 2^32 threads.  Kernels with tiles and heads both in x reach that
// sooner than those with heads in y, which then serve the call.
constexpr int64_t kMostInX = 0xffffffffll / 256;

// Tiles of one and of two column groups (of `tokens` tokens) in a packed batch, and the half blocks (32 keys) that a tile walks
// on average: a causal walk, or as far as one token's budget goes (neighbouring tokens share most of their blocks).
struct Walks {
    int64_t one = 0, two = 0;
    double half_blocks = 0;
    double filled = 0;                // part of the tiles of one group that holds tokens
};
inline Walks walks(const int32_t *cu_h, int batch, int tokens, bool sparse, int topk, int dense_below) {
    Walks r;
    int64_t total = 0;
    for (int s = 0; s < batch; ++s) {
        const int n = cu_h[s + 1] - cu_h[s];
        total += n;
        const int64_t tiles = (n + (int64_t)tokens - 1) / tokens;
        const double far = (n + kKeys / 2.) / kKeys;
        r.one += tiles;
        r.two += (tiles + 1) / 2;
        r.half_blocks += tiles * (sparse && n >= dense_below ? std::min(far, 2. * topk) : far);
    }
    if (r.one > 0) r.half_blocks /= r.one;
    if (r.one > 0) r.filled = (double)total / ((double)r.one * tokens);
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
    // tokens (1500) 140 / 126.  (Calls of this size take the
    // staged form unless their rows are not 16-byte multiples.)  fp32 is bound by its products (d 64, 1200 tiles 84 / 88; d 128: the
    // registers do not suffice).
    if (bf16 && x.half_blocks >= 6 && x.one * hkv > (d == 128 ? 380 : 600))
        return {2, rows_ahead(x.two * hkv, d == 128 ? 512 : 1024, x)};
    return {1, rows_ahead(x.one * hkv, 1024, x)};
}
// fp32 attention is bound by its products: rows requested ahead are worth their registers only where a CU has no other workgroup's wavefronts to fill the
// waits with.  The chip holds, ahead / not, 512 / 768 workgroups at d 64 and 256 / 512 at d 128.  Walks of fewer than six (d 128: four) half blocks are over
// before a second request would arrive.  Attention alone, ahead / not, by workgroups:
// d 64: one a CU and a few: 4 heads on 1, 1000 tokens (250) 17.5 / 17.9 us, 1050 (263) 18.5 / 19.7, 1450 (363) 24.6 / 25.2, 2048 (512) 31.6 / 28.5, 8 on 2, 1000 (500)
// 28.0 / 25.4.
// d 128: one or two KV heads, 4 heads on 1, 1600 tokens (400) 55 / 60, 1255 + 347 (401) 35 / 45, 1800 (450) 61.3 / 61.5, 3500 tokens on 2 of their own (438)
// 91 / 107; 8 on 2, 800 (400) 27 / 28, 1000 (500) 36.7 / 34.5; just over 512 without is a second, nearly empty round: 1000 + 50 tokens (526) 39.4 / 49.8, 1100 (550) 45.7 / 52.9, 1200 (600) 47 / 49, 1300
// (650) 57 / 54.  More heads come one after the other beyond 512 and their longest tiles late, all the later in long rounds: 16 on 4, 900 tokens (900) 62 / 69, 1000
// (1000) 71 / 78, 4 on 4, 4000 (1000) 221 / 262; within one round without they share the CUs evenly: 8 on 8, 1000 (504) 58 / 35, 4 on 4, 1200 (300) 36 / 38,
// 1600 (400) 66 / 52; of three heads beyond 370: 3 on 3, dense, 1642 tokens (309) 39 / 47, 1765 (333) 48 / 58, 1962 (369) 60 / 65, 6 on 3, 834 (315) 26 / 30, 917 (345) 29 / 31, 1008
// (378) 1.14 of the time, but 4 on 4, 1290 (324) 1.04, 8 on 8, 640 (320) 1.2.
// Over 2015 calls, half of them near these lines, the rule is from the faster form in the mean 0.2 % (d 64) and 0.9 % (d 128), rows_ahead 4 % each.
inline bool fp32_rows_ahead(int d, int hkv, int64_t workgroups, const Walks &x) {
    const double hb = x.half_blocks;
    if (d == 64) return hb >= 6 && workgroups <= (hb >= 12 ? 300 : 256);
    if (hb < 4) return false;
    if (hkv > 2) return workgroups <= std::min(hkv == 3 && hb >= 12 ? 370. : 300., 40 * hb) || (hb >= 12 && workgroups > 600 && workgroups <= 1024);
    return workgroups <= std::min(512., 64 * hb) || (hb >= 12 && workgroups <= 600);
}
// Order of a generic attention launch's workgroups, which all take the tiles from the last one down: one head after the other (SIDE_BY_SIDE, the staged form: heads side by
// side), or, where all workgroups are on the chip at once, heads side by side and rows of 256 back and forth, so that long and short tiles share a CU.  fp32 d 64, one order / the other: 2048
// tokens, 4 heads on 1 (512 workgroups) 29.3 / 26.8 us, with 16 blocks 38.3 / 32.5, 1000 tokens on 2 (500) 25.7 / 19.9, 1500 (750) 34.7 / 31.3; with one
// workgroup per CU the second row would start shortest first (36.5 / 44.1).
//
// Walks of a packed batch do not fall from tile to tile, so there the fullest CU is counted for both orders: fp32 d 64, 2 heads on 1, dense, 2463 + 2040 + 68 tokens
// (572) 58.6 / 40.5 us but 2490 and 100 of one (412) 41.6 / 45.2, 16 blocks, 2675 + 10 x 100 (535) 29.8 / 35.2; d 128, 4 on 1, 4 blocks, 1217 + 10 x 43 (415) 20.8 /
// 23.9.  127 packed calls are 0.5 % from the faster order, 1.1 % with the second for all, six instead of fifteen of them 3 % and more slower than
// with the first.
// Staged form, bf16, plain / back and forth: d 128, 4 on 4, 16 blocks, 2389 + 434 + 509 tokens (420) 32.1 / 38.0, 4 on 1, dense, 2496 + 5 x 269 (482) 41.0 / 46.0; 652 packed calls 0.4 % from
// the faster order (0.9 % and 2.1 % with one order for all), eight instead of 63 of them 3 % and more slower than with the plain one.
// Where walks are shorter than four half blocks the call is over before the count on the host pays (2 us: 500 sequences of 4 tokens 9.1 -> 12.0 us).
// tiles: launched, of `tokens` tokens (the sequences' partial ones may be fewer: empty ones come first); resident: workgroups that the chip holds.  cu_h: nullptr
// where a tile is a token of its own.
inline bool back_and_forth(const int32_t *cu_h, int batch, int tokens, int64_t tiles, int hkv, bool sparse, int topk, int dense_below, double half_blocks,
                           int resident, bool side_by_side) {
    const int64_t workgroups = tiles * hkv;
    if (workgroups <= 256 || workgroups > resident || resident > 1024) return false;
    if (cu_h == nullptr || batch == 1 || half_blocks < 4) return true;
    const int n = (int)workgroups;
    int work[1024];                                          // half blocks of the launch's nth tile, and a start and an end worth four
    int nth = (int)tiles;
    for (int s = 0; s < batch; ++s) {
        const int len = cu_h[s + 1] - cu_h[s], most = sparse && len >= dense_below ? 2 * topk : len;
        for (int t = 0; t < len && nth > 0; t += tokens) work[--nth] = 4 + std::min((std::min(t + tokens, len) + kKeys / 2 - 1) / (kKeys / 2), most);
    }
    while (nth > 0) work[--nth] = 0;
    int straight[256] = {}, back[256] = {};
    int b = 0, e = 0;
    for (int h = 0; h < hkv && !side_by_side; ++h)
        for (int t = 0; t < (int)tiles; ++t) straight[b++ & 255] += work[t];
    for (int t = 0; t < (int)tiles; ++t)
        for (int h = 0; h < hkv; ++h, ++e) {
            if (side_by_side) straight[e & 255] += work[t];
            const int row = e & ~255, last = std::min(255, n - 1 - row), at = e - row;
            back[e & 256 ? last - at : at] += work[t];
        }
    return *std::max_element(back, back + 256) < *std::max_element(straight, straight + 256);
}

// bf16 attention and dQ with tiles of two groups whose V (dQ: K) rows pass through LDS (attn_staged.hip): a step is shorter, but a
// workgroup takes 3 us longer to start and to end, so not where few of them leave the chip idle and each has few steps.  Calls by
// workgroups (tiles of two groups times KV heads), generic / staged.  Attention d 128, 8 heads on 2: 720 tokens (180) 13.6 / 16.6 us, 1020 (255)
// 19.6 / 19.3, 1200 (300) 21.4 / 22.2, 1520 (380) 27.3 / 25.0, 2080 (520) 40.0 / 33.3, 7000 268 / 236; 28 on 4, 330 tokens 11.0 / 13.2, 380 18.2 / 13.4;
// 40 x 100 tokens (1040, walks of two half blocks) 22.2 / 23.9.  d 64 (the generic form takes two groups beyond 300, for walks of six): 1200
// tokens (300) 13.2 / 16.2, 1320 (330) 17.1 / 16.7, 2080 25.2 / 19.7; 28 on 4, 330 tokens (walks of five) 8.3 / 9.5; 8 x 300 (608) 13.6 / 12.4, 40 x 100
// 13.6 / 13.9.  Backward d 128: 300 tokens (76) 27.7 / 30.3, 600 (150) 44.4 / 43.5, 6000 (1500) 519 / 399; 300 x 4 tokens, 28 heads on 4,
// 63.4 / 67.3; d 64, 1985 tokens 82 / 66.
//
// d 128, packed sequences with walks of less than five half blocks, staged / generic: 16 x 189, 4 heads on 1 (384) 12.3 / 10.7 us, 12 x 238 (360) 13.2 / 11.5, 234 + 121 + 216 +
// 177, 14 on 1 (375) 14.2 / 10.9, but 4 x 211 (424) 0.92 of the generic form's time, 4 x 224, 16 on 4 (448) 0.80, 12 x 192, 6 on 3 (432) 0.79; with longer walks 6 x 309 (360) 0.98.
//
// Where many tiles end with their sequences a second group is often empty, and short walks do not make up for it: attention d 128, 3000 tokens and
// 300 x 4, 4 blocks, 4 heads on 1 (675) 22.2 / 26.5, 1000 tokens and 300 x 4, 4 on 4 (1328) 27.7 / 33.8, but 3000 + 300 x 4 with every block 79 / 100 of the
// generic form's time; d 64, 1000 + 200 x 1, 4 on 1 (325) 11.3 / 14.4, on 2 with 4 blocks (650) 11.2 / 13.4, with every block 85 / 100.
// Backward, d 64, sequences that fill neither group: 4000 / hkv sequences, staged / generic: 1 token on 8 heads of their own 1.15, 4 tokens 1.09, 12 tokens 0.98; 4
// heads on 1, 1 token 1.11, 3 tokens 0.98, 4 tokens 0.94; 8 heads on 1, 1 token 0.88.
inline bool staged(bool bwd, int d, int64_t workgroups, const Walks &x) {
    if (workgroups > kMostInX) return false;
    const bool partial = 9 * x.two > 5 * x.one;
    if (bwd) return workgroups >= 150 && (d == 64 ? !(partial && x.filled < 0.45) : x.half_blocks >= 2);
    const double least = d == 128 ? 6 : workgroups <= 450 ? 10 : workgroups <= 1100 ? 6 : 0;
    if (partial && x.half_blocks < least) return false;
    if (d == 64) return workgroups > 300 && x.half_blocks >= (workgroups > 512 ? 3 : 6);
    return workgroups >= (x.half_blocks < 5 ? 400 : 340) && x.half_blocks >= 3;
}
// dQ reads K twice, so two groups pay earlier.  By tiles of one group times KV heads, one / two groups: bf16 d 128: 250 tiles 15.0 /
// 17.2 us, 300 20.0 / 18.8, 994 80 / 55; d 64: 400 17.7 / 16.1; fp32 d 64: 400 38 / 34, 800 74 / 58 (d 128: two groups need 54 registers
// more than there are).  Short walks are too little work per workgroup: whole call, 8 heads on 2, bf16 d 128: 500 x 4 tokens 49 / 63,
// 57 x 140 tokens (walks of 3 half blocks) 133 / 144, 40 x 200 172 / 180, 6 x 300 64 / 63, 8 x 1000 418 / 389; d 64: 800 x 10 tokens
// 97 / 102, 10 x 200 39.6 / 35.6.  Two groups without rows ahead are slower everywhere (d 128, 4000 tokens 394 / 432, 26 x 300 208 / 213).
inline GenericForm generic_dq_form(bool bf16, int d, int hkv, const Walks &x) {
    if ((bf16 || d == 64) && x.half_blocks >= (d == 128 ? 4 : 2) && x.one * hkv > (bf16 ? 280 : 350)) return {2, true};
    // (fp32 d 128 has one wavefront per SIMD either way: 28 heads on 4, 400 x 20 tokens, ahead / not 870 / 938)
    return {1, (!bf16 && d == 128) || rows_ahead(x.one * hkv, 1024, x)};
}

// Of one sequence and KV head, the workgroups that have tokens: chunks i of 32 << K tokens, blocks up to a chunk's last token.
// (Everything fits 32 bits for lengths below 2^20; a batch of thousands of sequences is counted for each call.)
template <int K>
inline uint32_t dkv_busy(uint32_t len) {
    const uint32_t q = len >> (5 + K), full = K > 0 ? (q * (q + 1) / 2) << (K > 0 ? K - 1 : 0) : (q + 1) / 2 * (q / 2 + 1);
    return full + (len & ((32u << K) - 1) ? (len + kKeys - 1) / kKeys : 0u);
}
// Generic dK/dV, bf16, d 64: 16 rows of Q and dO per step instead of 32 (bwd_dkv_kernel), whose workgroups are the smaller ones: where sequences have
// hardly more rows and there are many of them.  blocks: KV blocks of the batch times KV heads.  Whole backward, 32 / 16 rows, blocks of about 700 / 1500 / 4000:
// 4 heads on 1, 4 tokens 27.9 / 27.3, 54.9 / 51.4, 223 / 199 us, 12 tokens 41.8 / 41.6, 93.9 / 91.4, 371 / 348; 8 on 8, 8 tokens 20.2 / 19.6, 32.8 / 31.5,
// 89 / 81, 20 tokens 25.0 / 25.3, 44.4 / 46.6, 112 / 111; 16 on 1, 2 tokens 29.2 / 30.0, 61.3 / 61.8, 242 / 226.
inline bool dkv_short_steps(int d, int G, int max_len, int64_t blocks) { return d == 64 && max_len <= std::max(4, 16 / G) && blocks > 600; }

// Attention of short prompts (attn_short.hip; bf16, G = 16, d 128): wavefronts per token, or 0 where the tile kernel is faster.
//
// Tiles of four tokens read a block for fewer tokens than the tile kernel's, but their chain is shorter, which wins while a
// CU gets few of them.  Two wavefronts per token take a whole CU (128 KB of LDS): the choice while one round of workgroups is all there is,
// or one and a half where the rest are the short tiles of long walks; with one wavefront two workgroups share a CU.  Microseconds of the call,
// tile kernel / two / one, all of the present kernels (workgroups): 2 KV heads, 64 blocks, 300 tokens (150) 14.2 / 10.4 / 10.5, 600 (300) 20.4 / 15.0 / 16.5, 700 (350)
// 21.4 / 16.5 / 17.6, 777 (390) 23.7 / 19.4 / 19.9, 1000 (500) 27.0 / 24.0 / 23.6; 1 KV head, 1400 (350) 32.0 / 23.3 / 28.8, 1700 (425) 36.7 / 29.3 / 34.3, 2000
// (500) 41.5 / 35.9 / 40.0; 4 KV heads, 300 (300) 16.0 / 13.3 / 11.8, 500 (500) 19.4 / 18.1 / 15.1.
// Budgets that leave blocks out shorten the walks, so that the second round weighs more: 1 KV head, 16 blocks, 1700 tokens 32.8 / 29.5 / 33.7, 2000
// 35.4 / 36.1 / 37.9; 8 blocks, 1300 tokens (325) 24.7 / 20.5 / 24.6, 1700 26.8 / 28.6 / 26.0; 4 blocks, 1300 tokens 20.1 / 20.0 / 16.4; 2 KV
// heads, 8 blocks, 777 tokens (390) 22.3 / 19.3 / 19.5, 1000 24.2 / 24.1 / 22.4.
// One wavefront against the tile kernel: up to 600 tokens whatever the batch (tile kernel / one: 16 x 300 tokens on 2 53.8 / 47.2, 4 x 600 46.8 / 33.5, 500 x 10 169 /
// 48, 100 x 60 on 4 119 / 79); up to 1024 tokens while the tile kernel's time, which goes up by rounds of 256 tiles of 16, has had its
// step (3 x 900 on 1 35.6 / 27.6, on 2 51.6 / 46.2; 777 tokens on 4 32.8 / 25.0, 1000 39.4 / 34.5).
// The lines beyond 600 tokens were drawn when one wavefront took 250 registers; with 188 it is 6 to 9 % faster, and the tile kernel, which these
// calls keep, is no longer the faster one for 1024 to 1500 tokens on 2 KV heads (1200 tokens 30.4 / 27.0, 1400 33.7 / 30.6, 1500 36.3 / 34.5; 1700 42.9 / 43.0), for
// batches just over the lines (2 x 777 on 2 33.2 / 25.3, 4 x 777 55 / 47, 2 x 1024 41.2 / 36.1, 2 x 777 on 4 53.5 / 46.4; but 4 x 777 on 4 82 / 86, 3 x 900 78 / 82) and
// for small budgets (8 blocks, 777 tokens on 4 30.3 / 24.0).
// One sequence of 501 to 600 tokens on 2 KV heads has so few workgroups over one round that two are better: two / one, 520 tokens (260) 13.3 / 15.2, 600 (300) 15.0 /
// 16.5; but 4 x 300 on 2 (300) 22.2 / 16.1, 300 tokens on 4 (300) 13.3 / 11.8.
inline int short_attn_waves(const int32_t *cu_h, int batch, int max_len, int hkv, bool sparse, int topk, int dense_below) {
    int64_t wgs = 0, tiles16 = 0;
    for (int s = 0; s < batch; ++s) {
        wgs += (int64_t)((cu_h[s + 1] - cu_h[s] + 3) / 4) * hkv;
        tiles16 += (int64_t)((cu_h[s + 1] - cu_h[s] + 15) / 16) * hkv;
    }
    if (wgs > kMostInX) return 0;
    const int blocks = (max_len + kKeys - 1) / kKeys;
    const int walk = sparse && max_len >= dense_below ? std::min(topk, blocks) : blocks;
    const bool every = walk == blocks;
    if (wgs <= 256) return 2;
    if (wgs <= 512 && max_len > (batch == 1 && wgs <= 320 ? 500 : 600) && max_len <= 2048) {
        if (walk < 6) return 1;
        if (walk < 10 ? wgs <= 400 : every || max_len <= 1728) return 2;
    }
    if (max_len <= 600) return 1;
    const int64_t rounds = std::max<int64_t>((tiles16 - 16 + 255) / 256, 1);
    return max_len <= 1024 && rounds <= 2 && wgs <= (batch == 1 && every ? 1000 : 768) * rounds ? 1 : 0;
}

// Tile kernel of attention and dQ (bf16, G = 16, d 128): tokens per workgroup.
//
// Sixteen, or 8 or 4 while even those leave CUs without a workgroup (one fits a CU): a block in LDS then serves fewer tokens,
// but there is nobody else to serve, and an interval takes as long as its units.  (777 tokens, 2 KV heads: 28.9 us with 16,
// 20.7 with 8; dense, 1000 tokens: 36.4 and 27.4, 200 tokens 17.3 and, with 4, 13.5)
//
// A sequence of more than 1024 tokens that makes up most of the batch takes 8 up to two tiles for each CU: tiles start with the
// longest, so the CUs with the short ones of the first head take the long ones of the next.  16 / 8, dense or with 64 blocks, 2
// KV heads: 1400 tokens 44.4 / 33.0 us (dQ 71.0 / 45.8), 2040 tokens 62.6 / 55.1 (102 / 79), 2500 tokens 76.4 / 86.2 (125 /
// 119); 1 KV head: 2049 tokens 58.3 / 42.7, 3100 tokens 82.9 / 58.8, 4096 tokens 107 / 86.  Below 1024 a workgroup's start weighs more
// (500 tokens on 8 KV heads, whole call, 29.5 / 32.2).  Beside the long sequence, with 16 blocks: 1400 + 10 tokens on 2 KV heads
// 42.7 / 33.7, 1400 + 300 42.9 / 39.7, 1400 + 600 44.4 / 44.2, 2 x 1024 41.5 / 45.2; 1200 + 2800 on 1 55.0 / 57.7.
// Budgets cut the long tiles down to one length, and those behind the first 256 then begin when all of these end: they pay
// while they have few blocks themselves.  Attention, 1 KV head (4096 tokens: 32 such blocks): 16 blocks, 2800 tokens 54.0 / 43.7, 3400
// 57.5 / 57.9, 4096 63.5 / 68.5; 8 blocks, 2800 tokens 41.7 / 40.2, 3600 46.6 / 48.7; 2 KV heads (2048 tokens: 16): 4 blocks, 1200
// tokens 27.7 / 26.0, 1400 29.3 / 30.1, 12 blocks, 1600 41.0 / 38.5, 2040 46.6 / 48.8.  dQ, which does more for a block, gains there too (16
// blocks, 1 KV head, 4096 tokens, whole backward 283 / 229).
inline int attn_tile_tokens(const int32_t *cu_h, int batch, int max_len, int hkv, bool sparse, int topk, int dense_below, bool bwd) {
    const int64_t cus = 256 / hkv;
    int64_t tiles4 = 0, tiles8 = 0;
    for (int s = 0; s < batch; ++s) {
        tiles4 += (cu_h[s + 1] - cu_h[s] + 3) / 4;
        tiles8 += (cu_h[s + 1] - cu_h[s] + 7) / 8;
    }
    if (tiles4 <= cus) return 4;
    if (tiles8 <= cus) return 8;
    const int64_t total = batch > 0 ? cu_h[batch] - cu_h[0] : 0;
    if (tiles8 > 2 * cus || max_len <= 1024 || 4 * (int64_t)max_len < 3 * total) return 16;
    const bool budget = !bwd && sparse && max_len >= dense_below;
    return budget && (max_len + kKeys - 1) / kKeys - 8 * cus / kKeys > topk * 3 / 4 + cus * 3 / kKeys - 4 ? 16 : 8;
}

// dK/dV of the matrix-core path: tokens per workgroup, 32 to 1024.
//
// Every sequence gets the chunks of the longest, and its workgroups go round the eight XCDs (see attn_bwd_dkv.hip): this many
// are launched, most of the short sequences' to leave at once.
inline int64_t dkv_workgroups(int max_len, int hkv, int64_t nblocks, int chunk) {
    const int64_t groups = ((int64_t)max_len + chunk - 1) / chunk * hkv;
    return 8 * ((groups + 7) / 8) * nblocks;
}
struct DkvBatch {
    const int32_t *cu_h;
    int batch, max_len, hkv;
    int64_t nblocks;
    bool sparse;
    int topk, dense_below;
};
// The cheapest chunk by a model of the launch, in microseconds: a workgroup takes 33 for its keys and its adds (every chunk of a
// block adds to the same rows) and 1.9 per pair of tokens (down to 1.05 while SIMDs are idle), on the 128 SIMDs of each XCD, of
// which the one that has most of them counts while there are few; where they go round more than once, 0.45 of the longest
// list for the end; and one that leaves at once 3, more where it looks for its sequence among many.
// From the backward call with every chunk at 629 shapes (1 to 8 KV heads, 40 to 24000 tokens, dense, budgets of 16 to 96
// blocks, packed batches of up to 5000 sequences; profiles/backward_chunk_timings.txt): the one the model prefers is 0.9 % from
// the best on average, more than 5 % at 43 of them and 22 % at most (1300 tokens beside four sequences of 50 to 80). One sequence on 2 KV heads, training step with 32 /
// 64 / 128 / 256 / 512: 500 tokens 87 / 114 / 168 / 276 / 486 us, 1500 tokens 283 / 235 / 270 / 370 / 581, 3000 tokens 580 / 539 / 551 /
// 499 / 716, 8000 tokens 2.63 / 2.09 / 2.04 / 2.07 / 2.15 ms, 32768 tokens - / - / 12.5 / 11.15 / 11.0, with 1024 10.94; backward of
// 100 x 300 tokens 884 / 812 / 814 / 876 / 867, on 4 KV heads 1658 / 1481 / 1403 / 1555 / 1564.
// 0: no chunk makes a launch of at most `most` workgroups.
inline int dkv_chunk(const DkvBatch &b, int64_t most) {
    constexpr int N = 6;
    constexpr double kPair = 1.9, kIdlePair = 0.55, kFixed = 33, kTail = 0.45, kLeave = 3;
    int64_t busy[N] = {};                                   // by the chunk's size, 32 first
    double entries = 0;                                     // of the lists: every block up to the token's own, or the budget
    for (int s = 0; s < b.batch; ++s) {
        const uint32_t len = (uint32_t)(b.cu_h[s + 1] - b.cu_h[s]);
        const uint32_t most_of = b.sparse && (int)len >= b.dense_below ? (uint32_t)b.topk : ~0u;
        const uint32_t full = std::min(len / kKeys, most_of);
        busy[0] += dkv_busy<0>(len);
        busy[1] += dkv_busy<1>(len);
        busy[2] += dkv_busy<2>(len);
        busy[3] += dkv_busy<3>(len);
        busy[4] += dkv_busy<4>(len);
        busy[5] += dkv_busy<5>(len);
        entries += (double)kKeys * (full * (full + 1) / 2) + (double)(len - kKeys * full) * std::min(full + 1, most_of);
    }
    int chunk = 0;
    double best = 0;
    for (int i = N - 1; i >= 0; --i) {
        const int c = 32 << i;
        const int64_t launched = dkv_workgroups(b.max_len, b.hkv, b.nblocks, c);
        if (launched > most) break;
        const double wgs = (double)busy[i] * b.hkv;
        double load = wgs;
        const int64_t groups = ((int64_t)b.max_len + c - 1) / c * b.hkv;
        if (groups * b.batch <= 512) {                      // which XCD a workgroup is on matters while there are few
            double xcd[8] = {};
            for (int s = 0; s < b.batch; ++s) {
                const int64_t len = b.cu_h[s + 1] - b.cu_h[s];
                for (int64_t g = 0; g < groups && g / b.hkv * c < len; ++g)
                    xcd[(g - s - (s >> 3)) & 7] += (double)((std::min(g / b.hkv * c + c, len) - 1) / kKeys + 1);
            }
            load = 8 * *std::max_element(xcd, xcd + 8);
        }
        const double rounds = load / 1024, pair = kPair * (rounds < 1 ? kIdlePair + (1 - kIdlePair) * rounds : 1);
        const double longest = std::min(c, b.max_len) * pair / 2 + kFixed, mean = wgs > 0 ? entries * b.hkv / wgs * pair / 2 + kFixed : 0;
        const double cost = (rounds <= 1 ? longest : std::max(longest, rounds * mean + kTail * longest)) +
                            (launched - wgs) / 1024 * kLeave * (1 + b.batch / 128.);
        if (chunk == 0 || cost <= best) { best = cost; chunk = c; }
    }
    return chunk;
}

// Generic dK/dV: tokens per workgroup, 1 << the result, and the workgroups per KV head that this makes.
//
// The cheapest of 32 to 256 by a model of the launch, in steps (32 or 16 rows: as many tokens of G heads as that): a workgroup takes a fixed
// time for its list, its keys and its adds, and its tokens' steps, of which the last is half empty; while all workgroups run at once
// the longest counts, then the rounds of the average one and part of the longest.  From the backward call with every chunk at 8000 forms
// (60 to 6000 tokens, packed mixtures of up to 2000 sequences, 1 to 8 KV heads, groups of 1 to 16, budgets of 4 to 32 blocks and dense) the chosen chunk
// is from the best on average / at the worst hundredth: bf16 d 128 0.5 / 8 %, d 64 0.5 / 8 %, fp32 0.4 / 7 and 0.4 / 8 % (with one set of constants for all
// groups 1.8 / 20, 1.2 / 16, 0.9 / 13 and 0.9 / 12; profiles/generic_backward_chunk_timings.txt).  Whole backward, chunks of 32 / 64 / 128 / 256: bf16, 8 heads on 2, d 128, 16
// blocks, 346 tokens 30 / 35 / 48 / 75 us, 873 tokens 59 / 53 / 62 / 91, 1971 tokens 146 / 106 / 90 / 108; 2 heads on 1, 4 blocks, 2795 + 1317 + 794 + 648 tokens 93 / 75 / 70 / 74; fp32,
// d 128, 2 on 1, 4 blocks, 1558 tokens 61 / 77 / 82 / 123, 8 on 1, 5531 tokens 478 / 461 / 546 / 731.
inline int generic_dkv_shift(bool bf16, int d, int G, const DkvBatch &b, int64_t &pairs) {
    // a workgroup's fixed time, what the average one takes beyond its tokens' steps, workgroups in a round, the part of the longest
    struct Model { double fixed, end, slots, tail; };
    // by heads of a group: one, two, up to four, more
    static const Model fp32_64[4] = {{2.5, 0.5, 448, 0.3}, {1, 2, 640, 0.5}, {2.5, 0.5, 768, 0.7}, {1, 0, 512, 0.3}};
    static const Model fp32_128[4] = {{1, 2, 384, 0.2}, {2, 1, 512, 0.5}, {1.5, 2, 512, 0.7}, {1, 0.5, 512, 0.5}};
    static const Model bf16_64[4] = {{1, 0, 160, 0.3}, {1, 0, 192, 0.2}, {1, 3, 512, 0.3}, {2.5, 2, 640, 0.5}};
    static const Model bf16_128[4] = {{1.5, 0.5, 128, 0.3}, {1, 1, 160, 0.3}, {2, 3, 384, 0.3}, {2, 3, 512, 0.5}};
    const Model c = (bf16 ? d == 64 ? bf16_64 : bf16_128 : d == 64 ? fp32_64 : fp32_128)[G <= 2 ? G - 1 : G <= 4 ? 2 : 3];
    const double tokens = 16 / G * (bf16 ? 2 : 1);
    int64_t busy[4] = {};                                   // by the chunk's size, 32 first
    double entries = 0;
    for (int s = 0; s < b.batch; ++s) {
        const uint32_t len = (uint32_t)(b.cu_h[s + 1] - b.cu_h[s]);
        const uint32_t most_of = b.sparse && (int)len >= b.dense_below ? (uint32_t)b.topk : ~0u;
        const uint32_t full = std::min(len / kKeys, most_of);
        busy[0] += dkv_busy<0>(len);
        busy[1] += dkv_busy<1>(len);
        busy[2] += dkv_busy<2>(len);
        busy[3] += dkv_busy<3>(len);
        entries += (double)kKeys * ((double)full * (full + 1) / 2) + (double)(len - kKeys * full) * std::min(full + 1, most_of);
    }
    int best_i = 3;
    double best = 0;
    for (int i = 3; i >= (b.max_len < 1 << 20 ? 0 : 3); --i) {     // (the counts fit 32 bits)
        const double wgs = (double)busy[i] * b.hkv, rounds = wgs / c.slots;
        const double longest = c.fixed + std::min(32 << i, b.max_len) / tokens, mean = c.fixed + (wgs > 0 ? entries * b.hkv / wgs / tokens : 0) + c.end;
        const double cost = rounds <= 1 ? longest : std::max(longest, rounds * mean + c.tail * longest);
        if (i == 3 || cost < best) { best = cost; best_i = i; }
    }
    pairs = busy[best_i];
    return 5 + best_i;
}

// Decode behind the selection kernel: blocks per attend workgroup (of `waves` wavefronts, which take them in rounds) and workgroups per pair.  entries: blocks of
// the longest list.  Rounds are counted in a lane's number and dense sequences may be long: kDecodeRounds at most.
//
// As many workgroups as leave one for every CU make one round of them, with the fewest partial results to merge; two for each of more than 512 pairs.  Where that
// leaves CUs empty, or a few workgroups for a second round, another split whose fullest CU has a tenth fewer rounds (and half a round for each
// workgroup's start and end) is faster.  Step of that many pairs of 55 blocks with 1 / 2 / 3 / 4 / 6 workgroups each (* the old rule, ** this one): 66 85 73 69 70** 72
// us; 96 98 79*  ** 91 86 80; 130 113* 116 106** 111 108; 160 119* 125 118** 123 124; 192 134* ** 139 141 139 139; 264 207* 190 186** 186 183; 320 221* 208 209**
// 209 211; 400 247* ** 254 250 255 253; 512 292* ** 294 305 305 308.  Over 76 batches it is 0.2 % from the best (the old rule 1.2 %).
constexpr int kDecodeRounds = 16;
struct DecodeSplits {
    int bpw, nsplit;
};
inline DecodeSplits decode_splits(int64_t pairs, int entries, int waves) {
    const int64_t groups = (entries + waves - 1) / waves, least = std::max<int64_t>((groups + kDecodeRounds - 1) / kDecodeRounds, 1);
    auto cost = [&](int64_t ns) { return (double)((pairs * ns + 255) / 256 * ((groups + ns - 1) / ns)) + pairs * ns / 512.; };
    int64_t ns = std::max<int64_t>(pairs > 512 ? 2 : 256 / std::max<int64_t>(pairs, 1), least);
    double best = 0.9 * cost(ns);
    for (int64_t n = least; n <= std::min<int64_t>(4, groups); ++n)
        if (cost(n) < best) { best = cost(n); ns = n; }
    const int64_t bpw = std::max<int64_t>((groups + ns - 1) / ns, 1) * waves;
    return {(int)bpw, (int)std::max<int64_t>((entries + bpw - 1) / bpw, 1)};
}

}  // namespace rules
}  // namespace ifv2
