// What the files of the backward share: attn_bwd.hip (any shape), attn_bwd_mfma.hip and attn_bwd_dkv.hip (matrix-core path).
#pragma once
#include "common.h"

namespace ifv2 {

// is block j in the ascending, -1 padded list e[0 .. n)?
__device__ inline bool list_has(const int32_t *e, int n, int j) {
    int lo = 0, hi = n;                      // first position whose entry is >= j (padding counts as +inf)
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const int x = e[mid];
        if (x >= 0 && x < j) lo = mid + 1; else hi = mid;
    }
    return lo < n && e[lo] == j;
}

// the matrix-core path's arguments
struct BwdM {
    const uint16_t *q, *k, *v, *out, *dout;
    const float *lse;
    const int32_t *idx;          // nullptr: dense
    int topk_total, dense_below, hq;
    float scale;
    RowMap map;
    // scratch
    float *nlse, *ndelta;        // [T][hq]: -lse / scale and -<dO, O>, the seeds of the products q k and dO v
    int64_t nblocks;             // 64-key blocks over all sequences
    uint32_t *sel_bits;          // [hkv][sel_words]: per sequence and key block, one bit per token that selected it
    int64_t sel_words;           //   (block-major, rows of ceil(len / 32) words); nullptr: not built (too large)
    // results
    uint16_t *dq;
    float *dk, *dv;
};

// Words of the selection bitmap before sequence seq, by a whole wavefront: 64 sequences per step (a walk of one after the other,
// which every wavefront of the bitmap kernel makes, took 6.3 of the 15.9 ms of a backward call for 5000 sequences of 20
// tokens).  Fewer than 2^31 in all: at most 65535 blocks of at most 8192 words.
__device__ inline int sel_base(const RowMap &m, int seq) {
    if (seq == 0) return 0;
    int w = 0;
    for (int s = (int)threadIdx.x & 63; s < seq; s += 64) {
        const int len = m.cu[s + 1] - m.cu[s];
        w += (len + kBlock - 1) / kBlock * ((len + 31) / 32);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) w += __shfl_xor(w, o);
    return __builtin_amdgcn_readfirstlane(w);
}

// dQ: the forward's tile kernel with another unit (attn_mfma.hip)
int launch_bwd_dq(const Launch &L, const BwdM &a, const int32_t *cu_h);
// dK, dV with `chunk` tokens per workgroup (attn_bwd_dkv.hip)
int launch_bwd_dkv(const BwdM &a, int chunk, int32_t max_len, hipStream_t stream);

}  // namespace ifv2
