// The (token chunk, KV block) pairs of a sequence with a token that can see the block, numbered chunk by chunk (attn_bwd.hip).
// Apart from the kernel so that the numbering can be run on the host as well.  Chunks have 1 << shift tokens, 32 to 256.
#pragma once
#include <math.h>

namespace ifv2 {

// pairs of the first q chunks, all of them whole: a chunk sees the blocks up to its last token's
__device__ inline int chunk_pairs(int q, int shift) {
    return shift == 5 ? (q + 1) / 2 * (q / 2 + 1) : (q * (q + 1) / 2) << (shift - 6);
}
// pairs of a sequence of n tokens
__device__ inline int sequence_pairs(int n, int shift) {
    const int q = n >> shift;
    return chunk_pairs(q, shift) + ((q << shift) < n ? (n + 63) / 64 : 0);
}
// chunk and block of the nth pair
__device__ inline void pair_at(int nth, int shift, int &chunk, int &block) {
    chunk = shift == 5 ? (int)(2.f * sqrtf((float)nth)) : (int)sqrtf((float)(nth >> (shift - 6)) * 2.f);
    while (chunk_pairs(chunk + 1, shift) <= nth) ++chunk;
    while (chunk_pairs(chunk, shift) > nth) --chunk;
    block = nth - chunk_pairs(chunk, shift);
}

}  // namespace ifv2
