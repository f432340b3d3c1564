// Gradients of stage 4 on the matrix cores for the paper's head shape (bf16, 16 query heads per KV head,
// d_h = 128).  Same mathematics as attn_bwd.hip (chain rule on O = softmax(scale q K^T) V with the stored
// log-sum-exp; the paper prints no backward algorithm):
//     P = exp(z - lse),  dP = dO V^T,  dZ = P o (dP - Delta),  dQ = scale dZ K,  dK = scale dZ^T Q,  dV = P^T dO.
// Every product is an MFMA with the 16 heads of a token as one matrix dimension.
//   prep : (this file) -<dO, O> = -Delta and -lse / scale per (token, query head), token-major, into the caller's scratch;
//          both are the seeds of the products they are subtracted from
//   bits : (this file) the inverse of the block lists
//   dq   : the forward's tile kernel with another unit (TileKernel<.., BWD> in attn_mfma.hip, unit_bwd in attn_unit.h)
//   dkv  : attn_bwd_dkv.hip
// Measured at 32768 tokens, 64 selected blocks, 2 KV heads: dq 3.5 ms, dkv 5.1 ms (the forward attention kernel: 2.35 ms for
// 2/7 of their flops).  dq took 5.5 ms as a kernel of its own that walked the union one block per barrier with K, V and a
// transposed copy of K staged through registers.
#include "attn_bwd.h"
#include "launch_rules.h"

namespace ifv2 {

namespace {

constexpr int D = 128, G = 16;

// ------------------------------------------------------------------------------------------ pre-passes
__global__ void __launch_bounds__(256) bwd_prep_kernel(BwdM a) {
    // 16 threads per (token, query head): minus Delta = <dO, O> and minus lse / scale, both token-major; and the token's rows of
    // dK and dV cleared for the dK/dV kernel's adds (a launch less: 4.7 us of the call at 500
    // tokens; 11 us at 32768, where clearing beside the copy rate costs 8)
    const int row = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    (tid < D ? a.dk : a.dv)[((int64_t)h * a.map.total_rows + row) * D + (tid & (D - 1))] = 0.f;
    const int head = tid >> 4, d0 = (tid & 15) * 8;
    const int64_t off = ((int64_t)row * a.hq + h * G + head) * D + d0;
    const uint4 rg = *reinterpret_cast<const uint4 *>(a.dout + off);
    const uint4 ro = *reinterpret_cast<const uint4 *>(a.out + off);
    const uint32_t wg[4] = {rg.x, rg.y, rg.z, rg.w}, wo[4] = {ro.x, ro.y, ro.z, ro.w};
    float dot = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        dot += __uint_as_float(wg[e] << 16) * __uint_as_float(wo[e] << 16);
        dot += __uint_as_float(wg[e] & 0xffff0000u) * __uint_as_float(wo[e] & 0xffff0000u);
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) dot += __shfl_xor(dot, o);
    if ((tid & 15) == 0) {
        const int qh = h * G + head;
        a.ndelta[(int64_t)row * a.hq + qh] = -dot;
        a.nlse[(int64_t)row * a.hq + qh] = -a.lse[qhead_row(a.map, qh, a.hq, row)] / a.scale;
    }
}

// Inverse of the block lists: bit t of row j says that token t selected key block j.  The dK/dV kernel then gets
// the tokens of a (block, token chunk) pair with one short read instead of searching every token's list.
// One workgroup per 256 tokens of a sequence; a wavefront reads a token's list with one coalesced load (lane = list
// entry), eight of its 32 tokens requested at once.  The tile's eight words of every row are put together in LDS (rows nine
// words apart: the entries of a list are ascending blocks, which eight words apart would share eight banks) and stored
// whole: no atomics on memory, and nothing has to be cleared before (rows past the tile's last block are not written,
// which is why a reader of row j looks only at tokens from 64 j on).  Bound by the latency of the list reads: 26 us up to
// 2000 tokens and 37 at 32768, on 2 KV heads, with four wavefronts that read one list after the other, 6 and 9 now.
constexpr int BITS_TILE = 256, BITS_WORDS = BITS_TILE / 32, BITS_ROW = BITS_WORDS + 1, BITS_WAVES = 8;
constexpr size_t kBitsLdsMax = (size_t)262144 / kBlock * BITS_ROW * sizeof(uint32_t);       // longest sequence of this path
__global__ void __launch_bounds__(BITS_WAVES * 64) bwd_sel_bits_kernel(BwdM a) {
    extern __shared__ uint32_t bits[];                // [blocks up to the tile's last][BITS_ROW]
    __shared__ int s_tile[3];
    constexpr int NT = BITS_WAVES * 64, PER = BITS_TILE / BITS_WAVES, U = 8;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = blockIdx.y;
    int tile;
    const int seq = find_seq_tile(a.map.cu, a.map.batch, BITS_TILE, blockIdx.x, tile, s_tile);
    if (seq >= a.map.batch) return;
    const int tok0 = a.map.cu[seq], len = a.map.cu[seq + 1] - tok0;
    if (len < a.dense_below) return;                  // dense sequences need no lists
    const int words = (len + 31) / 32;
    const int n = (min(tile * BITS_TILE + BITS_TILE, len) - 1) / kBlock + 1;      // rows
    for (int i = tid; i < n * BITS_ROW; i += NT) bits[i] = 0u;
    __syncthreads();
    const int t_first = tile * BITS_TILE + w * PER, t_end = min(t_first + PER, len);
    const int32_t *lists = a.idx + head_row(a.map, h, tok0) * a.topk_total;
    for (int i = lane; i < a.topk_total; i += 64) {
        for (int t = t_first; t < t_end; t += U) {
            int j[U];
#pragma unroll
            for (int u = 0; u < U; ++u) j[u] = lists[(int64_t)min(t + u, t_end - 1) * a.topk_total + i];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int x = min(t + u, t_end - 1);  // (the last token again: the same bit)
                if (j[u] >= 0 && j[u] <= x / kBlock) atomicOr(&bits[j[u] * BITS_ROW + ((x >> 5) & (BITS_WORDS - 1))], 1u << (x & 31));
            }
        }
    }
    __syncthreads();
    uint32_t *rows = a.sel_bits + (int64_t)h * a.sel_words + sel_base(a.map, seq) + tile * BITS_WORDS;
    for (int i = tid; i < n * BITS_WORDS; i += NT)
        if (tile * BITS_WORDS + (i & (BITS_WORDS - 1)) < words)
            rows[(int64_t)(i / BITS_WORDS) * words + (i & (BITS_WORDS - 1))] = bits[i / BITS_WORDS * BITS_ROW + (i & (BITS_WORDS - 1))];
}

}  // namespace

bool bwd_mfma_params(const infllmv2_params *p) {
    return p->dtype == INFLLMV2_BF16 && p->head_dim == D && p->num_q_heads / p->num_kv_heads == G;
}

// two [rows, hq] float arrays (-lse / scale, -<dO, O>) and optionally the selection bitmap
size_t bwd_mfma_ws_bytes(const infllmv2_params *p, const BatchTotals &t, bool with_bitmap) {
    const size_t b_f = align256((size_t)t.rows * p->num_q_heads * sizeof(float));
    const size_t words = (size_t)(t.sel_words + 3) / 4 * 4;
    const size_t b_sel = with_bitmap ? align256((size_t)p->num_kv_heads * words * sizeof(uint32_t)) : 0;
    return 2 * b_f + b_sel;
}

// Returns INFLLMV2_ERR_UNSUPPORTED (nothing launched) for shapes this path does not cover.
int launch_attn_bwd_mfma(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx,
                         int dense_below, const void *out, const float *lse, const void *dout, void *dq, float *dk,
                         float *dv, const int32_t *cu_h) {
    const infllmv2_params *p = L.p;
    if (!bwd_mfma_params(p)) return INFLLMV2_ERR_UNSUPPORTED;
    if ((((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out | (uintptr_t)dout | (uintptr_t)dq) & 15) != 0 ||
        L.map.kv_tok_stride % 8 != 0 || L.map.kv_head_stride % 8 != 0)
        return INFLLMV2_ERR_UNSUPPORTED;
    const int64_t rows = L.map.total_rows;
    if (rows == 0) return INFLLMV2_OK;
    int64_t nblocks = 0;
    for (int s = 0; s < L.map.batch; ++s) nblocks += (cu_h[s + 1] - cu_h[s] + kBlock - 1) / kBlock;
    const int hkv = p->num_kv_heads, hq = p->num_q_heads;
    if (nblocks > 65535 || hkv > 65535 || rows > 0x7fffffff / 4) return INFLLMV2_ERR_UNSUPPORTED;
    // What follows is for sequences whose bitmap rows fit LDS and for token strides of which three, in bytes, fit 32 bits (a
    // card holds 500 tokens of the others); the rest takes the generic kernels.
    if (L.max_len > 262144 || L.map.kv_tok_stride >= (1 << 28)) return INFLLMV2_ERR_UNSUPPORTED;
    // (a launch has fewer than 2^32 threads in x; the dK/dV kernel's are 64 per workgroup)
    const int chunk = rules::dkv_chunk({cu_h, L.map.batch, L.max_len, hkv, nblocks, idx != nullptr, p->topk_total, dense_below},
                                       0xffffffffll / 64);
    if (chunk == 0) return INFLLMV2_ERR_UNSUPPORTED;
    const size_t b_f = align256((size_t)rows * hq * sizeof(float));
    // selection bitmap (block-major): only when block lists exist and it stays moderate (it grows with len^2 / 512
    // bytes per sequence and KV head: 32 MB at 128K tokens); otherwise the dK/dV kernel searches the lists
    int64_t sel_words = 0, sel_tiles = 0;
    if (idx != nullptr)
        for (int s = 0; s < L.map.batch; ++s) {
            const int64_t len = cu_h[s + 1] - cu_h[s];
            sel_words += ((len + kBlock - 1) / kBlock) * ((len + 31) / 32);
            sel_tiles += (len + BITS_TILE - 1) / BITS_TILE;
        }
    sel_words = (sel_words + 3) / 4 * 4;
    // the bitmap is built when the caller's workspace has room for it
    const size_t b_sel_full = align256((size_t)hkv * sel_words * sizeof(uint32_t));
    char *ws = (char *)L.ws;
    if (ws == nullptr || L.ws_bytes < 2 * b_f) return INFLLMV2_ERR_WORKSPACE_TOO_SMALL;
    const bool use_bits = idx != nullptr && sel_words > 0 && L.ws_bytes >= 2 * b_f + b_sel_full;
    BwdM a;
    a.q = (const uint16_t *)q;
    a.k = (const uint16_t *)k;
    a.v = (const uint16_t *)v;
    a.out = (const uint16_t *)out;
    a.dout = (const uint16_t *)dout;
    a.lse = lse;
    a.idx = idx;
    a.topk_total = p->topk_total;
    a.dense_below = dense_below;
    a.hq = hq;
    a.scale = p->softmax_scale;
    a.map = L.map;
    a.nlse = (float *)ws;
    a.ndelta = (float *)(ws + b_f);
    a.nblocks = nblocks;
    a.sel_bits = use_bits ? (uint32_t *)(ws + 2 * b_f) : nullptr;
    a.sel_words = sel_words;
    a.dq = (uint16_t *)dq;
    a.dk = dk;
    a.dv = dv;
    if (use_bits) {
        const size_t lds = (size_t)((L.max_len + kBlock - 1) / kBlock) * BITS_ROW * sizeof(uint32_t);
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(bwd_sel_bits_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kBitsLdsMax) != hipSuccess)
            return INFLLMV2_ERR_HIP;
        hipLaunchKernelGGL(bwd_sel_bits_kernel, dim3((unsigned)sel_tiles, hkv), dim3(BITS_WAVES * 64), lds, L.stream, a);
    }
    hipLaunchKernelGGL(bwd_prep_kernel, dim3((unsigned)rows, hkv), dim3(256), 0, L.stream, a);
    if (hipGetLastError() != hipSuccess) return INFLLMV2_ERR_HIP;
    const int rc = launch_bwd_dq(L, a, cu_h);
    if (rc != INFLLMV2_OK) return rc;
    return launch_bwd_dkv(a, chunk, L.max_len, L.stream);
}

}  // namespace ifv2
