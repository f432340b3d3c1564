// Stage 1: mean-pooled compressed keys, K^{C1}_i = Mean(K[i*s : i*s + l])  (Sec. 3.3, Eq. 3).
// HBM-bound for long sequences (every K element is needed by l/s (= 2) windows; the second use hits L2), bound by one
// trip to memory for short ones and for a decode step's new rows: a thread requests sixteen window rows at once.  The
// additions stay in the order of the window, so that a row's value does not depend on the call that makes it.
// Measured: 131072 tokens 26.6 (+ 4.5 for a prefix-sum kernel of its own) -> 20.5 us, 777 tokens 8.4 (+ 4) -> 4.9 us; new
// rows of a decode step 11.8 -> 5.4 us at batch 16, 16.8 -> 6.3 us at batch 128 (16-thread workgroups that walked the
// window a row at a time before).
#include "gen_unit.h"

namespace ifv2 {

namespace {

constexpr int VEC = 8;            // channels per thread

// sum over a window of lc rows (tok_stride elements apart) of this thread's VEC channels, in row order
template <typename T>
__device__ inline void window_sum(const T *src, int64_t tok_stride, int lc, float (&acc)[VEC]) {
    constexpr int U = 16;
    typedef typename std::conditional<sizeof(T) == 2, gen::u16x8_u, gen::f32x8_u>::type Vec;
#pragma unroll
    for (int c = 0; c < VEC; ++c) acc[c] = 0.f;
    for (int u0 = 0; u0 < lc; u0 += U) {
        Vec x[U];
#pragma unroll
        for (int i = 0; i < U; ++i) x[i] = *reinterpret_cast<const Vec *>(src + (int64_t)min(u0 + i, lc - 1) * tok_stride);
        __builtin_amdgcn_sched_barrier(0);       // (left alone, the scheduler trades the requests for registers)
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int c = 0; c < VEC; ++c) {
                float y;
                if constexpr (sizeof(T) == 2) y = bf16_to_float(x[i][c]);
                else y = x[i][c];
                acc[c] += u0 + i < lc ? y : 0.f;
            }
    }
}

template <typename T, int D>
__global__ void __launch_bounds__(256)
compress_k_kernel(const T *__restrict__ k, RowMap map, int lc, int sc, float *__restrict__ kc, int32_t *__restrict__ cu_c) {
    constexpr int VPR = D / VEC;                               // threads per row: whole rows per wave, coalesced
    const int rows = (int)blockDim.x / VPR;                    // compressed rows per workgroup, of one sequence
    __shared__ int s_tile[3];
    const int h = blockIdx.y, tid = threadIdx.x;
    // the prefix sums of the per-sequence counts, by one workgroup (nobody here reads them)
    if (blockIdx.x == 0 && h == 0 && tid < 64) {
        int sum = 0;
        if (tid == 0) cu_c[0] = 0;
        for (int s0 = 0; s0 < map.batch; s0 += 64) {
            const int s = s0 + tid;
            int n = s < map.batch ? num_cmp(map.cu[s + 1] - map.cu[s], lc, sc) : 0;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int up = __shfl_up(n, o);
                if (tid >= o) n += up;
            }
            if (s < map.batch) cu_c[s + 1] = sum + n;
            sum += __shfl(n, 63);
        }
    }
    if (map.total_rows == 0) return;
    int tile, before;
    const int seq = find_seq_count(map.cu, map.batch, blockIdx.x, tile, before, s_tile,
                                   [&](int n) { return (num_cmp(n, lc, sc) + rows - 1) / rows; },
                                   [&](int n) { return num_cmp(n, lc, sc); });
    if (seq >= map.batch) return;
    const int tok0 = map.cu[seq], i = tile * rows + tid / VPR, c0 = (tid % VPR) * VEC;
    if (i >= num_cmp(map.cu[seq + 1] - tok0, lc, sc)) return;
    float acc[VEC];
    window_sum(k + (int64_t)h * map.kv_head_stride + ((int64_t)tok0 + (int64_t)i * sc) * map.kv_tok_stride + c0,
               map.kv_tok_stride, lc, acc);
    const float inv = 1.0f / (float)lc;
#pragma unroll
    for (int c = 0; c < VEC; ++c) acc[c] *= inv;
    gen::store_row<float, VEC>(kc + ((int64_t)h * map.kc_total_c + before + i) * D + c0, acc);
}

template <typename T, int D>
int launch_t(const Launch &L, const void *k, float *kc, int32_t *cu_c, const int32_t *cu_h) {
    // 256 threads per workgroup, or 64 while that leaves CUs without one (64 / 256 threads on 2 KV heads: 777 tokens 4.9 / 5.1
    // us, 8000 tokens 5.0 / 5.4, 65000 tokens 12.8 / 11.9)
    const int lc = L.p->cmp_len, sc = L.p->cmp_stride;
    int threads = 256;
    int64_t tiles = 0;
    for (;;) {
        const int rows = threads / (D / VEC);
        tiles = 0;
        for (int s = 0; s < L.map.batch; ++s) tiles += (num_cmp(cu_h[s + 1] - cu_h[s], lc, sc) + rows - 1) / rows;
        if (threads == 64 || tiles * L.p->num_kv_heads >= 256) break;
        threads = 64;
    }
    dim3 grid((unsigned)(tiles > 0 ? tiles : 1), L.p->num_kv_heads);
    hipLaunchKernelGGL((compress_k_kernel<T, D>), grid, dim3(threads), 0, L.stream, (const T *)k, L.map, lc, sc, kc, cu_c);
    return hip_status(hipGetLastError());
}

// Compressed keys that became complete while a cached sequence grew from prev[b] to ctx[b] tokens: rows
// nc(prev[b]) .. nc(ctx[b]) - 1 of the pair's plane of the compressed-key cache.  D / 8 threads per (pair, new row); a workgroup
// takes `rows` (a power of two) consecutive new rows of as many pairs as its threads are enough for.
template <typename T, int D>
__global__ void __launch_bounds__(64)
compress_k_append_kernel(const T *__restrict__ k, int64_t kv_batch_stride, int64_t kv_head_stride, int64_t kv_tok_stride,
                         float *__restrict__ kc, int64_t kc_head_stride, const int32_t *__restrict__ prev,
                         const int32_t *__restrict__ ctx, int pairs, int hkv, int lc, int sc, int rows) {
    constexpr int VPR = D / VEC;
    const int slot = threadIdx.x / VPR, pair = (blockIdx.y * (64 / VPR) + slot) / rows;
    if (pair >= pairs) return;
    const int b = pair / hkv, h = pair - b * hkv;
    const int i = num_cmp(prev[b], lc, sc) + (int)blockIdx.x * rows + (slot & (rows - 1));
    if (i >= num_cmp(ctx[b], lc, sc)) return;
    const int c0 = (threadIdx.x % VPR) * VEC;
    float acc[VEC];
    window_sum(k + (int64_t)b * kv_batch_stride + (int64_t)h * kv_head_stride + (int64_t)i * sc * kv_tok_stride + c0,
               kv_tok_stride, lc, acc);
    const float inv = 1.0f / (float)lc;
#pragma unroll
    for (int c = 0; c < VEC; ++c) acc[c] *= inv;
    gen::store_row<float, VEC>(kc + (int64_t)pair * kc_head_stride + (int64_t)i * D + c0, acc);
}

template <typename T, int D>
int launch_append_t(const infllmv2_params *p, const void *k, int64_t bs, int64_t hs, int64_t ts, float *kc,
                    int64_t kc_head_stride, const int32_t *prev_d, const int32_t *ctx_d, int batch, int max_new,
                    hipStream_t stream) {
    // one new row per pair in an ordinary decode step; with several, rows of a pair share a workgroup (13331 rows of two pairs,
    // windows of 7, fp32: 21.8 us with a workgroup per row)
    const int pairs = batch * p->num_kv_heads, per = 64 / (D / VEC);
    int rows = 1;
    while (rows < per && rows < max_new) rows *= 2;
    hipLaunchKernelGGL((compress_k_append_kernel<T, D>), dim3((max_new + rows - 1) / rows, (pairs * rows + per - 1) / per),
                       dim3(64), 0, stream, (const T *)k, bs, hs, ts, kc, kc_head_stride, prev_d, ctx_d, pairs, p->num_kv_heads,
                       p->cmp_len, p->cmp_stride, rows);
    return hip_status(hipGetLastError());
}

}  // namespace

int launch_compress_k_append(const infllmv2_params *p, const void *k, int64_t bs, int64_t hs, int64_t ts, float *kc,
                             int64_t kc_head_stride, const int32_t *prev_d, const int32_t *ctx_d, int batch, int max_new,
                             hipStream_t stream) {
    const bool bf = p->dtype == INFLLMV2_BF16;
    if (p->head_dim == 128)
        return bf ? launch_append_t<bf16_t, 128>(p, k, bs, hs, ts, kc, kc_head_stride, prev_d, ctx_d, batch, max_new, stream)
                  : launch_append_t<float, 128>(p, k, bs, hs, ts, kc, kc_head_stride, prev_d, ctx_d, batch, max_new, stream);
    return bf ? launch_append_t<bf16_t, 64>(p, k, bs, hs, ts, kc, kc_head_stride, prev_d, ctx_d, batch, max_new, stream)
              : launch_append_t<float, 64>(p, k, bs, hs, ts, kc, kc_head_stride, prev_d, ctx_d, batch, max_new, stream);
}

int launch_compress_k(const Launch &L, const void *k, float *kc, int32_t *cu_c, const int32_t *cu_h) {
    const bool bf = L.p->dtype == INFLLMV2_BF16;
    if (L.p->head_dim == 128)
        return bf ? launch_t<bf16_t, 128>(L, k, kc, cu_c, cu_h) : launch_t<float, 128>(L, k, kc, cu_c, cu_h);
    return bf ? launch_t<bf16_t, 64>(L, k, kc, cu_c, cu_h) : launch_t<float, 64>(L, k, kc, cu_c, cu_h);
}

}  // namespace ifv2
