// Stage 4, generic form: block-sparse causal attention over the selected blocks (Appendix Alg. 2) and dense causal
// attention (Eq. 1 / Appendix Alg. 3) for any G <= 16, d in {64, 128}, fp32 or bf16 data, any stride and alignment,
// prefill and single-row (decode) calls.  The bf16 G = 16 d = 128 shape has its own tile kernel; this one serves the
// rest.
//
// A workgroup owns a tile of 16 / G consecutive tokens of one KV head (16 columns, see gen_unit.h) and walks the union
// of their block lists; its wavefronts take the union's blocks in turn, each with a softmax state of its own, and the
// partial results are merged in LDS at the end.  Operands come straight from global memory: a K row fragment is what
// the row product wants as it is, a V row is spread over the 16 lanes of a group, so nothing passes through LDS and no
// barrier stands between blocks.
//
// What bounds it: the chain of a block (K rows, logits, softmax, V rows, products) at two to three wavefronts per SIMD.
// Measured: fp32, 2048 tokens, 4 heads on 1, d 64, 8 blocks: 217 -> 33 us; bf16, 1985 tokens, 8 heads on 2, d 128, 16
// blocks: 648 -> 58 us (one workgroup per token with fp32 vector arithmetic before).  Eight wavefronts per workgroup
// instead of four: 32 and 69 us; the next block's rows requested ahead: 37 and 96 us (one wavefront per SIMD).
#include "gen_unit.h"

namespace ifv2 {

namespace {

using namespace gen;

constexpr int NW = 4;             // wavefronts per workgroup

template <typename T, int D>
__global__ void __launch_bounds__(NW * 64)
attn_generic_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v,
                    const int32_t *__restrict__ idx, int topk_total, int dense_below, RowMap map, int hq,
                    float scale, T *__restrict__ out, float *__restrict__ lse) {
    constexpr int N = D / 16;
    __shared__ Union un;
    __shared__ float o_s[NW][kCols][D + 4], m_s[NW][kCols], l_s[NW][kCols];
    __shared__ int s_tile[3];
    const int h = blockIdx.y, G = hq / map.num_kv_heads;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    Tile t;
    // (late tiles first: they have the most blocks)
    if (!find_tile(map, gridDim.x - 1 - blockIdx.x, tile_tokens(map, G), t, s_tile)) return;
    const bool dense = idx == nullptr || t.len < dense_below;
    const int32_t *lists = dense ? nullptr : idx + head_row(map, h, t.row0) * topk_total;
    const int nblk = (t.t0 + t.ntok - 1) / kBlock + 1;
    const T *kb = k + t.kv_base + (int64_t)h * map.kv_head_stride;
    const T *vb = v + t.kv_base + (int64_t)h * map.kv_head_stride;
    const float c = scale * kLog2e;

    // this lane's column: token ti of the tile, head of the group (unused columns repeat column 0 and see nothing)
    const int m = lane & 15, g = lane >> 4;
    const int ti = m / G;
    const bool used = ti < t.ntok;
    RowFrag<T, D> qf;
    qf.load(q + ((int64_t)(t.row0 + (used ? ti : 0)) * hq + h * G + (used ? m - ti * G : 0)) * D, g);

    // One pass serves all tokens of the tile.  A key that only some of them see enters the others' sums with
    // probability 0, which is exact unless its V row holds an infinity or a NaN: a result that is not finite is
    // therefore computed again token by token (solo >= 0) with the V rows the token does not see taken as 0.
    uint32_t all = (1u << t.ntok) - 1u;
    int solo = -1;
    for (;;) {
        const int solo_t = t.t0 + solo;                  // (used when solo >= 0)
        float m_run = -INFINITY, l_run = 0.f;
        f32x4 o[N];                                      // O^T: dim N (4 g + r) + j, this lane's column
#pragma unroll
        for (int j = 0; j < N; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int c0 = 0; c0 < nblk; c0 += kChunk) {
            un.build(lists, topk_total, t, c0, nblk, all, tid, NW * 64);
            const int count = un.count;
            for (int e = w; e < count; e += NW) {
                const int2 ent = un.list[e];
                const int u0 = ent.x * kBlock;
                const int lim = used && ((ent.y >> ti) & 1) ? t.t0 + ti - u0 : -1;       // last visible key of the block
                f32x4 s[4];
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) {
                    RowFrag<T, D> kf;
                    kf.load(kb + (int64_t)min(u0 + 16 * kt + m, t.len - 1) * map.kv_tok_stride, g);
                    s[kt] = row_product<D>(kf, qf);
                }
                // lane: keys 16 kt + 4 g + r of the block
                float mx = -INFINITY;
#pragma unroll
                for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (16 * kt + 4 * g + r > lim) s[kt][r] = -INFINITY;
                        mx = fmaxf(mx, s[kt][r]);
                    }
                const float m_new = fmaxf(m_run, groups_max(mx));
                const float ref = m_new == -INFINITY ? 0.f : m_new;
                const float alpha = exp2_fast((m_run - ref) * c);         // exp2(-inf) = 0 on the first block
                m_run = m_new;
                float ls = 0.f;
#pragma unroll
                for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        s[kt][r] = exp2_fast((s[kt][r] - ref) * c);
                        ls += s[kt][r];
                    }
                l_run = l_run * alpha + ls;
#pragma unroll
                for (int j = 0; j < N; ++j) o[j] *= alpha;
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) {
                    Spread<T, D> vr[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int u = u0 + 16 * kt + 4 * g + r;
                        vr[r].load(vb + (int64_t)min(u, t.len - 1) * map.kv_tok_stride, m);
                        if (solo >= 0 && u > solo_t) vr[r].zero();
                    }
                    weighted_rows<false, D>(o, s[kt], vr);
                }
            }
            __syncthreads();                             // the list may be rebuilt
        }
        l_run = groups_sum(l_run);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < N; ++j) o_s[w][m][N * (4 * g + r) + j] = o[j][r];
        if (g == 0) { m_s[w][m] = m_run; l_s[w][m] = l_run; }
        __syncthreads();
        // thread (column, N dims): merge the wavefronts' partial results
        static_assert(NW * 64 == kCols * 16, "sixteen threads per column");
        const int col = tid >> 4, d0 = (tid & 15) * N, tc = col / G;
        float mm = m_s[0][col];
#pragma unroll
        for (int x = 1; x < NW; ++x) mm = fmaxf(mm, m_s[x][col]);
        const float ref = mm == -INFINITY ? 0.f : mm;
        float L = 0.f, y[N];
#pragma unroll
        for (int j = 0; j < N; ++j) y[j] = 0.f;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            const float wg = exp2_fast((m_s[x][col] - ref) * c);
            L += l_s[x][col] * wg;
#pragma unroll
            for (int j = 0; j < N; ++j) y[j] += o_s[x][col][d0 + j] * wg;
        }
        bool bad = false;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            y[j] /= L;
            bad |= !finite(y[j]);
        }
        const bool mine = tc < t.ntok && ((all >> tc) & 1u);
        const bool again = solo < 0 && __syncthreads_or(mine && bad);
        if (!again && mine) {
            const int qh = h * G + col - tc * G;
            store_row<T, N>(out + ((int64_t)(t.row0 + tc) * hq + qh) * D + d0, y);
            if (lse != nullptr && (tid & 15) == 0) lse[qhead_row(map, qh, hq, t.row0 + tc)] = mm * scale + __logf(L);
        }
        if (solo < 0 && !again) return;
        if (++solo >= t.ntok) return;
        all = 1u << solo;
        __syncthreads();                                 // o_s is overwritten by the next pass
    }
}

template <typename T, int D>
int launch_t(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, void *out,
             float *lse) {
    if (L.map.total_rows == 0) return INFLLMV2_OK;
    const int tokens = tile_tokens(L.map, L.p->num_q_heads / L.p->num_kv_heads);
    // at most this many tiles (every sequence may end with a partial one)
    const unsigned tiles = L.map.ctx ? L.map.total_rows : L.map.total_rows / tokens + L.map.batch;
    hipLaunchKernelGGL((attn_generic_kernel<T, D>), dim3(tiles, L.p->num_kv_heads), dim3(NW * 64), 0, L.stream,
                       (const T *)q, (const T *)k, (const T *)v, idx, L.p->topk_total, dense_below, L.map,
                       L.p->num_q_heads, L.p->softmax_scale, (T *)out, lse);
    return hip_status(hipGetLastError());
}

}  // namespace

int launch_attn_generic(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx,
                        int dense_below, void *out, float *lse) {
    const bool bf = L.p->dtype == INFLLMV2_BF16;
    if (L.p->head_dim == 128)
        return bf ? launch_t<bf16_t, 128>(L, q, k, v, idx, dense_below, out, lse)
                  : launch_t<float, 128>(L, q, k, v, idx, dense_below, out, lse);
    return bf ? launch_t<bf16_t, 64>(L, q, k, v, idx, dense_below, out, lse)
              : launch_t<float, 64>(L, q, k, v, idx, dense_below, out, lse);
}

}  // namespace ifv2
