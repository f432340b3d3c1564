// Stage 4, generic form: block-sparse causal attention over the selected blocks (Appendix Alg. 2) and dense causal
// attention (Eq. 1 / Appendix Alg. 3) for any G <= 16, d in {64, 128}, fp32 or bf16 data, any stride and alignment,
// prefill and single-row (decode) calls.  The bf16 G = 16 d = 128 shape has its own tile kernel, and large bf16
// calls with rows of 16-byte multiples pass theirs through LDS (attn_staged.hip); this one serves the rest.
//
// A workgroup owns a tile of one or two groups of 16 / G consecutive tokens of one KV head (16 columns each, see gen_unit.h)
// and walks the union of their block lists; its wavefronts take the union's half blocks (32 keys) in turn, each with a
// softmax state of its own, and the partial results are merged in LDS at the end.  Operands come straight from global
// memory: a K row fragment is what the row product wants as it is, a V row is spread over the 16 lanes of a group, so
// nothing passes through LDS and no barrier stands between blocks.  The rows of the next half block are requested as soon
// as the registers of this one's are free (AHEAD), or, in launches of many workgroups, as late as they are needed: fewer
// registers, one wavefront more per SIMD (launch_rules.h).
//
// What bounds it: bf16, the trips of the rows from the L2 to the CUs (255 MB in the case below, 6.5 TB/s), which is why two column groups share them;
// fp32, the products (32 clocks each) and how evenly a tile's half blocks fall on its wavefronts.  Half as many vector
// instructions (rows addressed by a scalar base and a constant lane offset, products over 32 keys, no checks for
// infinities in the first pass, sums rescaled only when a logit is larger than all before) alone took the bf16 case below
// from 58 to 47 us.  Measured: fp32, 2048 tokens, 4 heads on 1, d 64, 8 blocks: 34 -> 27 us; bf16, 1985 tokens, 8 heads
// on 2, d 128, 16 blocks: 58 -> 39 us; fp32, 600 / 2000 tokens, 8 heads on 2, d 128: 36 -> 20, 131 -> 113 us; bf16, 4000 tokens,
// 8 heads on 2, d 128: 153 -> 95 us.  Taken back: the wavefronts of two tiles side by side, meeting in the L1 (51 us).
#include "attn_staged.h"
#include "gen_unit.h"
#include "launch_rules.h"

namespace ifv2 {

namespace {

using namespace gen;

constexpr int NW = 4;             // wavefronts per workgroup

// Workgroups per CU that the registers of a form allow
template <typename T, int D, int CG, bool AHEAD>
constexpr uint32_t kPerCu = (D == 64 ? 2 : 1) + (AHEAD ? 0 : 1) + (sizeof(T) == 2 && CG == 1 ? 1 : 0);

template <typename T, int D, int CG, bool AHEAD>
__global__ void __launch_bounds__(NW * 64)
attn_generic_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v,
                    const int32_t *__restrict__ idx, int topk_total, int dense_below, RowMap map, int hq,
                    float scale, T *__restrict__ out, float *__restrict__ lse, uint32_t back) {
    constexpr int N = D / 16;
    __shared__ Union un;
    __shared__ float o_s[NW][CG * kCols][D + 4], m_s[NW][CG * kCols], l_s[NW][CG * kCols];
    __shared__ int s_tile[3];
    // Late tiles first, for they have the most blocks, one head after the other; or heads side by side and rows of 256 workgroups back and forth
    // (rules::back_and_forth).  (back: the launch's workgroups, or 0; as a flag it would have the grid's size fetched behind it, 0.3 us of every call.)
    const uint32_t workgroups = gridDim.x * gridDim.y;                  // (modulo 2^32)
    uint32_t h = blockIdx.y, nth = blockIdx.x;
    if ((workgroups == back) & (back != 0)) {
        const uint32_t b = back_and_forth(blockIdx.y * gridDim.x + blockIdx.x, workgroups);
        nth = b / gridDim.y;
        h = b - nth * gridDim.y;
    }
    const int G = hq / map.num_kv_heads;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    Tile t;
    if (!find_tile(map, (int)(gridDim.x - 1 - nth), CG * tile_tokens(map, G), t, s_tile)) return;
    const bool dense = idx == nullptr || t.len < dense_below;
    const int32_t *lists = dense ? nullptr : idx + head_row(map, h, t.row0) * topk_total;
    const int nblk = (t.t0 + t.ntok - 1) / kBlock + 1;
    const T *kb = k + t.kv_base + (int64_t)h * map.kv_head_stride;
    const T *vb = v + t.kv_base + (int64_t)h * map.kv_head_stride;
    const float c = scale * kLog2e;

    // this lane's columns: token ti of the tile, head of the group (unused columns repeat column 0 and see nothing)
    const int m = lane & 15, g = lane >> 4;
    const int tokens = tile_tokens(map, G), head = m % G;
    int ti[CG];
    bool used[CG];
    RowFrag<T, D> qf[CG];
#pragma unroll
    for (int x = 0; x < CG; ++x) {
        ti[x] = x * tokens + m / G;
        used[x] = m / G < tokens && ti[x] < t.ntok;
        qf[x].load(q + ((int64_t)(t.row0 + (used[x] ? ti[x] : 0)) * hq + h * G + (used[x] ? head : 0)) * D, g);
    }
    const KeyRows<T, D> krows(kb, map.kv_tok_stride, t.len, m, g), vrows(vb, map.kv_tok_stride, t.len, m, g);

    // One pass serves all tokens of the tile.  A key that only some of them see enters the others' sums with
    // probability 0, which is exact unless its V row holds an infinity or a NaN: a result that is not finite is
    // therefore computed again token by token (solo >= 0) with the V rows the token does not see taken as 0.
    uint32_t all = t.ntok == 32 ? ~0u : (1u << t.ntok) - 1u;
    int solo = -1;
    for (;;) {
        float ref[CG], l_run[CG];                        // largest logit so far, sum relative to it
        f32x4 o[CG][N];                                  // O^T: dim N (4 g + r) + j, this lane's column
#pragma unroll
        for (int x = 0; x < CG; ++x) {
            ref[x] = -INFINITY;
            l_run[x] = 0.f;
#pragma unroll
            for (int j = 0; j < N; ++j) o[x][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int c0 = 0; c0 < nblk; c0 += kChunk) {
            un.build(lists, topk_total, t, c0, nblk, all, tid, NW * 64);
            const int items = un.half_blocks(t);
            RowFrag<T, D> kf[2];
            Spread<T, D> vr[2][4];
            int2 ent = {0, 0};
            auto key_of = [&](int it) -> int {
                ent = un.list[it >> 1];
                ent.x = __builtin_amdgcn_readfirstlane(ent.x);
                ent.y = __builtin_amdgcn_readfirstlane(ent.y);
                return ent.x * kBlock + 32 * (it & 1);
            };
            int u0 = 0;
            if (AHEAD && w < items) {
                u0 = key_of(w);
                krows.frags(kf, u0, m, g);
                vrows.spread(vr, u0, m, g);
            }
            for (int it = w; it < items; it += NW) {
                if (!AHEAD) {
                    u0 = key_of(it);
                    krows.frags(kf, u0, m, g);
                }
                f32x4 s[CG][2];
#pragma unroll
                for (int x = 0; x < CG; ++x)
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt) s[x][kt] = row_product<D>(kf[kt], qf[x]);
                // lane: keys 16 kt + 4 g + r of the half block
                const int here = u0;
                const uint32_t takers = (uint32_t)ent.y;
                const bool more = AHEAD && it + NW < items;
                if (!AHEAD) vrows.spread(vr, u0, m, g);
                if (more) {                              // the next half block's K rows, while this one's softmax runs
                    u0 = key_of(it + NW);
                    krows.frags(kf, u0, m, g);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (solo >= 0) {
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (here + 16 * kt + 4 * g + r > t.t0 + solo) vr[kt][r].zero();
                }
#pragma unroll
                for (int x = 0; x < CG; ++x) {
                    if (CG > 1 && ((takers >> (x * tokens)) & ((1u << tokens) - 1u)) == 0u) continue;
                    const bool takes = used[x] && ((takers >> ti[x]) & 1u);
                    if (here + 31 > t.t0) {              // the own block: keys behind a token
                        const int lim = takes ? t.t0 + ti[x] - here : -1;
#pragma unroll
                        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (16 * kt + 4 * g + r > lim) s[x][kt][r] = -INFINITY;
                    }
                    float mx = fmaxf(fmaxf(fmaxf(s[x][0][0], s[x][0][1]), fmaxf(s[x][0][2], s[x][0][3])),
                                     fmaxf(fmaxf(s[x][1][0], s[x][1][1]), fmaxf(s[x][1][2], s[x][1][3])));
                    mx = takes ? mx : -INFINITY;
                    if (__any(mx > ref[x])) {            // the reference is a column's largest logit so far
                        const float top = fmaxf(ref[x], groups_max(mx));
                        const float alpha = top == -INFINITY ? 0.f : exp2_fast((ref[x] - top) * c);    // exp2(-inf) = 0 at first
                        ref[x] = top;
                        l_run[x] *= alpha;
#pragma unroll
                        for (int j = 0; j < N; ++j) o[x][j] *= alpha;
                    }
                    const float sub = takes && ref[x] != -INFINITY ? ref[x] : INFINITY;      // (a column that does not take part: 0)
                    float ls[2] = {0.f, 0.f};
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            s[x][kt][r] = exp2_fast((s[x][kt][r] - sub) * c);
                            ls[kt] += s[x][kt][r];
                        }
                    l_run[x] += ls[0] + ls[1];
                    weighted_rows32<false, false, D>(o[x], s[x][0], s[x][1], vr[0], vr[1]);
                }
                if (more) vrows.spread(vr, u0, m, g);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();                             // the list may be rebuilt
        }
#pragma unroll
        for (int x = 0; x < CG; ++x) {
            const float lg = groups_sum(l_run[x]);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < N; ++j) o_s[w][x * kCols + m][N * (4 * g + r) + j] = o[x][j][r];
            if (g == 0) { m_s[w][x * kCols + m] = ref[x]; l_s[w][x * kCols + m] = lg; }
        }
        __syncthreads();
        // thread (column, N dims): merge the wavefronts' partial results
        static_assert(NW * 64 == kCols * 16, "sixteen threads per column");
        const int d0 = (tid & 15) * N;
        float y[CG][N], lse_x[CG];
        bool bad = false;
#pragma unroll
        for (int x = 0; x < CG; ++x) {
            const int col = x * kCols + (tid >> 4), tc = x * tokens + (tid >> 4) / G;
            float mm = m_s[0][col];
#pragma unroll
            for (int u = 1; u < NW; ++u) mm = fmaxf(mm, m_s[u][col]);
            const float base = mm == -INFINITY ? 0.f : mm;
            float L = 0.f;
#pragma unroll
            for (int j = 0; j < N; ++j) y[x][j] = 0.f;
#pragma unroll
            for (int u = 0; u < NW; ++u) {
                const float wg = exp2_fast((m_s[u][col] - base) * c);
                L += l_s[u][col] * wg;
#pragma unroll
                for (int j = 0; j < N; ++j) y[x][j] += o_s[u][col][d0 + j] * wg;
            }
            lse_x[x] = mm * scale + __logf(L);
            const bool mine = (tid >> 4) / G < tokens && tc < t.ntok && ((all >> tc) & 1u);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                y[x][j] /= L;
                bad |= mine && !finite(y[x][j]);
            }
        }
        const bool again = solo < 0 && __syncthreads_or(bad);
        if (!again) {
#pragma unroll
            for (int x = 0; x < CG; ++x) {
                const int tc = x * tokens + (tid >> 4) / G;
                if ((tid >> 4) / G >= tokens || tc >= t.ntok || !((all >> tc) & 1u)) continue;
                const int qh = h * G + (tid >> 4) % G;
                store_row<T, N>(out + ((int64_t)(t.row0 + tc) * hq + qh) * D + d0, y[x]);
                if (lse != nullptr && (tid & 15) == 0) lse[qhead_row(map, qh, hq, t.row0 + tc)] = lse_x[x];
            }
        }
        if (solo < 0 && !again) return;
        if (++solo >= t.ntok) return;
        all = 1u << solo;
        __syncthreads();                                 // o_s is overwritten by the next pass
    }
}

template <typename T, int D, int CG, bool AHEAD>
int launch_cg(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, void *out,
              float *lse, const int32_t *cu_h, double half_blocks) {
    const int tokens = CG * tile_tokens(L.map, L.p->num_q_heads / L.p->num_kv_heads);
    // at most this many tiles (every sequence may end with a partial one)
    const unsigned tiles = L.map.ctx ? L.map.total_rows : L.map.total_rows / tokens + L.map.batch;
    const bool back = rules::back_and_forth(cu_h, L.map.batch, tokens, tiles, L.p->num_kv_heads, idx != nullptr, L.p->topk_total, dense_below,
                                            half_blocks, 256 * kPerCu<T, D, CG, AHEAD>, false);
    hipLaunchKernelGGL((attn_generic_kernel<T, D, CG, AHEAD>), dim3(tiles, L.p->num_kv_heads), dim3(NW * 64), 0, L.stream,
                       (const T *)q, (const T *)k, (const T *)v, idx, L.p->topk_total, dense_below, L.map,
                       L.p->num_q_heads, L.p->softmax_scale, (T *)out, lse, back ? tiles * L.p->num_kv_heads : 0);
    return hip_status(hipGetLastError());
}

template <typename T, int D>
int launch_t(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, void *out,
             float *lse, const int32_t *cu_h) {
    if (L.map.total_rows == 0) return INFLLMV2_OK;
    if (L.map.ctx != nullptr) return launch_cg<T, D, 1, true>(L, q, k, v, idx, dense_below, out, lse, nullptr, 0);      // (one token per tile)
    const int hkv = L.p->num_kv_heads;
    const rules::Walks x = rules::walks(cu_h, L.map.batch, tile_tokens(L.map, L.p->num_q_heads / hkv), idx != nullptr,
                                        L.p->topk_total, dense_below);
    if (sizeof(T) == 2 && rules::staged(false, D, x.two * hkv, x) && attn_staged_takes(L, k, v))
        return launch_attn_staged(L, q, k, v, idx, dense_below, out, lse, cu_h, x);
    const rules::GenericForm form = rules::generic_form(sizeof(T) == 2, D, hkv, x);
    if constexpr (sizeof(T) == 2)
        if (form.groups == 2)
            return form.ahead ? launch_cg<T, D, 2, true>(L, q, k, v, idx, dense_below, out, lse, cu_h, x.half_blocks)
                              : launch_cg<T, D, 2, false>(L, q, k, v, idx, dense_below, out, lse, cu_h, x.half_blocks);
    const bool ahead = sizeof(T) == 2 ? form.ahead : rules::fp32_rows_ahead(D, hkv, x.one * hkv, x);
    return ahead ? launch_cg<T, D, 1, true>(L, q, k, v, idx, dense_below, out, lse, cu_h, x.half_blocks)
                 : launch_cg<T, D, 1, false>(L, q, k, v, idx, dense_below, out, lse, cu_h, x.half_blocks);
}

}  // namespace

int launch_attn_generic(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx,
                        int dense_below, void *out, float *lse, const int32_t *cu_h) {
    const bool bf = L.p->dtype == INFLLMV2_BF16;
    if (L.p->head_dim == 128)
        return bf ? launch_t<bf16_t, 128>(L, q, k, v, idx, dense_below, out, lse, cu_h)
                  : launch_t<float, 128>(L, q, k, v, idx, dense_below, out, lse, cu_h);
    return bf ? launch_t<bf16_t, 64>(L, q, k, v, idx, dense_below, out, lse, cu_h)
              : launch_t<float, 64>(L, q, k, v, idx, dense_below, out, lse, cu_h);
}

}  // namespace ifv2
