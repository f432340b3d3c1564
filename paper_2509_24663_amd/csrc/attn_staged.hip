// Stage 4 and its dQ, generic form, bf16: large calls (launch_rules.h says which).  As attn_generic.hip and the dQ of attn_bwd.hip, with tiles
// of two column groups: a wavefront takes every fourth half block (32 keys) of the tile's walk, for both groups.  What differs:
//   * V rows (dQ: K rows), the second operand of the products with computed weights, are copied to LDS asynchronously, one half block
//     ahead, into two buffers of the wavefront's own, and read transposed: no registers hold them in flight and no byte permutes spread
//     them, so that two wavefronts per SIMD (d 64: three) fit with everything requested ahead.  Nobody else reads a wavefront's
//     buffers: no barrier stands in the walk;
//   * softmax references move only when a logit exceeds them by a factor of 2^8 (forward): fewer rescales, the same 24 bits;
//   * long and short tiles share a CU (see the order of the workgroups).
// What bounds it: the chain of a wavefront's step (its requests take 1100 clocks of 4200 to go out, the 64 products with their LDS reads 1500, the
// softmax 1250; two wavefronts per SIMD) and, per workgroup, 3.6 us of chained requests before its first step and 2.5 after the last.  In the
// case below rows come at 8 TB/s (255 MB, nine tenths from the L2) and the matrix cores are busy for a sixth of the time.  Measured, 1985 tokens, 8 heads on 2, 16 blocks: attention d 128 40 -> 31 us (37.8 without the order of
// the workgroups), d 64 30 -> 22.4; backward call d 128 109 -> 97, d 64 82 -> 66.  6000 tokens, d 128: attention 181 -> 158, backward 517 -> 390.
// Measured and not built: tiles of four groups in eight wavefronts with K and V in LDS (half the traffic, but a barrier per interval keeps
// the wavefronts of a SIMD in step: 44 us); first copies before the lists where a walk has all blocks (2 us slower: registers);
// forward operands requested between the last products (37 us), which the backward at d 128 needs for its registers (107 -> 99).
#include "attn_staged.h"
#include "attn_unit.h"
#include "gen_unit.h"
#include "lds_rows.h"

namespace ifv2 {

namespace {

using namespace gen;

constexpr int NW = 4;                  // wavefronts; each takes every fourth half block (32 keys) of the walk
constexpr int CG = 2;                  // column groups
constexpr int kTileCols = CG * kCols;
using lds_rows::kRowBytes;             // of LDS; d 64: rows r and 16 + r of the half block side by side

// 16 bytes per lane from global memory to LDS address lds + 16 lane; the caller waits before it reads them
__device__ inline void copy16(const char *src, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory", "m0");
}

// Half blocks of K or V rows in LDS, two buffers of a wavefront's own: nobody else reads them, so a wait takes the place of a barrier.
template <int D>
struct Stage {
    static constexpr uint32_t kBytes = 32 * D * 2;
    const char *src;                   // row lane / 16 of the tensor
    int64_t stride;                    // bytes from token to token
    int len;
    uint32_t lds0, row_at, trans_at;

    __device__ inline Stage(const bf16_t *rows, int64_t tok_stride, int len_, int lane, uint32_t lds)
        : stride(tok_stride * 2), len(len_), lds0(lds) {
        src = reinterpret_cast<const char *>(rows) + (lane >> 4) * stride;
        const int m = lane & 15, g = lane >> 4;
        row_at = lds + address(lds_rows::operand_row(m), g);
        trans_at = lds + address(lds_rows::piece_row(m, g), lds_rows::piece_chunk(m)) + lds_rows::piece_half(m);
    }
    static __device__ inline uint32_t address(int row, int chunk) {
        return D == 128 ? lds_rows::offset(row, chunk) : lds_rows::offset(row & 15, chunk + 8 * (row >> 4));
    }
    // keys key0 .. + 31, 1 KB (four LDS rows) at a time
    __device__ inline void copy(int key0, int buf) const {
        constexpr int P = kBytes / 1024;
        const uint32_t dst = lds0 + buf * kBytes;
        int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(l));                      // (the lane and its offsets are formed here, not kept in registers over the walk)
        const char *from = src + (int64_t)key0 * stride;
        const int c = (l & 15) ^ (4 * (l >> 4)), up = D == 128 ? 0 : 16 * (c >> 3);
        auto chunk_at = [&](int p) -> int { return ((c ^ (2 * ((p >> 1) & 1) + (p >> 2))) & (D / 8 - 1)) * 16; };
        if (key0 + 32 <= len) {
            const char *lane_from = from + up * stride;
#pragma unroll
            for (int p = 0; p < P; ++p) copy16(lane_from + 4 * p * stride + chunk_at(p), dst + 1024u * p);
        } else {                                         // past the end: the last row, never visible
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int row = min(key0 + up + (l >> 4) + 4 * p, len - 1) - (l >> 4);
                copy16(src + (int64_t)row * stride + chunk_at(p), dst + 1024u * p);
            }
        }
    }
    __device__ inline bf16x8 row_frag(int buf, int kt, int s) const { return lds_rows::operand(row_at + buf * kBytes, kt, s); }
    // rows 8 g .. 8 g + 7 of dim 16 i + lane % 16
    __device__ inline bf16x8 trans_frag(int buf, int i) const { return lds_rows::transposed((trans_at + buf * kBytes) ^ (uint32_t)(32 * i)); }
};

struct StagedArgs {
    const bf16_t *q, *k, *v;
    const int32_t *idx;         // nullptr: dense
    int topk_total, dense_below, hq;
    float scale;
    RowMap map;
    bf16_t *out;                // forward: O; backward: dQ
    float *lse;                 // forward: output (or nullptr); backward: input
    const bf16_t *dout;         // backward
    const float *delta;
    uint32_t resident;          // workgroups that the chip holds at once, or 0: in the plain order
};

// acc[x] += (weights of column group x) x (the half block's rows), weights in three exact pieces (see weighted_rows32); x of [X0, X1)
// mid(i), i = 0 .. D / 16 - 1: what goes out between the products
template <int D, int X0, int X1, bool SOLO, class Mid>
__device__ inline void accumulate(f32x4 (&acc)[CG][D / 16], const bf16x8 (&pc)[CG][3], const Stage<D> &st, int buf, attn_unit::u32x4 keep, Mid mid) {
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
        mid(i);
        bf16x8 r = st.trans_frag(buf, i);
        if (SOLO) r = attn_unit::keep_keys(r, keep);
#pragma unroll
        for (int p = 2; p >= 0; --p)
#pragma unroll
            for (int x = X0; x < X1; ++x) acc[x][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(r, pc[x][p], acc[x][i], 0, 0, 0);
    }
}

template <int D, bool BWD>
__global__ void __launch_bounds__(NW * 64, D == 128 ? 2 : 3) attn_staged_kernel(StagedArgs a, int num_tiles) {
    constexpr int N = D / 16;
    constexpr bool LATE = BWD && D == 128;               // operands requested between the last products: registers
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    __shared__ Union un;
    __shared__ float m_s[NW][kTileCols], l_s[NW][kTileCols];
    __shared__ int s_tile[3], s_bad;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // longest tiles first, heads side by side
    const uint32_t b = gridDim.x <= a.resident ? back_and_forth(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t hkv = (uint32_t)a.map.num_kv_heads, nth = b / hkv;
    const int h = (int)(b - nth * hkv), G = a.hq / (int)hkv;
    const int tokens = kCols / G;
    Tile t;
    if (!find_tile(a.map, num_tiles - 1 - (int)nth, CG * tokens, t, s_tile)) return;
    const bool dense = a.idx == nullptr || t.len < a.dense_below;
    const int32_t *lists = dense ? nullptr : a.idx + head_row(a.map, h, t.row0) * a.topk_total;
    const int nblk = (t.t0 + t.ntok - 1) / kBlock + 1;
    const int64_t head_off = t.kv_base + (int64_t)h * a.map.kv_head_stride, stride = a.map.kv_tok_stride * 2;
    const float c = a.scale * kLog2e, lag = c > 0.f ? fminf(8.f / c, 1e30f) : 0.f;

    const int m = lane & 15, g = lane >> 4;
    int ti[CG];
    bool used[CG];
    RowFrag<bf16_t, D> qf[CG], gf[CG];
    float lse[CG], delta[CG];
#pragma unroll
    for (int x = 0; x < CG; ++x) {
        ti[x] = x * tokens + m / G;
        used[x] = m / G < tokens && ti[x] < t.ntok;
        const int row = t.row0 + (used[x] ? ti[x] : 0), qh = h * G + (used[x] ? m % G : 0);
        qf[x].load(a.q + ((int64_t)row * a.hq + qh) * D, g);
        if (BWD) {
            gf[x].load(a.dout + ((int64_t)row * a.hq + qh) * D, g);
            lse[x] = a.lse[qhead_row(a.map, qh, a.hq, row)];
            delta[x] = a.delta[qhead_row(a.map, qh, a.hq, row)];
        }
    }
    // forward: K rows are operands as they are, V rows pass through LDS; backward: the other way round
    const uint32_t lds = __builtin_amdgcn_readfirstlane(attn_unit::lds_address(smem)) + (uint32_t)w * 2 * Stage<D>::kBytes;
    const Stage<D> st((BWD ? a.k : a.v) + head_off, a.map.kv_tok_stride, t.len, lane, lds);
    const int r0 = 8 * (m >> 2) + (m & 3);
    const char *direct = reinterpret_cast<const char *>((BWD ? a.v : a.k) + head_off) + r0 * stride + 16 * g;

    float ref[CG], l_run[CG];                            // a column's largest logit when last moved, sum relative to it
    f32x4 acc[CG][N];                                    // O^T or dQ^T: dim 16 i + 4 g + r, this lane's column
    // One pass serves all tokens of the tile; a result that is not finite is computed again token by token (solo >= 0) with
    // the rows that the token does not see taken as 0 (0 x infinity), and with references that do not lag: sums of V of more than 1.3e36 overflow
    // with weights of 2^8 where they do not with weights of 1.
    uint32_t all = t.ntok == 32 ? ~0u : (1u << t.ntok) - 1u;
    auto pass = [&](auto solo_pass, int solo) {
        constexpr bool SOLO = decltype(solo_pass)::value;
        const float slack = SOLO ? 0.f : lag;
#pragma unroll
        for (int x = 0; x < CG; ++x) {
            ref[x] = -INFINITY;
            l_run[x] = 0.f;
#pragma unroll
            for (int i = 0; i < N; ++i) acc[x][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int c0 = 0; c0 < nblk; c0 += kChunk) {
            RowFrag<bf16_t, D> df[2];
            int next_key = 0;
            // a half block's rows into LDS and, in the order of Stage::row_frag, as operands: where this lane's two rows are, and a part of them
            auto direct_rows = [&](const char *(&p)[2]) {
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) p[kt] = direct + (int64_t)(min(next_key + 4 * kt + r0, t.len - 1) - r0) * stride;
            };
            auto load_part = [&](const char *const (&p)[2], int i) {
                constexpr int S = D / 32;
                df[i / S].x[i % S] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8_u *>(p[i / S] + 64 * (i % S)));
            };
            auto load_all = [&]() {
                const char *p[2];
                direct_rows(p);
#pragma unroll
                for (int i = 0; i < N; ++i) load_part(p, i);
            };
            auto half_block = [&](int it, int block) { return block * kBlock + 32 * (it & 1); };
            un.build(lists, a.topk_total, t, c0, nblk, all, tid, NW * 64);
            const int items = __builtin_amdgcn_readfirstlane(un.half_blocks(t));
            if (w < items) {
                next_key = half_block(w, __builtin_amdgcn_readfirstlane(un.list[w >> 1].x));
                st.copy(next_key, 0);
                load_all();
            }
            int buf = 0;
            for (int it = w; it < items; it += NW, buf ^= 1) {
                __builtin_amdgcn_s_waitcnt(attn_unit::WAIT_VMCNT0);      // the copies have landed (and the operands, requested after them)
                asm volatile("" ::: "memory");
                const int here = next_key;
                const uint32_t takers = __builtin_amdgcn_readfirstlane((uint32_t)un.list[it >> 1].y);
                f32x4 s[CG][2], dp[CG][2];                               // lane: keys 8 g + 4 kt + r of the half block
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) {
                    if (BWD) {
                        RowFrag<bf16_t, D> f;
#pragma unroll
                        for (int ks = 0; ks < D / 32; ++ks) f.x[ks] = st.row_frag(buf, kt, ks);
#pragma unroll
                        for (int x = 0; x < CG; ++x) {
                            dp[x][kt] = row_product<D>(df[kt], gf[x]);
                            s[x][kt] = row_product<D>(f, qf[x]);
                        }
                    } else {
#pragma unroll
                        for (int x = 0; x < CG; ++x) s[x][kt] = row_product<D>(df[kt], qf[x]);
                    }
                }
                if (it + NW < items) {
                    next_key = half_block(it, __builtin_amdgcn_readfirstlane(un.list[(it + NW) >> 1].x));
                    st.copy(next_key, buf ^ 1);
                    if (!LATE) load_all();
                }
                __builtin_amdgcn_sched_barrier(0);
                const bool on0 = takers & ((1u << tokens) - 1u), on1 = takers >> tokens;
                bf16x8 pc[CG][3];
#pragma unroll
                for (int x = 0; x < CG; ++x) {
                    if (!(x ? on1 : on0)) {
                        pc[x][0] = pc[x][1] = pc[x][2] = bf16x8{};
                        continue;
                    }
                    const bool takes = used[x] && ((takers >> ti[x]) & 1u);
                    const int lim = takes ? t.t0 + ti[x] - here - 8 * g : -1;       // last visible key of this lane's eight
                    if (BWD) {
#pragma unroll
                        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const float p = exp2_fast(__builtin_fmaf(s[x][kt][r], a.scale, -lse[x]) * kLog2e);
                                s[x][kt][r] = p * (dp[x][kt][r] - delta[x]);
                            }
                        if (__any(lim < 7)) {
#pragma unroll
                            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                                for (int r = 0; r < 4; ++r) s[x][kt][r] = 4 * kt + r <= lim ? s[x][kt][r] : 0.f;
                        }
                        float top = 0.f;
#pragma unroll
                        for (int r = 0; r < 4; ++r) top = fmaxf(top, fmaxf(fabsf(s[x][0][r]), fabsf(s[x][1][r])));
                        if (__any(top == INFINITY)) {
#pragma unroll
                            for (int p = 0; p < 3; ++p) pc[x][p] = take_piece32<true>(s[x][0], s[x][1]);
                        } else {
#pragma unroll
                            for (int p = 0; p < 3; ++p) pc[x][p] = take_piece32<false>(s[x][0], s[x][1]);
                        }
                    } else {
                        if (here + 31 > t.t0) {                          // keys behind a token
#pragma unroll
                            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                                for (int r = 0; r < 4; ++r)
                                    if (4 * kt + r > lim) s[x][kt][r] = -INFINITY;
                        }
                        float mx = fmaxf(fmaxf(fmaxf(s[x][0][0], s[x][0][1]), fmaxf(s[x][0][2], s[x][0][3])),
                                         fmaxf(fmaxf(s[x][1][0], s[x][1][1]), fmaxf(s[x][1][2], s[x][1][3])));
                        mx = takes ? mx : -INFINITY;
                        // (weights up to 2^8 have the same 24 bits as weights up to 1)
                        if (__any(mx > ref[x] + slack)) {
                            const float top = fmaxf(ref[x], groups_max(mx));
                            const float alpha = top == -INFINITY ? 0.f : exp2_fast((ref[x] - top) * c);    // exp2(-inf) = 0 at first
                            ref[x] = top;
                            l_run[x] *= alpha;
#pragma unroll
                            for (int j = 0; j < N; ++j) acc[x][j] *= alpha;
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
#pragma unroll
                        for (int p = 0; p < 3; ++p) pc[x][p] = take_piece32<false>(s[x][0], s[x][1]);
                    }
                }
                attn_unit::u32x4 keep = {0u, 0u, 0u, 0u};
                if (SOLO) keep = attn_unit::keep_mask(t.t0 + solo - here - 8 * g);
                __builtin_amdgcn_sched_barrier(0);
                const char *next_rows[2];                // (after the walk's last half block: its own once more)
                if (LATE) direct_rows(next_rows);
                auto mid = [&](int i) {
                    if (LATE) load_part(next_rows, i);
                };
                if (SOLO || (on0 && on1)) accumulate<D, 0, 2, SOLO>(acc, pc, st, buf, keep, mid);
                else if (on0) accumulate<D, 0, 1, SOLO>(acc, pc, st, buf, keep, mid);
                else accumulate<D, 1, 2, SOLO>(acc, pc, st, buf, keep, mid);
            }
            __syncthreads();                             // the list may be rebuilt, the stages are free
        }
    };
    // partial results of the wavefronts, merged and stored by eight threads per column; a 16-byte chunk of column m at chunk ^ m
    auto finish = [&]() -> bool {
        int tid = w * 64 + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(tid));                    // (as above)
        const int m = tid & 15, g = (tid >> 4) & 3;
        f32x4 *part = reinterpret_cast<f32x4 *>(smem);
#pragma unroll
        for (int x = 0; x < CG; ++x) {
            const int col = x * kCols + m;
#pragma unroll
            for (int i = 0; i < N; ++i) part[(w * kTileCols + col) * (D / 4) + ((4 * i + g) ^ m)] = acc[x][i];
            if (!BWD) {
                const float lg = groups_sum(l_run[x]);
                if (g == 0) { m_s[w][col] = ref[x]; l_s[w][col] = lg; }
            }
        }
        __syncthreads();
        const int col = tid >> 3, mc = col & 15, tc = (col >> 4) * tokens + mc / G;
        const bool mine = mc / G < tokens && tc < t.ntok && ((all >> tc) & 1u);
        float wg[NW], L = 0.f, lse_out = 0.f;
        if (!BWD) {
            float mm = m_s[0][col];
#pragma unroll
            for (int u = 1; u < NW; ++u) mm = fmaxf(mm, m_s[u][col]);
            const float base = mm == -INFINITY ? 0.f : mm;
#pragma unroll
            for (int u = 0; u < NW; ++u) {
                wg[u] = exp2_fast((m_s[u][col] - base) * c);
                L += l_s[u][col] * wg[u];
            }
            // (in 64 bits, and the logarithm of the mantissa alone: a reference may lie 8 binary orders below the largest logit, and the terms
            // are the larger for it.  Root mean square error, 1985 tokens: 1.7e-7; in 32 bits 3.2e-7, with the largest logit 3.0e-7)
            int e;
            const float f = frexpf(L, &e);
            lse_out = (float)((double)mm * (double)a.scale + ((double)e * 0.6931471805599453 + (double)__logf(f)));
            const float inv = 1.f / L;
#pragma unroll
            for (int u = 0; u < NW; ++u) wg[u] *= inv;
        }
        float y[D / 32][4];
        bool bad = false;
#pragma unroll
        for (int n = 0; n < D / 32; ++n) {
            const int ch = (tid & 7) + 8 * n;
            f32x4 v[NW];
#pragma unroll
            for (int u = 0; u < NW; ++u) v[u] = part[(u * kTileCols + col) * (D / 4) + (ch ^ mc)];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                y[n][r] = BWD ? ((v[0][r] + v[1][r]) + (v[2][r] + v[3][r])) * a.scale
                              : v[0][r] * wg[0] + v[1][r] * wg[1] + v[2][r] * wg[2] + v[3][r] * wg[3];
                bad |= mine && !finite(y[n][r]);
            }
        }
        if (mine) {
            const int qh = h * G + mc % G;
            bf16_t *p = a.out + ((int64_t)(t.row0 + tc) * a.hq + qh) * D + 4 * (tid & 7);
#pragma unroll
            for (int n = 0; n < D / 32; ++n) store_row<bf16_t, 4>(p + 32 * n, y[n]);
            if (!BWD && a.lse != nullptr && (tid & 7) == 0) a.lse[qhead_row(a.map, qh, a.hq, t.row0 + tc)] = lse_out;
        }
        return bad;
    };
    pass(std::false_type{}, -1);
    if (tid == 0) s_bad = 0;
    if (__any(finish())) s_bad = 1;                      // (a barrier lies between the two)
    __syncthreads();
    if (s_bad == 0) return;
    for (int solo = 0; solo < t.ntok; ++solo) {
        all = 1u << solo;
        __syncthreads();                                 // the partial results have been read
        pass(std::true_type{}, solo);
        finish();
    }
}

template <int D, bool BWD>
int launch_t(const Launch &L, StagedArgs a, const int32_t *cu_h, const rules::Walks &walks) {
    constexpr size_t lds = (size_t)NW * 2 * Stage<D>::kBytes;
    static_assert(lds == (size_t)NW * kTileCols * D * sizeof(float), "the partial results take the stages' place");
    const int64_t tiles = walks.two;
    const int resident = D == 128 ? 512 : 768, hkv = L.p->num_kv_heads;
    a.resident = rules::back_and_forth(cu_h, L.map.batch, CG * tile_tokens(L.map, a.hq / hkv), tiles, hkv, a.idx != nullptr, a.topk_total, a.dense_below,
                                       walks.half_blocks, resident, true) ? resident : 0;
    void (*kern)(StagedArgs, int) = attn_staged_kernel<D, BWD>;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return INFLLMV2_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * hkv)), dim3(NW * 64), lds, L.stream, a, (int)tiles);
    return hip_status(hipGetLastError());
}

}  // namespace

bool attn_staged_takes(const Launch &L, const void *k, const void *v) {
    return L.p->dtype == INFLLMV2_BF16 && L.map.ctx == nullptr && (((uintptr_t)k | (uintptr_t)v) & 15) == 0 &&
           L.map.kv_tok_stride % 8 == 0 && L.map.kv_head_stride % 8 == 0;
}

int launch_attn_staged(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, void *out,
                       float *lse, const int32_t *cu_h, const rules::Walks &walks) {
    const StagedArgs a{(const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v, idx, L.p->topk_total, dense_below, L.p->num_q_heads,
                       L.p->softmax_scale, L.map, (bf16_t *)out, lse, nullptr, nullptr, 0};
    return L.p->head_dim == 128 ? launch_t<128, false>(L, a, cu_h, walks) : launch_t<64, false>(L, a, cu_h, walks);
}

int launch_dq_staged(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, const float *lse,
                     const float *delta, const void *dout, void *dq, const int32_t *cu_h, const rules::Walks &walks) {
    const StagedArgs a{(const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v, idx, L.p->topk_total, dense_below, L.p->num_q_heads,
                       L.p->softmax_scale, L.map, (bf16_t *)dq, const_cast<float *>(lse), (const bf16_t *)dout, delta, 0};
    return L.p->head_dim == 128 ? launch_t<128, true>(L, a, cu_h, walks) : launch_t<64, true>(L, a, cu_h, walks);
}

}  // namespace ifv2
