// Gradients of stage 4 -- block-sparse causal attention over a given selection (Appendix Alg. 2), or dense causal
// attention (Eq. 1) -- with respect to Q, K and V.  The selection of stages 1-3 only picks blocks (Sec. 3.3), so it
// carries no gradient and is an input here.  The paper gives no backward algorithm; this is the chain rule on
// O = softmax(z) V, z = scale * q k^T, using the log-sum-exp the forward pass stored (Alg. 2 keeps it for this):
//     p_u  = exp(z_u - lse)                     dp_u = <dO, v_u>             Delta = <dO, O> (= sum_u p_u dp_u)
//     dz_u = p_u (dp_u - Delta)                 dq   = scale * sum_u dz_u k_u
//     dk_u += scale * dz_u q                    dv_u += p_u dO               (summed over rows and over the group)
// This file: any G <= 16, d in {64, 128}, fp32 or bf16 data (the paper's head shape in bf16 takes the matrix-core path of
// attn_bwd_mfma.hip instead).  All weights and sums are fp32; the products run on the matrix cores as described in
// gen_unit.h.  Three kernels:
//   delta : Delta per (row, query head)
//   dq    : the workgroup and block walk of the generic forward kernel: per block S^T = K Q^T and dP^T = V dO^T
//           (keys x columns), dZ^T in registers, dQ^T += K^T dZ^T
//   dkv   : one workgroup of 4 wavefronts per (KV block, chunk of later tokens, KV head): lists the tokens of its chunk
//           that selected the block and takes 16 / G of them at a time, 16 rows of Q and dO (bf16: twice that); wavefront w holds keys
//           16 w .. 16 w + 15 (their K and V rows stay in registers): S = Q K^T, dP = dO V^T (rows x keys), then
//           dV += P^T dO and dK += dZ^T Q, contracted over the rows.  The block's 64 rows of dK and dV are added to
//           the float32 result with atomics (one add per element and workgroup; the order of the adds, and with it
//           the last bits of dK and dV, can differ from run to run).
// Measured, bf16, 1985 tokens, 8 heads on 2, d 128, 16 blocks: dq 87 -> 55 us (bound by the rows' trips from the L2, as the
// forward kernel: two column groups per wavefront, half blocks requested ahead), dkv 108 -> 103 -> 55 (bf16 kernel of its own, 79 us of it by
// its steps, 91 -> 55 by launching only the workgroups that have work); fp32, 2000 tokens, dkv 346 -> 251 with the products' operands and
// sums in vector registers.
#include <algorithm>

#include "attn_bwd.h"
#include "attn_staged.h"
#include "chunk_pairs.h"
#include "gen_unit.h"
#include "launch_rules.h"
#include "lds_rows.h"

namespace ifv2 {

namespace {

using namespace gen;

constexpr int NW = 4;               // wavefronts per workgroup of the dq and dkv kernels
constexpr int BWD_CHUNK = 256;      // most tokens a dkv workgroup looks at
constexpr int kWaitVm0 = 0x0F70;    // s_waitcnt vmcnt(0), other counters untouched

template <typename T>
struct BwdArgs {
    const T *q, *k, *v, *out, *dout;
    const float *lse;
    const int32_t *idx;         // nullptr: dense
    int topk_total, dense_below, hq;
    float scale;
    RowMap map;
    float *delta;               // [hq, T] scratch
    T *dq;
    float *dk, *dv;             // [hkv, T, D]
};

template <typename T, int D>
__global__ void __launch_bounds__(256) bwd_delta_kernel(BwdArgs<T> a) {
    // one wave per (row, query head)
    const int lane = threadIdx.x & 63;
    const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (item >= (int64_t)a.map.total_rows * a.hq) return;
    const int row = (int)(item / a.hq), qh = (int)(item % a.hq);
    const T *o = a.out + ((int64_t)row * a.hq + qh) * D, *g = a.dout + ((int64_t)row * a.hq + qh) * D;
    float s = 0.f;
    for (int c = lane; c < D; c += 64) s += Elem<T>::load(o + c) * Elem<T>::load(g + c);
    s = wave_sum(s);
    if (lane == 0) a.delta[qhead_row(a.map, qh, a.hq, row)] = s;
}

template <typename T, int D, int CG, bool AHEAD>
__global__ void __launch_bounds__(NW * 64) bwd_dq_kernel(BwdArgs<T> a) {
    constexpr int N = D / 16;
    __shared__ Union un;
    __shared__ float o_s[NW][CG * kCols][D + 4];
    __shared__ int s_tile[3];
    const int h = blockIdx.y, G = a.hq / a.map.num_kv_heads;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    Tile t;
    if (!find_tile(a.map, gridDim.x - 1 - blockIdx.x, CG * tile_tokens(a.map, G), t, s_tile)) return;
    const bool dense = a.idx == nullptr || t.len < a.dense_below;
    const int32_t *lists = dense ? nullptr : a.idx + head_row(a.map, h, t.row0) * a.topk_total;
    const int nblk = (t.t0 + t.ntok - 1) / kBlock + 1;
    const T *kb = a.k + t.kv_base + (int64_t)h * a.map.kv_head_stride;
    const T *vb = a.v + t.kv_base + (int64_t)h * a.map.kv_head_stride;

    const int m = lane & 15, g = lane >> 4;
    const int tokens = tile_tokens(a.map, G);
    int ti[CG];
    bool used[CG];
    RowFrag<T, D> qf[CG], gf[CG];
    float lse[CG], delta[CG];
#pragma unroll
    for (int x = 0; x < CG; ++x) {
        ti[x] = x * tokens + m / G;
        used[x] = m / G < tokens && ti[x] < t.ntok;
        const int row = t.row0 + (used[x] ? ti[x] : 0), qh = h * G + (used[x] ? m % G : 0);
        qf[x].load(a.q + ((int64_t)row * a.hq + qh) * D, g);
        gf[x].load(a.dout + ((int64_t)row * a.hq + qh) * D, g);
        lse[x] = a.lse[qhead_row(a.map, qh, a.hq, row)];
        delta[x] = a.delta[qhead_row(a.map, qh, a.hq, row)];
    }
    const KeyRows<T, D> krows(kb, a.map.kv_tok_stride, t.len, m, g), vrows(vb, a.map.kv_tok_stride, t.len, m, g);

    // as in the forward kernel: one pass for all tokens of the tile, and again token by token with the K rows that a
    // token does not see taken as 0 if something came out that is not finite (0 x infinity)
    uint32_t all = t.ntok == 32 ? ~0u : (1u << t.ntok) - 1u;
    int solo = -1;
    for (;;) {
        f32x4 acc[CG][N];                                // dQ^T: dim N (4 g + r) + j, this lane's column
#pragma unroll
        for (int x = 0; x < CG; ++x)
#pragma unroll
            for (int j = 0; j < N; ++j) acc[x][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int c0 = 0; c0 < nblk; c0 += kChunk) {
            un.build(lists, a.topk_total, t, c0, nblk, all, tid, NW * 64);
            const int items = un.half_blocks(t);
            RowFrag<T, D> kf[2], vf[2];
            Spread<T, D> kr[2][4];
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
                vrows.frags(vf, u0, m, g);
                krows.spread(kr, u0, m, g);
            }
            for (int it = w; it < items; it += NW) {
                if (!AHEAD) {
                    u0 = key_of(it);
                    krows.frags(kf, u0, m, g);
                    vrows.frags(vf, u0, m, g);
                }
                f32x4 s[CG][2], dp[CG][2];
#pragma unroll
                for (int x = 0; x < CG; ++x)
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt) {
                        s[x][kt] = row_product<D>(kf[kt], qf[x]);
                        dp[x][kt] = row_product<D>(vf[kt], gf[x]);
                    }
                const int here = u0;
                const uint32_t takers = (uint32_t)ent.y;
                const bool more = AHEAD && it + NW < items;
                if (!AHEAD) krows.spread(kr, u0, m, g);
                if (more) {                              // the next half block's rows, while this one's weights are formed
                    u0 = key_of(it + NW);
                    krows.frags(kf, u0, m, g);
                    vrows.frags(vf, u0, m, g);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (solo >= 0) {
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (here + 16 * kt + 4 * g + r > t.t0 + solo) kr[kt][r].zero();
                }
#pragma unroll
                for (int x = 0; x < CG; ++x) {
                    if (CG > 1 && ((takers >> (x * tokens)) & ((1u << tokens) - 1u)) == 0u) continue;
                    const int lim = used[x] && ((takers >> ti[x]) & 1u) ? t.t0 + ti[x] - here : -1;   // last visible key
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float p = exp2_fast(__builtin_fmaf(s[x][kt][r], a.scale, -lse[x]) * kLog2e);
                            s[x][kt][r] = 16 * kt + 4 * g + r <= lim ? p * (dp[x][kt][r] - delta[x]) : 0.f;
                        }
                    weighted_rows32<false, true, D>(acc[x], s[x][0], s[x][1], kr[0], kr[1]);
                }
                if (more) krows.spread(kr, u0, m, g);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
        }
#pragma unroll
        for (int x = 0; x < CG; ++x)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < N; ++j) o_s[w][x * kCols + m][N * (4 * g + r) + j] = acc[x][j][r];
        __syncthreads();
        static_assert(NW * 64 == kCols * 16, "sixteen threads per column");
        const int d0 = (tid & 15) * N;
        float y[CG][N];
        bool bad = false;
#pragma unroll
        for (int x = 0; x < CG; ++x) {
            const int col = x * kCols + (tid >> 4), tc = x * tokens + (tid >> 4) / G;
            const bool mine = (tid >> 4) / G < tokens && tc < t.ntok && ((all >> tc) & 1u);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                y[x][j] = ((o_s[0][col][d0 + j] + o_s[1][col][d0 + j]) + (o_s[2][col][d0 + j] + o_s[3][col][d0 + j])) * a.scale;
                bad |= mine && !finite(y[x][j]);
            }
        }
        const bool again = solo < 0 && __syncthreads_or(bad);
        if (!again) {
#pragma unroll
            for (int x = 0; x < CG; ++x) {
                const int tc = x * tokens + (tid >> 4) / G;
                if ((tid >> 4) / G < tokens && tc < t.ntok && ((all >> tc) & 1u))
                    store_row<T, N>(a.dq + ((int64_t)(t.row0 + tc) * a.hq + h * G + (tid >> 4) % G) * D + d0, y[x]);
            }
        }
        if (solo < 0 && !again) return;
        if (++solo >= t.ntok) return;
        all = 1u << solo;
        __syncthreads();
    }
}

// Workgroups of the dkv kernels: (token chunk, KV block) pairs with at least one token that can see the block.  Nothing else is
// launched: in a grid of all pairs half of the workgroups are empty, and as these come at regular intervals while workgroups are
// dealt out in turn to the dies and to the engines of a die, some engines got several times the work of others (1985 tokens, 8 heads on
// 2, chunks of 64: the workgroups' times sum up to 42 us of the chip and took 91 from first to last; whole backward 149 -> 140 us).
// Sequence (>= batch past the last pair), chunk and block of this workgroup; s_tile: 3 ints of LDS.  ONE chunk holds every sequence: a
// workgroup is a block, as cheap to find in a batch as a tile (2000 sequences of one token, 8 heads on 2, d 64, bf16: dkv 54 -> 49 us).
__device__ inline int dkv_place(const RowMap &m, int shift, bool one, int &chunk, int &block, int *s_tile) {
    int nth, before;
    const int seq = find_seq_count(m.cu, m.batch, (int)(blockIdx.y * gridDim.x + blockIdx.x), nth, before, s_tile,
                                   [&](int n) { return one ? (n + kBlock - 1) / kBlock : sequence_pairs(n, shift); }, [](int) { return 0; });
    chunk = 0;
    block = nth;
    if (!one && seq < m.batch) pair_at(nth, shift, chunk, block);
    return seq;
}

// is block j in the list e[0 .. n)?  Short lists whole (a search is a chain of five or six trips to memory)
__device__ inline bool selected(const int32_t *e, int n, int j) {
    if (n > 64) return list_has(e, n, j);
    typedef int32_t Four __attribute__((ext_vector_type(4), aligned(4)));
    bool hit = false;
    int i = 0;
    for (; i + 16 <= n; i += 16) {
        Four x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = *reinterpret_cast<const Four *>(e + i + 4 * u);
#pragma unroll
        for (int u = 0; u < 4; ++u) hit |= x[u][0] == j || x[u][1] == j || x[u][2] == j || x[u][3] == j;
    }
    for (; i < n; ++i) hit |= e[i] == j;
    return hit;
}

template <typename T, int D>
__global__ void __launch_bounds__(NW * 64) bwd_dkv_kernel(BwdArgs<T> a, int shift, bool one) {
    constexpr int N = D / 16;
    constexpr int ROWS = kCols;                                        // of Q and dO per step
    __shared__ __attribute__((aligned(16))) T rows_s[2][2][ROWS][D + 16 / sizeof(T)];      // [buffer][Q, dO][row]
    __shared__ float lse_s[2][ROWS], delta_s[2][ROWS];
    __shared__ int t_s[2][ROWS];
    __shared__ int s_tile[3], s_list[BWD_CHUNK], s_wave_cnt[NW];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int h = blockIdx.z, G = a.hq / a.map.num_kv_heads;
    int j, at;
    const int seq = dkv_place(a.map, shift, one, at, j, s_tile);
    if (seq >= a.map.batch) return;
    const int tok0 = a.map.cu[seq], len = a.map.cu[seq + 1] - tok0;
    // tokens of this chunk that can see the block: [max(chunk start, 64 j), min(chunk end, len))
    const int c0 = at << shift, c1 = min(c0 + (1 << shift), len);
    const bool dense = a.idx == nullptr || len < a.dense_below;

    // ---- which tokens of the chunk selected the block (in token order); a chunk has at most one token per thread
    const int t_mine = c0 + tid;
    bool sel = t_mine < c1 && t_mine >= j * kBlock;
    if (sel && !dense) sel = selected(a.idx + head_row(a.map, h, tok0 + t_mine) * a.topk_total, a.topk_total, j);
    const uint64_t bal = __ballot(sel);
    if (lane == 0) s_wave_cnt[w] = __popcll(bal);
    __syncthreads();
    int base = 0, total = 0;
    for (int x = 0; x < NW; ++x) {
        if (x < w) base += s_wave_cnt[x];
        total += s_wave_cnt[x];
    }
    if (sel) s_list[base + __popcll(bal & ((1ull << lane) - 1ull))] = t_mine;
    if (total == 0) return;
    __syncthreads();

    // ---- the wavefront's 16 keys: K and V rows as operands (past the end of the sequence: the last row, never visible)
    const int m = lane & 15, g = lane >> 4;
    const int key = j * kBlock + 16 * w + m;
    const int64_t kv_off = (int64_t)(tok0 + min(key, len - 1)) * a.map.kv_tok_stride + (int64_t)h * a.map.kv_head_stride;
    RowFrag<T, D> kf, vf;
    kf.load(a.k + kv_off, g);
    vf.load(a.v + kv_off, g);
    f32x4 acc_k[N], acc_v[N];                                  // keys 16 w + 4 g + r, dim N m + i
#pragma unroll
    for (int i = 0; i < N; ++i) acc_k[i] = acc_v[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A step is the list's next `tokens` entries with their G heads: row x is entry x / G, head x % G.  The four
    // wavefronts need the same rows of Q and dO twice (as row operands and spread over lanes), so they pass through
    // LDS once: thread (row, part) brings a sixteenth of its row, the next step's in flight in registers while
    // the current one is computed; one barrier per step.  Unused rows hold zeros and see no key.
    const int tokens = kCols / G;
    const int x_row = tid >> 4, x_slot = x_row / G, x_head = h * G + x_row - x_slot * G;
    struct Pre { Spread<T, D> q, g; float lse, delta; int t; };
    auto fetch = [&](int it) -> Pre {
        Pre pr;
        const int e = it + x_slot;
        const bool used = x_slot < tokens && e < total;
        const int t = s_list[used ? e : 0];
        const int64_t off = ((int64_t)(tok0 + t) * a.hq + (used ? x_head : h * G)) * D;
        pr.q.load(a.q + off, tid & 15);
        pr.g.load(a.dout + off, tid & 15);
        const int64_t lr = qhead_row(a.map, used ? x_head : h * G, a.hq, tok0 + t);
        pr.lse = a.lse[lr];
        pr.delta = a.delta[lr];
        pr.t = used ? t : -1;
        return pr;
    };
    // (unused rows become zeros here: where they are requested it would mean to wait for them, half a microsecond of each step)
    auto stage = [&](int buf, Pre &pr) {
        if (pr.t < 0) { pr.q.zero(); pr.g.zero(); }
        pr.q.store_lds(&rows_s[buf][0][x_row][0], tid & 15);
        pr.g.store_lds(&rows_s[buf][1][x_row][0], tid & 15);
        if ((tid & 15) == 0) {
            lse_s[buf][x_row] = pr.lse;
            delta_s[buf][x_row] = pr.delta;
            t_s[buf][x_row] = pr.t;
        }
    };
    {
        Pre first = fetch(0);
        stage(0, first);
    }
    // (the keys' own rows, requested first, are waited for here: left to the compiler that wait stands in the loop's first products, where it also
    // waits for the rows just requested for the next step)
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
    int buf = 0;
    for (int it = 0; it < total; it += tokens, buf ^= 1) {
        const bool more = it + tokens < total;
        Pre nxt;
        if (more) nxt = fetch(it + tokens);
        RowFrag<T, D> qf, gf;
        qf.load_lds(&rows_s[buf][0][m][0], g);
        gf.load_lds(&rows_s[buf][1][m][0], g);
        const f32x4 s = row_product<D>(qf, kf);
        const f32x4 dp = row_product<D>(gf, vf);
        f32x4 p, dz;
        Spread<T, D> qr[4], gr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int x = 4 * g + r;
            p[r] = exp2_fast(__builtin_fmaf(s[r], a.scale, -lse_s[buf][x]) * kLog2e);
            dz[r] = p[r] * (dp[r] - delta_s[buf][x]);
            asm volatile("" : "+v"(p[r]), "+v"(dz[r]));        // (no branch round the hidden ones: six waits for LDS, one after the other)
            qr[r].load_lds(&rows_s[buf][0][x][0], m);
            gr[r].load_lds(&rows_s[buf][1][x][0], m);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool vis = key <= t_s[buf][4 * g + r];
            p[r] = vis ? p[r] : 0.f;
            dz[r] = vis ? dz[r] : 0.f;
        }
        if constexpr (sizeof(T) == 2) {                        // 16 of the 32 indices; the others are 0 times 0
            const f32x4 none = {0.f, 0.f, 0.f, 0.f};
            Spread<T, D> zeros[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) zeros[r].zero();
            weighted_rows32<true, true, D>(acc_v, p, none, gr, zeros);
            weighted_rows32<true, true, D>(acc_k, dz, none, qr, zeros);
        } else {
            weighted_rows<true, D>(acc_v, p, gr);
            weighted_rows<true, D>(acc_k, dz, qr);
        }
        if (more) stage(buf ^ 1, nxt);
        __syncthreads();
    }
    // Results through LDS (the row stages are free now), so that the 64 lanes of an atomic add cover consecutive
    // addresses: as the accumulators lie, neighbouring lanes are N floats apart and an add would touch a cache line per
    // two lanes.
    float *tr = reinterpret_cast<float *>(&rows_s[0][0][0][0]) + w * (4 * (D + 4));
    static_assert(sizeof(rows_s) >= NW * 4 * (D + 4) * sizeof(float), "four rows per wavefront");
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        float *dst = which ? a.dv : a.dk;
#pragma unroll
        for (int r = 0; r < 4; ++r) {                              // keys 16 w + 4 g + r, g = 0 .. 3
#pragma unroll
            for (int i = 0; i < N; ++i) tr[g * (D + 4) + N * m + i] = which ? acc_v[i][r] : acc_k[i][r] * a.scale;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                const int u = j * kBlock + 16 * w + 4 * y + r;
                if (u < len) {
                    float *p = dst + ((int64_t)h * a.map.total_rows + tok0 + u) * D;
#pragma unroll
                    for (int d0 = 0; d0 < D; d0 += 64) unsafeAtomicAdd(p + d0 + lane, tr[y * (D + 4) + d0 + lane]);    // the L2's own float add
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// dK and dV of bf16 rows.  As above, with everything arranged for few instructions: with two wavefronts on a SIMD a step of 32 rows in the form
// above took 2.84 us, 500 vector instructions per wavefront; this one 2.5 us, 310 (2.1 without its loads from memory):
//   * a step is 32 rows, 32 / 16 times 16 / G tokens, staged in LDS (lds_rows.h) so that a lane's eight weights are the operand of
//     the second products as it is, whose other operand (the same rows, transposed) comes from transposing LDS reads: no
//     spread rows, no byte permutes;
//   * dP starts at -Delta; keys are hidden only in steps with tokens of the block itself; weights are checked for infinities
//     once per step and cut into pieces without checks otherwise;
//   * an accumulator register holds 16 consecutive dims of 4 keys, whole 64-byte pieces, so the adds leave the registers as they are.
using lds_rows::kRowBytes;                                             // (d 64: half of it used)

template <int D>
__global__ void __launch_bounds__(NW * 64, 2) bwd_dkv_bf16_kernel(BwdArgs<bf16_t> a, int shift, bool one) {
    constexpr int N = D / 16, ROWS = 32;
    constexpr uint32_t kTile = ROWS * kRowBytes, kBuf = 2 * kTile;     // Q rows, then dO rows
    __shared__ __attribute__((aligned(1024))) char rows_s[2 * kBuf];
    __shared__ __attribute__((aligned(16))) float lse_s[2][ROWS], delta_s[2][ROWS];      // -lse and -Delta
    __shared__ __attribute__((aligned(16))) int t_s[2][ROWS];
    __shared__ int s_tile[3], s_list[BWD_CHUNK], s_wave_cnt[NW], s_own_cnt[NW];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.z, G = a.hq / a.map.num_kv_heads;
    int j, at;
    const int seq = dkv_place(a.map, shift, one, at, j, s_tile);
    if (seq >= a.map.batch) return;
    const int tok0 = a.map.cu[seq], len = a.map.cu[seq + 1] - tok0;
    // tokens of this chunk that can see the block: [max(chunk start, 64 j), min(chunk end, len))
    const int c0 = at << shift, c1 = min(c0 + (1 << shift), len);
    const bool dense = a.idx == nullptr || len < a.dense_below;

    // ---- which tokens of the chunk selected the block (in token order); a chunk has at most one token per thread
    const int t_mine = c0 + tid;
    bool sel = t_mine < c1 && t_mine >= j * kBlock;
    if (sel && !dense) sel = selected(a.idx + head_row(a.map, h, tok0 + t_mine) * a.topk_total, a.topk_total, j);
    // the wavefront's 16 keys: K and V rows as operands (past the end of the sequence: the last row, never visible)
    const int m = lane & 15, g = lane >> 4;
    const int key = j * kBlock + 16 * w + m;
    const int64_t kv_off = (int64_t)(tok0 + min(key, len - 1)) * a.map.kv_tok_stride + (int64_t)h * a.map.kv_head_stride;
    RowFrag<bf16_t, D> kf, vf;
    kf.load(a.k + kv_off, g);
    vf.load(a.v + kv_off, g);
    const uint64_t bal = __ballot(sel);
    const uint64_t own_bal = __ballot(sel && t_mine < (j + 1) * kBlock);
    if (lane == 0) {
        s_wave_cnt[w] = __popcll(bal);
        s_own_cnt[w] = __popcll(own_bal);
    }
    __syncthreads();
    int base = 0, total = 0, own = 0;                         // own: tokens of the block itself, the first of the list
    for (int x = 0; x < NW; ++x) {
        if (x < w) base += s_wave_cnt[x];
        total += s_wave_cnt[x];
        own += s_own_cnt[x];
    }
    if (sel) s_list[base + __popcll(bal & ((1ull << lane) - 1ull))] = t_mine;
    total = __builtin_amdgcn_readfirstlane(total);
    own = __builtin_amdgcn_readfirstlane(own);
    if (total == 0) return;
    __syncthreads();

    f32x4 acc_k[N], acc_v[N];                                  // keys 16 w + 4 g + r, dim 16 i + m
#pragma unroll
    for (int i = 0; i < N; ++i) acc_k[i] = acc_v[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Thread (x, part) brings sixteenth `part` of rows x and 16 + x: head x % G of the list's entries x / G and tokens + x / G behind the
    // step's first.  The next step's are in flight in registers while the current one is computed; one barrier per step.
    // Unused rows hold zeros and see no key.
    const int tokens = kCols / G;
    const int x_row = tid >> 4, part = tid & 15, x_slot = x_row / G, x_head = h * G + (x_slot < tokens ? x_row - x_slot * G : 0);
    typedef uint32_t Part __attribute__((ext_vector_type(D / 32), aligned(2)));             // a sixteenth of a row, wherever it lies
    struct Pre { Part q[2], g[2]; float lse[2], delta[2]; int t[2]; };
    const int64_t row0 = ((int64_t)tok0 * a.hq + x_head) * D + part * N, lr0 = (int64_t)x_head * a.map.total_rows + tok0;
    const bf16_t *qp = a.q + row0, *gp = a.dout + row0;
    const float *lp = a.lse + lr0, *dp0 = a.delta + lr0;
    const int t_step = a.hq * D;                               // elements from token to token
    auto whole = [&](int it) { return it + 2 * tokens <= total && tokens * G == kCols; };     // no unused rows
    auto fetch = [&](int it) -> Pre {
        Pre pr;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int t = s_list[min(it + i * tokens + x_slot, total - 1)];
            pr.q[i] = *reinterpret_cast<const Part *>(qp + (int64_t)t * t_step);
            pr.g[i] = *reinterpret_cast<const Part *>(gp + (int64_t)t * t_step);
            pr.lse[i] = -lp[t];
            pr.delta[i] = -dp0[t];
            pr.t[i] = t;
        }
        return pr;
    };
    auto drop_unused = [&](int it, Pre &pr) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (x_slot >= tokens || it + i * tokens + x_slot >= total) {
                pr.q[i] = pr.g[i] = 0u;
                pr.t[i] = -1;
            }
    };
    auto stage = [&](int buf, const Pre &pr) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = i * kCols + x_row;
            typedef uint32_t LPart __attribute__((ext_vector_type(D / 32), aligned(D / 8)));
            char *p = rows_s + buf * kBuf + row * kRowBytes + (((D == 128 ? part : part >> 1) ^ lds_rows::swizzle(row)) << 4) + (D == 128 ? 0 : part & 1) * 8;
            *reinterpret_cast<LPart *>(p) = pr.q[i];
            *reinterpret_cast<LPart *>(p + kTile) = pr.g[i];
            if (part == 0) {
                lse_s[buf][row] = pr.lse[i];
                delta_s[buf][row] = pr.delta[i];
                t_s[buf][row] = pr.t[i];
            }
        }
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)rows_s;
    const uint32_t row_at = lds0 + lds_rows::offset(lds_rows::operand_row(m), g);
    const uint32_t trans_at = lds0 + lds_rows::offset(lds_rows::piece_row(m, g), lds_rows::piece_chunk(m)) + lds_rows::piece_half(m);
    // acc += weights^T x rows, weights in three exact pieces (see weighted_rows32)
    auto accumulate = [&](f32x4 (&acc)[N], f32x4 w0, f32x4 w1, uint32_t at) {
        float top = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) top = fmaxf(top, fmaxf(fabsf(w0[r]), fabsf(w1[r])));
        bf16x8 p0, p1, p2;
        if (__any(top == INFINITY)) {
            p0 = take_piece32<true>(w0, w1);
            p1 = take_piece32<true>(w0, w1);
            p2 = take_piece32<true>(w0, w1);
        } else {
            p0 = take_piece32<false>(w0, w1);
            p1 = take_piece32<false>(w0, w1);
            p2 = take_piece32<false>(w0, w1);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const bf16x8 rows = lds_rows::transposed(at ^ (uint32_t)(32 * i));
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p2, rows, acc[i], 0, 0, 0);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p1, rows, acc[i], 0, 0, 0);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p0, rows, acc[i], 0, 0, 0);
        }
    };
    {
        Pre first = fetch(0);
        if (!whole(0)) drop_unused(0, first);
        stage(0, first);
    }
    __syncthreads();
    int buf = 0;
    for (int it = 0; it < total; it += 2 * tokens, buf ^= 1) {
        const bool more = it + 2 * tokens < total;
        Pre nxt;
        if (more) nxt = fetch(it + 2 * tokens);
        const uint32_t ra = row_at + buf * kBuf, ta = trans_at + buf * kBuf;
        f32x4 p[2], dz[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            f32x4 s = {0.f, 0.f, 0.f, 0.f};
            f32x4 dp = *reinterpret_cast<const f32x4 *>(&delta_s[buf][8 * g + 4 * kt]);
#pragma unroll
            for (int ks = 0; ks < D / 32; ++ks) {
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds_rows::operand(ra, kt, ks), kf.x[ks], s, 0, 0, 0);
                dp = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds_rows::operand(ra + kTile, kt, ks), vf.x[ks], dp, 0, 0, 0);
            }
            const f32x4 nl = *reinterpret_cast<const f32x4 *>(&lse_s[buf][8 * g + 4 * kt]);
#pragma unroll
            for (int r = 0; r < 4; ++r) p[kt][r] = exp2_fast(__builtin_fmaf(s[r], a.scale, nl[r]) * kLog2e);
            dz[kt] = dp;
        }
        if (it < own || !whole(it)) {                          // hidden keys, unused rows

#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool vis = key <= t_s[buf][8 * g + 4 * kt + r];
                    p[kt][r] = vis ? p[kt][r] : 0.f;
                    dz[kt][r] = vis ? dz[kt][r] : 0.f;
                }
        }
        accumulate(acc_v, p[0], p[1], ta + kTile);
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) dz[kt] *= p[kt];
        accumulate(acc_k, dz[0], dz[1], ta);
        if (more) {
            if (!whole(it + 2 * tokens)) drop_unused(it + 2 * tokens, nxt);
            stage(buf ^ 1, nxt);
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int u = j * kBlock + 16 * w + 4 * g + r;
        if (u >= len) continue;
        const int64_t at = ((int64_t)h * a.map.total_rows + tok0 + u) * D + m;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            unsafeAtomicAdd(a.dk + at + 16 * i, acc_k[i][r] * a.scale);      // the L2's own float add
            unsafeAtomicAdd(a.dv + at + 16 * i, acc_v[i][r]);
        }
    }
}

// dk[0 .. n) = dv[0 .. n) = 0 by one launch; n % 4 == 0, both 16-byte aligned
__global__ void __launch_bounds__(256) bwd_zero_kernel(float4 *dk, float4 *dv, int64_t n4) {
    float4 *p = blockIdx.y ? dv : dk;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256)
        p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

template <typename T, int D, int CG, bool AHEAD>
void launch_dq(const Launch &L, const BwdArgs<T> &a) {
    const int tokens = CG * tile_tokens(L.map, a.hq / L.map.num_kv_heads);
    // at most this many tiles (every sequence may end with a partial one)
    hipLaunchKernelGGL((bwd_dq_kernel<T, D, CG, AHEAD>), dim3((unsigned)(L.map.total_rows / tokens + L.map.batch), L.map.num_kv_heads),
                       dim3(NW * 64), 0, L.stream, a);
}

template <typename T, int D>
int launch_t(const Launch &L, BwdArgs<T> a, const int32_t *cu_h) {
    const int64_t rows = L.map.total_rows;
    if (rows == 0) return INFLLMV2_OK;
    int64_t nblocks = 0;
    for (int s = 0; s < L.map.batch; ++s) nblocks += (cu_h[s + 1] - cu_h[s] + kBlock - 1) / kBlock;
    const int hkv = L.p->num_kv_heads;
    // grid.z; and what the (chunk, block) pairs' 32 bits hold (one sequence of 65535 blocks: 537 million pairs with chunks of 256 tokens)
    if (nblocks > 65535 || hkv > 65535) return INFLLMV2_ERR_UNSUPPORTED;
    void *ws = L.ws;         // <dO, O> per (row, head)
    if (ws == nullptr || L.ws_bytes < (size_t)rows * a.hq * sizeof(float)) return INFLLMV2_ERR_WORKSPACE_TOO_SMALL;
    a.delta = (float *)ws;
    const int64_t n4 = rows * hkv * D / 4;
    hipLaunchKernelGGL(bwd_zero_kernel, dim3((unsigned)std::min<int64_t>((n4 + 255) / 256, 8192), 2), dim3(256), 0, L.stream,
                       (float4 *)a.dk, (float4 *)a.dv, n4);
    hipLaunchKernelGGL((bwd_delta_kernel<T, D>), dim3((unsigned)((rows * a.hq + 3) / 4)), dim3(256), 0, L.stream, a);
    const rules::Walks x = rules::walks(cu_h, L.map.batch, tile_tokens(L.map, a.hq / hkv), a.idx != nullptr, a.topk_total, a.dense_below);
    const rules::GenericForm form = rules::generic_dq_form(sizeof(T) == 2, D, hkv, x);
    const bool two = D * sizeof(T) < 512 && form.groups == 2;
    if (sizeof(T) == 2 && rules::staged(true, D, x.two * hkv, x) && attn_staged_takes(L, a.k, a.v)) {
        const int st = launch_dq_staged(L, a.q, a.k, a.v, a.idx, a.dense_below, a.lse, a.delta, a.dout, a.dq, cu_h, x);
        if (st != INFLLMV2_OK) return st;
    } else {
        if constexpr (D * sizeof(T) < 512)
            if (two) launch_dq<T, D, 2, true>(L, a);
        if (!two && form.ahead) launch_dq<T, D, 1, true>(L, a);
        if constexpr (D * sizeof(T) < 512)
            if (!two && !form.ahead) launch_dq<T, D, 1, false>(L, a);
    }
    int64_t pairs;
    const int shift = rules::generic_dkv_shift(sizeof(T) == 2, D, a.hq / hkv, {cu_h, L.map.batch, L.max_len, hkv, nblocks, a.idx != nullptr,
                                               a.topk_total, a.dense_below}, pairs);
    const bool one = L.max_len <= 1 << shift;
    const int64_t gx = std::min<int64_t>(pairs, 1 << 20);
    const dim3 grid((unsigned)gx, (unsigned)((pairs + gx - 1) / gx), hkv);
    if constexpr (sizeof(T) == 2) {
        const bool few = rules::dkv_short_steps(D, a.hq / hkv, L.max_len, nblocks * hkv);
        if (few) hipLaunchKernelGGL((bwd_dkv_kernel<T, 64>), grid, dim3(NW * 64), 0, L.stream, a, shift, one);
        else hipLaunchKernelGGL((bwd_dkv_bf16_kernel<D>), grid, dim3(NW * 64), 0, L.stream, a, shift, one);
    } else {
        hipLaunchKernelGGL((bwd_dkv_kernel<T, D>), grid, dim3(NW * 64), 0, L.stream, a, shift, one);
    }
    return hip_status(hipGetLastError());
}

template <typename T>
int launch_d(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below,
             const void *out, const float *lse, const void *dout, void *dq, float *dk, float *dv, const int32_t *cu_h) {
    BwdArgs<T> a{(const T *)q, (const T *)k, (const T *)v, (const T *)out, (const T *)dout, lse, idx,
                 L.p->topk_total, dense_below, L.p->num_q_heads, L.p->softmax_scale, L.map, nullptr, (T *)dq, dk, dv};
    return L.p->head_dim == 128 ? launch_t<T, 128>(L, a, cu_h) : launch_t<T, 64>(L, a, cu_h);
}

}  // namespace

// matrix-core path for the paper's head shape (attn_bwd_mfma.hip); INFLLMV2_ERR_UNSUPPORTED = not covered
int launch_attn_bwd_mfma(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx,
                         int dense_below, const void *out, const float *lse, const void *dout, void *dq, float *dk,
                         float *dv, const int32_t *cu_h);

bool bwd_mfma_params(const infllmv2_params *p);
size_t bwd_mfma_ws_bytes(const infllmv2_params *p, const BatchTotals &t, bool with_bitmap);

size_t attn_bwd_ws_bytes(const infllmv2_params *p, const BatchTotals &t, bool with_bitmap) {
    // (a call whose pointers or strides rule out the matrix-core path needs less: the bound still holds)
    if (bwd_mfma_params(p)) return bwd_mfma_ws_bytes(p, t, with_bitmap);
    return align256((size_t)t.rows * p->num_q_heads * sizeof(float));
}

int launch_attn_bwd(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below,
                    const void *out, const float *lse, const void *dout, void *dq, float *dk, float *dv,
                    const int32_t *cu_h) {
    const int st = launch_attn_bwd_mfma(L, q, k, v, idx, dense_below, out, lse, dout, dq, dk, dv, cu_h);
    if (st != INFLLMV2_ERR_UNSUPPORTED) return st;
    return L.p->dtype == INFLLMV2_BF16
               ? launch_d<bf16_t>(L, q, k, v, idx, dense_below, out, lse, dout, dq, dk, dv, cu_h)
               : launch_d<float>(L, q, k, v, idx, dense_below, out, lse, dout, dq, dk, dv, cu_h);
}

}  // namespace ifv2
