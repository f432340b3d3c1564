// Stage 2: S^shared = sum over the GQA group of softmax(scale * Q K^{C1 T})  (Sec. 3.3 Eq. 4-5).
// Both kernels follow the two-pass scheme of Alg. 1 / Sec. 3.4: pass 1 finds the log-sum-exp of
// every (token, head) row on chip, pass 2 recomputes the logits, normalises, sums the G heads of
// the group on chip and stores only the group sum.  Per-head score rows never reach HBM.
//
// LSE Approximation (Sec. 3.4, Eq. 7; lse_mode 1): pass 1 runs over the four times coarser keys K^{C2}
// instead.  K^{C2}_i is the mean of 4 l_C1 keys starting at 4 s_C1 i, i.e. (when s_C1 divides l_C1) the mean of
// the four disjoint K^{C1} windows 4i + m l_C1 / s_C1, m = 0..3, so it is formed on the fly from K^{C1} and
// needs no input of its own.  A row that sees no coarse key gets all-zero scores.

#include <type_traits>

#include "gen_unit.h"

namespace ifv2 {

// ------------------------------------------------------------------------------------------
// Generic kernel: any G <= 16, d in {64,128}, fp32 or bf16 inputs.  Used for fp32 data, unusual head shapes and
// single-row (decode) calls.
//
// A workgroup owns a tile of 16 / G consecutive tokens of one KV head (16 columns, see gen_unit.h); the logits are
// float32 products (16x16x4) of the compressed keys and the queries widened to fp32.  Pass 1: the wavefronts take the
// key tiles in turn and keep a running (max, sum) per column, merged through LDS.  Pass 2 goes through the keys in
// chunks of 256: each wavefront recomputes the logits of 64, sums the G heads of every token through a small LDS tile,
// and the chunk's group scores are stored from LDS, one row per token -- or, with the pooling of Eq. 6, the maxima of
// the windows that start in it (a chunk then begins where the first window of the next blocks does, so windows never
// straddle chunks; the few keys between are computed twice).  fp32, 2048 tokens, 4 heads on 1, d 64: 80 -> 9.7 us (one
// workgroup per token and vector arithmetic before).
// ------------------------------------------------------------------------------------------
namespace {
constexpr int GS_WAVES = 4, GS_CHUNK = 64 * GS_WAVES;      // keys per pass-2 chunk
}

template <typename T, int D>
__global__ void __launch_bounds__(GS_WAVES * 64)
block_scores_generic(const T *__restrict__ q, const float *__restrict__ kc, RowMap map, int hq, int lc, int sc,
                     float scale, int dense_below, int lse_mode, float *__restrict__ s_shared, int64_t row_stride,
                     PoolArgs pool) {
    using namespace gen;
    constexpr int NT = GS_WAVES * 64;
    __shared__ float red_m[GS_WAVES][kCols], red_l[GS_WAVES][kCols];
    __shared__ float ps[GS_WAVES][16][kCols + 1];          // probabilities of one key tile, per wavefront
    __shared__ float sh[kCols][GS_CHUNK];                  // group scores of the chunk, per token
    __shared__ int s_tile[3];
    const int h = blockIdx.y, G = hq / map.num_kv_heads;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    Tile t;
    if (!find_tile(map, blockIdx.x, tile_tokens(map, G), t, s_tile)) return;
    if (t.len < dense_below) return;                       // dense sequences need no scores
    const int v_max = visible_cmp(t.t0 + t.ntok - 1, lc, sc);
    if (v_max == 0) return;
    const int m = lane & 15, g = lane >> 4;
    const int ti = m / G;
    const bool used = ti < t.ntok;
    const int pos = t.t0 + (used ? ti : 0);
    const float c = scale * kLog2e;
    RowFrag<float, D> qf;
    qf.load(q + ((int64_t)(t.row0 + (used ? ti : 0)) * hq + h * G + (used ? m - ti * G : 0)) * D, g);
    const float *kcb = kc_base(map, kc, t.seq, h, D);

    // ---- pass 1 over the fine keys, or the coarse ones made of `cstep`-spaced groups of four
    const int cstep = lc / sc;
    auto visible1 = [&](int p) -> int {
        return lse_mode == 0 ? visible_cmp(p, lc, sc) : min(visible_cmp(p, 4 * lc, 4 * sc), num_cmp(t.len, 4 * lc, 4 * sc));
    };
    const int v1 = used ? visible1(pos) : 0, v1_max = visible1(t.t0 + t.ntok - 1);
    float m_run = -INFINITY, l_run = 0.f;
    for (int k0 = 32 * w; k0 < v1_max; k0 += 32 * GS_WAVES) {
        f32x4 s[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int key = min(k0 + 16 * u + m, v1_max - 1);
            RowFrag<float, D> kf;
            if (lse_mode == 0) {
                kf.load(kcb + (int64_t)key * D, g);
            } else {
                RowFrag<float, D> k1, k2, k3;
                kf.load(kcb + (int64_t)(4 * key) * D, g);
                k1.load(kcb + (int64_t)(4 * key + cstep) * D, g);
                k2.load(kcb + (int64_t)(4 * key + 2 * cstep) * D, g);
                k3.load(kcb + (int64_t)(4 * key + 3 * cstep) * D, g);
#pragma unroll
                for (int e = 0; e < D / 16; ++e) kf.x[e] = ((kf.x[e] + k1.x[e]) + (k2.x[e] + k3.x[e])) * 0.25f;
            }
            s[u] = row_product<D>(kf, qf);
        }
        float mx = m_run;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (k0 + 16 * u + 4 * g + r >= v1) s[u][r] = -INFINITY;
                mx = fmaxf(mx, s[u][r]);
            }
        const float ref = mx == -INFINITY ? 0.f : mx;
        float ls = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) ls += exp2_fast((s[u][r] - ref) * c);
        l_run = l_run * exp2_fast((m_run - ref) * c) + ls;
        m_run = mx;
    }
    {   // four lane groups, then the wavefronts
        const float mg = groups_max(m_run);
        const float lg = groups_sum(l_run * exp2_fast((m_run - (mg == -INFINITY ? 0.f : mg)) * c));
        if (g == 0) { red_m[w][m] = mg; red_l[w][m] = lg; }
    }
    __syncthreads();
    float lse2;                                            // log2 of sum_i 2^(c z) of this lane's column
    {
        float mm = red_m[0][m];
#pragma unroll
        for (int x = 1; x < GS_WAVES; ++x) mm = fmaxf(mm, red_m[x][m]);
        const float ref = mm == -INFINITY ? 0.f : mm;
        float ll = 0.f;
#pragma unroll
        for (int x = 0; x < GS_WAVES; ++x) ll += red_l[x][m] * exp2_fast((red_m[x][m] - ref) * c);
        lse2 = ref * c + __log2f(ll);
    }

    // ---- pass 2: group scores of the keys [k0, k1), k1 - k0 <= GS_CHUNK, into sh (called by every thread; the caller
    // synchronises before and after).  A row that sees no coarse key has all-zero scores.
    auto chunk_scores = [&](int k0, int k1) {
#pragma unroll 1
        for (int u = 0; u < 4; ++u) {
            const int kb0 = k0 + 64 * w + 16 * u;
            if (kb0 >= k1) break;
            RowFrag<float, D> kf;
            kf.load(kcb + (int64_t)min(kb0 + m, v_max - 1) * D, g);
            const f32x4 s = row_product<D>(kf, qf);
#pragma unroll
            for (int r = 0; r < 4; ++r) ps[w][4 * g + r][m] = v1 > 0 ? exp2_fast(__builtin_fmaf(s[r], c, -lse2)) : 0.f;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // lane (key m, token slot g): the heads of tokens g, g + 4, ... added up
            for (int x = g; x < t.ntok; x += 4) {
                float sum = 0.f;
                for (int e = 0; e < G; ++e) sum += ps[w][m][x * G + e];
                sh[x][64 * w + 16 * u + m] = sum;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    };
    float *out = s_shared + head_row(map, h, t.row0) * row_stride;       // rows of the tile's tokens are consecutive
    if (!pool.on) {
        for (int k0 = 0; k0 < v_max; k0 += GS_CHUNK) {
            const int k1 = min(k0 + GS_CHUNK, v_max);
            chunk_scores(k0, k1);
            __syncthreads();
            for (int x = 0; x < t.ntok; ++x) {
                const int v = visible_cmp(t.t0 + x, lc, sc);
                if (k0 + tid < min(k1, v)) out[x * row_stride + k0 + tid] = sh[x][tid];
            }
            __syncthreads();
        }
        return;
    }
    // one item per (token, selection block up to the token's own): the max over its pooling window (Eq. 6), clipped to
    // the visible keys.  nb blocks' windows fit one chunk; a window longer than a chunk is taken in pieces (nb = 1).
    const int nb = pool.len <= GS_CHUNK ? min((GS_CHUNK - pool.len) / pool.stride + 1, GS_CHUNK) : 1;
    const int range = pool.stride * (nb - 1) + pool.len;
    const int bt_max = (t.t0 + t.ntok - 1) / kBlock;
    for (int j0 = 0; j0 <= bt_max; j0 += nb) {
        const int64_t first = (int64_t)pool.stride * j0 - pool.pad;
        if (first >= v_max) break;                         // no window from here on holds a visible key
        const int span = (int)min((int64_t)range, v_max - first);
        float keep = 0.f;                                  // nb == 1: running maximum over the pieces
        for (int off = 0; off < span; off += GS_CHUNK) {
            const int k0 = (int)max(first + off, (int64_t)0), k1 = (int)(first + min(off + GS_CHUNK, span));
            if (k0 < k1) chunk_scores(k0, k1);
            __syncthreads();
            for (int it = tid; it < t.ntok * nb; it += NT) {
                const int x = it / nb, j = j0 + it - x * nb;
                const int v = visible_cmp(t.t0 + x, lc, sc);
                const int lo = (int)(first + (int64_t)pool.stride * (j - j0));
                const int hi = (int)min((int64_t)lo + pool.len, (int64_t)min(k1, v));
                float mx = nb == 1 ? keep : 0.f;
                for (int i = max(lo, k0); i < hi; ++i) mx = fmaxf(mx, sh[x][i - k0]);
                keep = mx;
                const bool last = off + GS_CHUNK >= span;
                if (last && j <= (t.t0 + x) / kBlock && max(lo, 0) < v) out[x * row_stride + j] = mx;
            }
            __syncthreads();
        }
    }
}

template <typename T, int D>
static int launch_generic(const Launch &L, const void *q, const float *kc, float *s_shared, int64_t row_stride,
                          const PoolArgs &pool) {
    if (L.map.total_rows == 0) return INFLLMV2_OK;
    // at most this many tiles (every sequence may end with a partial one)
    const int tokens = gen::tile_tokens(L.map, L.p->num_q_heads / L.p->num_kv_heads);
    dim3 grid(L.map.ctx ? L.map.total_rows : L.map.total_rows / tokens + L.map.batch, L.p->num_kv_heads);
    hipLaunchKernelGGL((block_scores_generic<T, D>), grid, dim3(GS_WAVES * 64), 0, L.stream, (const T *)q, kc, L.map,
                       L.p->num_q_heads, L.p->cmp_len, L.p->cmp_stride, L.p->softmax_scale, L.p->dense_threshold,
                       L.p->lse_mode, s_shared, row_stride, pool);
    return hip_status(hipGetLastError());
}


// ------------------------------------------------------------------------------------------
// MFMA kernel for bf16 Q, G = 16, d = 128 (the paper's head shape).
//
// A workgroup owns T consecutive tokens of one KV head; every wave keeps the Q rows of its TPW tokens in
// registers as MFMA A operands (M = the 16 heads of the group).  Compressed keys stream through LDS in
// tiles of 64 and each B fragment read from LDS is reused by all TPW tokens of the wave.  A lane then owns
// one key column and four heads, so
//   pass 1 keeps a private running (reference, sum 2^(y - reference)) per head with no cross-lane traffic
//          in the loop; the reference is only moved when a logit exceeds it by 2^16, and
//   pass 2 sums its four heads in registers and finishes the head-group sum with a 3-step butterfly
//          across the four lane groups, after which the 64 lanes hold 64 consecutive keys' group sums.
//
// Precision.  The ranking of blocks is sensitive to ~1e-3 relative changes of the scores, so the operands
// are not rounded to bf16.  Q (bf16) converts to fp16 exactly and K^{C1} (float32 means of 32 keys) is
// rounded to fp16, whose 11-bit significand keeps the logit error near 1e-4 -- one fp16 MFMA instead of a
// bf16 high/low pair.  fp16's narrow exponent range is handled by exact power-of-two scalings: a token whose Q
// magnitudes would leave the range gets its own exponent, and a key tile that holds a magnitude above 2^15
// (never the case for real activations) is re-staged with its own shift; both are undone by a multiply on the
// accumulator, on a slower path.  Both passes see the same logits.
//
// What a workgroup does before its first product and between its passes is paid once per 32 tokens, which at 10000 tokens is
// a third of the kernel: counts by shift instead of division, the Q rows and the first key tile requested together, lane
// maxima by lane moves, no reference in the merge of a pass that had none.  Kernel at 5000 tokens 35.2 -> 33.1 us, LSE
// Approximation at 20011 tokens 199 -> 186, 65536 tokens 1.2 % less.  (One resident workgroup per CU that goes through the
// tiles gains nothing more: 102.3 against 102.8 us for the call at 10000 tokens, 2084 against 2078 at 65536.)
//
// Vector-instruction budget.  MFMA and vector instructions share one issue port, and a (token, key tile) pair
// has 16 MFMAs against 16 exponentials plus their sums, so every other vector instruction per logit shows up
// in the run time.  Two are avoided: softmax_scale * log2(e) is multiplied into K^{C1} when a tile is converted
// to fp16 (the conversion rounds anyway, so this adds no error), and the accumulator is seeded with minus the
// row's reference (pass 1) or minus its log-sum-exp (pass 2), so the MFMA result is the exponent itself.  The
// rare tiles or tokens that carry a power-of-two rescaling take a slower path with an explicit multiply.
// ------------------------------------------------------------------------------------------
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

namespace {

constexpr int SD = 128, SG = 16;
constexpr int SKS = SD + 8;                    // LDS row stride (fp16) of a compressed-key tile
constexpr int S_TILE = kBlock * SKS;           // one 64-key tile
constexpr float S_LOG2E = 1.4426950408889634f;
constexpr float S_SLACK = 16.0f;               // pass 1 moves its reference when a logit exceeds it by 2^16
constexpr float S_FP16_SAFE = 32768.0f;

// fp16 copy of the compressed keys in tiles of 64 rows (written by kc_half_kernel): per KV head `tiles` tiles of
// 64 x 128 halves, sequences back to back (sequence s starts at tile sum_{s' < s} ceil(nc(s') / 64)), rows past a
// sequence's last key are zero; tile values are K * cm * 2^-shift with the tile's shift stored beside.
struct HalfTiles {
    const _Float16 *data;
    const int32_t *shift;
    int32_t tiles;            // per KV head
};

struct ScoreArgs {
    const uint16_t *q;
    const float *kc;
    HalfTiles fine, coarse;   // K^{C1}; K^{C2} (only with the LSE Approximation)
    float *out;
    RowMap map;
    int hq, lc, sc, dense_below, lse_mode;
    float scale;
    int64_t row_stride;
    int sc_shift;             // log2(sc) where sc is a power of two, else -1
};

__device__ inline float s_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// data-parallel-primitive moves of a 32-bit value: lane i receives the value of another lane without touching LDS
template <int CTRL>
__device__ inline unsigned dpp_move(unsigned x) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
// max (MAX) or sum over the 16 lanes of a row (lanes with equal lane / 16), result in every lane: swaps inside quads,
// then the mirror images inside 8 and 16 lanes
template <bool MAX>
__device__ inline float row16_all(float x) {
    auto step = [](float v, float o) { return MAX ? fmaxf(v, o) : v + o; };
    x = step(x, __uint_as_float(dpp_move<0xB1>(__float_as_uint(x))));       // quad_perm [1,0,3,2]
    x = step(x, __uint_as_float(dpp_move<0x4E>(__float_as_uint(x))));       // quad_perm [2,3,0,1]
    x = step(x, __uint_as_float(dpp_move<0x141>(__float_as_uint(x))));      // row_half_mirror
    return step(x, __uint_as_float(dpp_move<0x140>(__float_as_uint(x))));   // row_mirror
}
// max over the wave, result in every lane
__device__ inline float wave64_max(float x) {
    x = row16_all<true>(x);
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
// element e of eight bf16 values
__device__ inline float bf16_at(const uint4 &v, int e) {
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
    return __uint_as_float(e & 1 ? u[e >> 1] & 0xffff0000u : u[e >> 1] << 16);
}
constexpr int DPP_QUAD_SWAP1 = 0xB1;   // quad_perm [1,0,3,2]
constexpr int DPP_QUAD_SWAP2 = 0x4E;   // quad_perm [2,3,0,1]
constexpr int DPP_WAVE_SHR1 = 0x138;   // lane i <- lane i - 1 (lane 0 <- 0)

// Pre-pass of the matrix-core kernel: one workgroup per 64-row key tile.  Converts K^{C1} (or, for tiles
// >= fine.tiles, the coarse keys of Eq. 7: row i = mean of K^{C1} rows 4i + m l_C1/s_C1, m = 0..3) to fp16,
// multiplied by cm = the mantissa of softmax_scale * log2(e), and by 2^-shift where shift is the smallest power of
// two that brings the tile's largest magnitude below 2^15 (0 for any real activations).
__global__ void __launch_bounds__(256)
kc_half_kernel(const float *__restrict__ kc, RowMap map, int lc, int sc, int dense_below, float cm,
               _Float16 *__restrict__ fine, int32_t *__restrict__ sh_fine, int tiles_fine,
               _Float16 *__restrict__ coarse, int32_t *__restrict__ sh_coarse, int tiles_coarse) {
    __shared__ int s_seq, s_local;
    __shared__ float s_red[4];
    const int tid = threadIdx.x, h = blockIdx.y;
    const bool is_coarse = (int)blockIdx.x >= tiles_fine;
    const int tile = is_coarse ? blockIdx.x - tiles_fine : blockIdx.x;
    const int wl = is_coarse ? 4 * lc : lc, ws = is_coarse ? 4 * sc : sc;
    if (tid == 0) {
        int rem = tile, s = 0;
        for (; s < map.batch; ++s) {
            const int nt = (num_cmp(map.cu[s + 1] - map.cu[s], wl, ws) + kBlock - 1) / kBlock;
            if (rem < nt) break;
            rem -= nt;
        }
        s_seq = s;
        s_local = rem;
    }
    __syncthreads();
    const int seq = s_seq;
    if (seq >= map.batch) return;
    const int len = map.cu[seq + 1] - map.cu[seq];
    if (len < dense_below) return;                    // dense sequences are never scored
    const int rows = num_cmp(len, wl, ws), cstep = lc / sc;
    const float *kcb = kc + ((int64_t)h * map.kc_total_c + map.cu_c[seq]) * SD;
    float4 x[8];
    float amax = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int c = tid + r * 256;
        const int row = s_local * kBlock + (c >> 5), col = (c & 31) * 4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row < rows) {
            if (!is_coarse) {
                v = *reinterpret_cast<const float4 *>(kcb + (int64_t)row * SD + col);
            } else {
                const float *b = kcb + (int64_t)4 * row * SD + col;
                const float4 k0 = *reinterpret_cast<const float4 *>(b);
                const float4 k1 = *reinterpret_cast<const float4 *>(b + (int64_t)cstep * SD);
                const float4 k2 = *reinterpret_cast<const float4 *>(b + (int64_t)2 * cstep * SD);
                const float4 k3 = *reinterpret_cast<const float4 *>(b + (int64_t)3 * cstep * SD);
                v.x = ((k0.x + k1.x) + (k2.x + k3.x)) * 0.25f;
                v.y = ((k0.y + k1.y) + (k2.y + k3.y)) * 0.25f;
                v.z = ((k0.z + k1.z) + (k2.z + k3.z)) * 0.25f;
                v.w = ((k0.w + k1.w) + (k2.w + k3.w)) * 0.25f;
            }
        }
        x[r] = v;
        amax = fmaxf(fmaxf(amax, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w)));
    }
    amax = wave_max(amax);
    if ((tid & 63) == 0) s_red[tid >> 6] = amax;
    __syncthreads();
    amax = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
    if (!(amax < 3.0e38f)) amax = 3.0e38f;            // Inf / NaN inputs: keep going, results are Inf / NaN anyway
    int ek = 0;
    if (amax > 0.f) (void)frexpf(amax, &ek);          // amax < 2^ek and cm < 1
    const int shift = max(0, ek - 15);
    const float f = __builtin_ldexpf(cm, -shift);
    _Float16 *dst = (is_coarse ? coarse + ((int64_t)h * tiles_coarse + tile) * (kBlock * SD)
                               : fine + ((int64_t)h * tiles_fine + tile) * (kBlock * SD));
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int c = tid + r * 256;
        typedef _Float16 half4 __attribute__((ext_vector_type(4)));
        const half4 hv = {(_Float16)(x[r].x * f), (_Float16)(x[r].y * f), (_Float16)(x[r].z * f), (_Float16)(x[r].w * f)};
        *reinterpret_cast<half4 *>(dst + (c >> 5) * SD + (c & 31) * 4) = hv;
    }
    if (tid == 0) (is_coarse ? sh_coarse : sh_fine)[(int64_t)h * (is_coarse ? tiles_coarse : tiles_fine) + tile] = shift;
}

// W = 32: lanes 0..31 get x[lane] + x[lane + 32], lanes 32..63 get y[lane - 32] + y[lane].
// W = 16 (rows of 16 lanes): rows 0 and 2 get x's rows 0+1 and 2+3, rows 1 and 3 get y's rows 0+1 and 2+3.
template <int W>
__device__ inline float swap_add(float x, float y) {
    const unsigned ux = __float_as_uint(x), uy = __float_as_uint(y);
    const auto r = W == 32 ? __builtin_amdgcn_permlane32_swap(ux, uy, false, false)
                           : __builtin_amdgcn_permlane16_swap(ux, uy, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// num_cmp with a shift where the stride is a power of two: a division is some forty scalar instructions, and a workgroup needs
// four of these counts before it can request its first byte
struct CmpCount {
    int lc, sc, shift;         // shift < 0: sc is no power of two
    __device__ inline int operator()(int n) const {
        const int d = n - lc;
        return d < 0 ? 0 : (shift >= 0 ? d >> shift : d / sc) + 1;
    }
};
// visible_cmp of consecutive tokens, from the first one on: one division for all of them
struct VisibleCount {
    int v, left, sc;           // keys the next token sees; tokens until it is one more
    __device__ inline VisibleCount(int t, const CmpCount &c) : v(c(t + 1)), sc(c.sc) {
        left = v == 0 ? c.lc - 1 - t : v * sc - (t - (c.lc - 1));      // key v completes at token v sc + lc - 1
    }
    __device__ inline int next() {
        const int now = v;
        if (--left == 0) { ++v; left = sc; }
        return now;
    }
};

// DIRECT: the key tiles are converted from K^{C1} as they are staged, with no pre-pass (see launch_block_scores).
template <int NW, int TPW, bool DIRECT>
struct ScoreKernel {
    static constexpr int T = NW * TPW;
    static constexpr int NTHR = NW * 64;
    static constexpr int NCH = 1024 / NTHR;        // 16-byte chunks of a 64 x 128 fp16 tile per thread

    // one thread's share of a tile in flight, NCH times eight elements; passed and returned by value so that it stays in
    // registers
    struct TilePre {
        uint4 c[DIRECT ? 2 * NCH : NCH];
    };
    // tile kt of a sequence's fp16 tiles, or of its nc rows of K^{C1}
    __device__ static inline TilePre load_tile(const void *keys, int kt, int nc, int tid) {
        const uint4 *src = reinterpret_cast<const uint4 *>(keys) + (int64_t)kt * (DIRECT ? 2048 : 1024);
        TilePre pf;
#pragma unroll
        for (int r = 0; r < NCH; ++r) {
            const int c = tid + r * NTHR;
            if (DIRECT) {
                const bool in = kt * kBlock + (c >> 4) < nc;
                pf.c[2 * r] = in ? src[2 * c] : make_uint4(0, 0, 0, 0);
                pf.c[2 * r + 1] = in ? src[2 * c + 1] : make_uint4(0, 0, 0, 0);
            } else {
                pf.c[r] = src[c];
            }
        }
        return pf;
    }
    // registers -> LDS (padded rows), then a workgroup barrier: every thread calls it
    __device__ static inline void stage_tile(_Float16 *tile, int tid, const TilePre pf) {
#pragma unroll
        for (int r = 0; r < NCH; ++r) {
            const int c = tid + r * NTHR;
            *reinterpret_cast<uint4 *>(tile + (c >> 4) * SKS + (c & 15) * 8) = pf.c[r];
        }
        __syncthreads();
    }
    // The same with the conversion of kc_half_kernel on the way.  Returns the tile's shift, 0 unless a magnitude reaches 2^15:
    // each wavefront says whether it holds one (flags), and only then the tile's largest is looked for and the tile staged again.
    __device__ static inline int stage_direct(_Float16 *tile, int tid, const TilePre pf, float cm, int *flags, float *tops) {
        const int lane = tid & 63, w = tid >> 6;
        auto element = [&](int i) -> float {
            const uint32_t u[4] = {pf.c[i >> 2].x, pf.c[i >> 2].y, pf.c[i >> 2].z, pf.c[i >> 2].w};
            return __uint_as_float(u[i & 3]);
        };
        auto put = [&](float f) {
#pragma unroll
            for (int r = 0; r < NCH; ++r) {
                const int c = tid + r * NTHR;
                half8 hv;
#pragma unroll
                for (int e = 0; e < 8; ++e) hv[e] = (_Float16)(element(8 * r + e) * f);
                *reinterpret_cast<half8 *>(tile + (c >> 4) * SKS + (c & 15) * 8) = hv;
            }
        };
        put(cm);
        float top = 0.f;
#pragma unroll
        for (int i = 0; i < 8 * NCH; ++i) top = fmaxf(top, fabsf(element(i)));
        const bool large = __any(!(top < S_FP16_SAFE));
        if (lane == 0) flags[w] = large;
        __syncthreads();
        int any = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) any |= flags[k];
        if (__builtin_amdgcn_readfirstlane(any) == 0) return 0;
        top = wave64_max(top);
        if (lane == 0) tops[w] = top;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NW; ++k) top = fmaxf(top, tops[k]);
        if (!(top < 3.0e38f)) top = 3.0e38f;              // as in kc_half_kernel
        int ek = 0;
        (void)frexpf(top, &ek);
        const int shift = __builtin_amdgcn_readfirstlane(max(0, ek - 15));
        put(__builtin_ldexpf(cm, -shift));
        __syncthreads();
        return shift;
    }

    template <bool SEEDED>
    __device__ static inline void tile_mma(const half8 (&qf)[TPW][4], const _Float16 *tile, int lane,
                                           f32x4 (&acc)[TPW][4], const f32x4 (&seed)[TPW]) {
        const int n16 = lane & 15, g = lane >> 4;
        const _Float16 *bp = tile + n16 * SKS + g * 8;
        half8 b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)            // u -> (nt = u / 4, ks = u % 4)
            b[u] = *reinterpret_cast<const half8 *>(bp + (u >> 2) * 16 * SKS + (u & 3) * 32);
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int nt = u >> 2, ks = u & 3;
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const f32x4 c0 = SEEDED ? seed[i] : f32x4{0.f, 0.f, 0.f, 0.f};
                acc[i][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qf[i][ks], b[u & 3], ks == 0 ? c0 : acc[i][nt], 0, 0, 0);
            }
            if (u + 4 < 16) b[u & 3] = *reinterpret_cast<const half8 *>(bp + ((u + 4) >> 2) * 16 * SKS + ((u + 4) & 3) * 32);
        }
    }

    // POOL < 0: one output per compressed key.  POOL = 0 / 1: one output per selection block, the max over the
    // pooling window [4j - POOL, 4j - POOL + 5) of Eq. 6 (see vec2 below).
    template <int POOL>
    __device__ static void run(const ScoreArgs &a, int num_tiles) {
        extern __shared__ __attribute__((aligned(16))) _Float16 smem[];     // two tiles (double buffer)
        __shared__ int s_where[4], s_flags[2][NW];
        __shared__ float s_tops[NW];
        const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int h = blockIdx.y;
        const int tile_id = num_tiles - 1 - (int)blockIdx.x;     // longest rows first
        int seq = 0, tile_in_seq = tile_id, tb_fine = 0, tb_coarse = 0;    // tb: first key tile of the sequence
        if (a.map.batch > 1) {                                   // (one sequence needs no walk: two trips to memory less)
            if (tid == 0) {
                int s = 0;
                for (; s < a.map.batch; ++s) {
                    const int slen = a.map.cu[s + 1] - a.map.cu[s];
                    const int nt = (slen + T - 1) / T;
                    if (tile_in_seq < nt) break;
                    tile_in_seq -= nt;
                    tb_fine += (num_cmp(slen, a.lc, a.sc) + kBlock - 1) / kBlock;
                    tb_coarse += (num_cmp(slen, 4 * a.lc, 4 * a.sc) + kBlock - 1) / kBlock;
                }
                s_where[0] = s;
                s_where[1] = tile_in_seq;
                s_where[2] = tb_fine;
                s_where[3] = tb_coarse;
            }
            __syncthreads();
            seq = __builtin_amdgcn_readfirstlane(s_where[0]);
            tile_in_seq = __builtin_amdgcn_readfirstlane(s_where[1]);
            tb_fine = __builtin_amdgcn_readfirstlane(s_where[2]);
            tb_coarse = __builtin_amdgcn_readfirstlane(s_where[3]);
        }
        if (seq >= a.map.batch) return;
        const int tok0 = a.map.cu[seq], len = a.map.cu[seq + 1] - tok0;
        if (len < a.dense_below) return;
        const int t0 = tile_in_seq * T;
        if (t0 >= len) return;                                   // (grid: every tile exists; one sequence is not searched)
        const int ntok = min(T, len - t0);
        const CmpCount fine_count{a.lc, a.sc, a.sc_shift};
        const CmpCount coarse_count{4 * a.lc, 4 * a.sc, a.sc_shift < 0 ? -1 : a.sc_shift + 2};
        const int nc = fine_count(len);
        const int vis_last = min(fine_count(t0 + ntok), nc);
        if (vis_last == 0) return;
        const int nkt = (vis_last + kBlock - 1) / kBlock;
        const int row0 = tok0 + t0;
        // this sequence's key tiles and their shifts (wave-uniform addresses)
        const void *kt_fine = a.fine.data + ((int64_t)h * a.fine.tiles + tb_fine) * (kBlock * SD);
        const int32_t *sh_fine = a.fine.shift + (int64_t)h * a.fine.tiles + tb_fine;
        const void *kt_coarse = a.lse_mode ? a.coarse.data + ((int64_t)h * a.coarse.tiles + tb_coarse) * (kBlock * SD) : kt_fine;
        const int32_t *sh_coarse = a.lse_mode ? a.coarse.shift + (int64_t)h * a.coarse.tiles + tb_coarse : sh_fine;
        if (DIRECT) kt_fine = kt_coarse = a.kc + ((int64_t)h * a.map.kc_total_c + a.map.cu_c[seq]) * SD;      // (lse_mode 0)
        const int n16 = lane & 15, g = lane >> 4;

        // ---- Q rows of this wave's tokens: bf16 -> fp16, times a power of two (exact).  With
        // softmax_scale * log2(e) = cm * 2^ce (0.5 <= cm < 1), the keys carry cm (multiplied in when a tile is
        // converted to fp16) and the queries carry 2^ce, so the MFMA accumulator is the logit in the log2 domain.
        // A token whose magnitudes would leave fp16's comfortable range that way gets its own exponent instead and
        // takes the slower path that multiplies the accumulator by the difference.
        int ce;
        const float cm = frexpf(a.scale * S_LOG2E, &ce);
        ce = __builtin_amdgcn_readfirstlane(ce);
        half8 qf[TPW][4];
        int vis[TPW];
        // keys of pass 1: the fine ones, or with the LSE Approximation the coarse ones (Eq. 7)
        const int nc2 = a.lse_mode ? coarse_count(len) : 0;
        int vis1[TPW];
        int vis1_min = 1 << 30;
        float cq[TPW];                   // 2^(ce - token's exponent): multiplies the accumulator (normally 1)
        bool q_plain = true;
        int vis_min = 1 << 30;
        // every row of the wave is requested before the first is looked at, and with them the first key tile of pass 1: one
        // trip to memory (rows past the sequence's end repeat its last token and see no key)
        uint4 raw[TPW][4];
        VisibleCount fine_keys(t0 + w * TPW, fine_count), coarse_keys(t0 + w * TPW, coarse_count);
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int ti = w * TPW + i;
            vis[i] = ti < ntok ? min(fine_keys.next(), nc) : 0;
            vis_min = min(vis_min, vis[i]);
            vis1[i] = a.lse_mode == 0 ? vis[i] : (ti < ntok ? min(coarse_keys.next(), nc2) : 0);
            vis1_min = min(vis1_min, vis1[i]);
            const uint16_t *qp = a.q + ((int64_t)(row0 + min(ti, ntok - 1)) * a.hq + h * SG + n16) * SD + g * 8;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) raw[i][ks] = *reinterpret_cast<const uint4 *>(qp + ks * 32);
        }
        const int vis1_last = a.lse_mode == 0 ? vis_last : min(coarse_count(t0 + ntok), nc2);
        const int nkt1 = (vis1_last + kBlock - 1) / kBlock;
        TilePre first = {};
        if (nkt1 > 0) first = load_tile(kt_coarse, 0, nc, tid);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            float amax = 0.f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(bf16_at(raw[i][ks], e)));
            amax = wave64_max(amax);
            if (!(amax < 3.0e38f)) amax = 3.0e38f;     // Inf / NaN inputs: keep going, results are Inf / NaN anyway
            int exq = 0;
            if (amax > 0.f) (void)frexpf(amax, &exq);  // amax = f * 2^exq, 0.5 <= f < 1
            // keep the largest magnitude within [2^-8, 2^15): 18+ binades of full precision below it
            int eq = ce;
            if (exq + ce > 15 || exq + ce < -8) eq = 4 - exq;
            const float sc = __builtin_ldexpf(1.0f, eq);
            cq[i] = __builtin_ldexpf(1.0f, ce - eq);
            q_plain &= eq == ce;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) qf[i][ks][e] = (_Float16)(bf16_at(raw[i][ks], e) * sc);
        }
        f32x4 acc[TPW][4];
        f32x4 nm[TPW];                   // per lane and head row: minus the reference (log2 domain)
        float l[TPW][4];                 // ... and the sum of 2^(y - reference)
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            nm[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 4; ++r) l[i][r] = 0.f;
        }

        // Matrix-core step of either pass: acc = y - seed for tile kt (y = the logit in the log2 domain)
        int direct_shift = 0;                          // DIRECT: of the tile staged last
        auto stage = [&](int kt, const TilePre pf) {
            if constexpr (DIRECT) direct_shift = stage_direct(smem + (kt & 1) * S_TILE, tid, pf, cm, s_flags[kt & 1], s_tops);
            else stage_tile(smem + (kt & 1) * S_TILE, tid, pf);
        };
        auto mma = [&](int kt, const int32_t *shifts, const f32x4 (&seed)[TPW]) {
            const _Float16 *tile = smem + (kt & 1) * S_TILE;
            const int tshift = DIRECT ? direct_shift : shifts[kt];
            if (q_plain && tshift == 0) {
                tile_mma<true>(qf, tile, lane, acc, seed);
            } else {
                tile_mma<false>(qf, tile, lane, acc, seed);
                const float tsc = __builtin_ldexpf(1.0f, tshift);
#pragma unroll
                for (int i = 0; i < TPW; ++i)
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[i][nt][r] = __builtin_fmaf(acc[i][nt][r], cq[i] * tsc, seed[i][r]);
            }
        };
        // The two waves that share a SIMD (w and w + NW/2) run half a step apart: between two barriers the first
        // does the matrix-core step of tile kt and then its vector step, the second does the vector step of tile
        // kt - 1 (still in its accumulators) and then the matrix-core step of tile kt.  Matrix core and vector
        // unit of a SIMD are then busy at the same time although each wave alternates between them.
        const bool late = w >= NW / 2;

        // ------------------------------------------------ pass 1: log-sum-exp of every (token, head) row
        // First attempt without a running reference: sum 2^y as it is.  For ordinary activations |y| stays far
        // below fp32's exponent range, and the max tracking (a fifth of the vector work of this pass) is saved.
        // If any row's sum then overflowed, vanished or is NaN, the workgroup repeats the pass with the reference.
        auto vec1 = [&](int kt, auto tracked_c) {
            constexpr bool tracked = decltype(tracked_c)::value;
            const int kbase = kt * kBlock;
            const bool edge_tile = kbase + kBlock > vis1_min;
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                if (edge_tile) {
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt)
                        if (kbase + nt * 16 + n16 >= vis1[i]) acc[i][nt] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
                }
                // The reference moves only when an exponent exceeds S_SLACK; the first tile sets it (up or down).
                if (tracked) {
                    float mx[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) mx[r] = fmaxf(fmaxf(acc[i][0][r], acc[i][1][r]), fmaxf(acc[i][2][r], acc[i][3][r]));
                    const float mxall = fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3]));
                    if (kt == 0 || __any(mxall > S_SLACK)) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            float d = kt == 0 ? mx[r] : fmaxf(mx[r], 0.f);
                            if (!(d > -3.0e38f)) d = 0.f;              // nothing visible in this lane's columns yet
                            l[i][r] *= s_exp2(-d);
                            nm[i][r] -= d;
#pragma unroll
                            for (int nt = 0; nt < 4; ++nt) acc[i][nt][r] -= d;
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float sum = l[i][r];
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt) sum += s_exp2(acc[i][nt][r]);
                    l[i][r] = sum;
                }
            }
        };
        float lse2[TPW][4];
        auto pass1 = [&](auto tracked_c) -> bool {       // returns true if some row's sum cannot be trusted
            constexpr bool tracked = decltype(tracked_c)::value;
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                nm[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 4; ++r) l[i][r] = 0.f;
            }
            TilePre pf = first;
            if (nkt1 > 0) stage(0, tracked ? load_tile(kt_coarse, 0, nc, tid) : first);
            for (int kt = 0; kt < nkt1; ++kt) {
                if (kt + 1 < nkt1) pf = load_tile(kt_coarse, kt + 1, nc, tid);
                if (late && kt > 0) vec1(kt - 1, tracked_c);
                mma(kt, sh_coarse, nm);
                if (!late) vec1(kt, tracked_c);
                if (kt + 1 < nkt1) stage(kt + 1, pf);
                else __syncthreads();
            }
            if (late && nkt1 > 0) vec1(nkt1 - 1, tracked_c);
            // merge the 16 key lanes of each lane group; lse2 = log2 of the row's sum of 2^y
            bool bad = false;
#pragma unroll
            for (int i = 0; i < TPW; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // (lane moves inside the 16-lane row: no LDS round trips)
                    float mm = 0.f, ll = l[i][r];
                    if (tracked) {                       // (untracked references are all zero)
                        mm = -nm[i][r];
                        const float mrow = row16_all<true>(mm);
                        ll *= s_exp2(mm - mrow);
                        mm = mrow;
                    }
                    ll = row16_all<false>(ll);
                    // a row that saw no key at all (possible with the coarse keys of the LSE Approximation while
                    // fine keys are already visible) normalises everything to zero
                    lse2[i][r] = ll > 0.f ? mm + __log2f(ll) : INFINITY;
                    // untracked sums are trusted only well inside fp32's range (2^-64 .. 3e38)
                    bad |= vis1[i] > 0 && !(ll >= 5.4e-20f && ll < 3.0e38f);
                }
            return bad;
        };
        if (__syncthreads_or(pass1(std::false_type{}))) (void)pass1(std::true_type{});

        // ------------------------------------------------ pass 2: normalised scores, group sum, store
        f32x4 nlse[TPW];
#pragma unroll
        for (int i = 0; i < TPW; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) nlse[i][r] = -lse2[i][r];
        // Fused pooling (POOL >= 0).  After the butterfly lane x of the wave holds the group sum of key kbase + x,
        // so the four keys 4m .. 4m + 3 of the tile sit in one lane quad and their max takes two quad swaps.  The
        // fifth key of a window lies one lane below the quad (POOL = 1: window = key 4m - 1 and quad m, block
        // 16 kt + m) or is the first lane of the next quad (POOL = 0: window = quad m - 1 and key 4m, block
        // 16 kt + m - 1): either way lane 4m combines its own value with one shifted up by a lane, and what
        // lane 0 needs from the previous tile of the same token is carried in a scalar.
        unsigned carry[TPW];                 // bit patterns of non-negative floats
#pragma unroll
        for (int i = 0; i < TPW; ++i) carry[i] = 0u;
        // The tile's own block is the last that is written.  (Said only where windows are shifted by one: with compressed
        // windows of one stride the last key of a block is visible to the block's last token, and the next block's window
        // starts there.)
        static_assert(kBlock % T == 0, "a tile's tokens lie in one block");
        const int bt = __builtin_amdgcn_readfirstlane(t0) / kBlock;
        auto written = [&](int jb, int visible) -> bool { return max(4 * jb - POOL, 0) < visible && (POOL <= 0 || jb <= bt); };
        float *const out_w = a.out + ((int64_t)h * a.map.total_rows + row0 + w * TPW) * a.row_stride;
        auto vec2_body = [&](int kt, auto edge_c) {
            constexpr bool edge_tile = decltype(edge_c)::value;   // the tile reaches past some token's visible keys
            const int kbase = kt * kBlock;
            const int jb = kt * (kBlock / 4) + (lane >> 2) - (POOL > 0 ? 0 : 1);     // the block lane 4m completes
            const bool writer = (lane & 3) == 0 && jb >= 0;
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                float s[4];
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    s[nt] = (s_exp2(acc[i][nt][0]) + s_exp2(acc[i][nt][1])) + (s_exp2(acc[i][nt][2]) + s_exp2(acc[i][nt][3]));
                // butterfly over the four lane groups: afterwards lane (n16, g) holds n-tile g, i.e. key kbase + lane
                // (a half swap of (s0, s2) and of (s1, s3), then a row swap of the two sums: no LDS round trip)
                const float a0 = swap_add<32>(s[0], s[2]);
                const float a1 = swap_add<32>(s[1], s[3]);
                const float f = swap_add<16>(a0, a1);
                const int key = kbase + lane;
                if (POOL < 0) {
                    if (key < vis[i]) out_w[i * a.row_stride + key] = f;
                } else {
                    // scores are >= 0: an invisible key counts as 0, and the maxima are taken on the bit patterns
                    // (same order as the floats; an integer max folds the lane move into itself)
                    const unsigned fz = edge_tile && key >= vis[i] ? 0u : __float_as_uint(f);
                    unsigned qm = max(fz, dpp_move<DPP_QUAD_SWAP1>(fz));
                    qm = max(qm, dpp_move<DPP_QUAD_SWAP2>(qm));
                    const unsigned shifted_src = POOL ? fz : qm, own = POOL ? qm : fz;
                    unsigned below = dpp_move<DPP_WAVE_SHR1>(shifted_src);
                    if (lane == 0) below = carry[i];
                    carry[i] = __builtin_amdgcn_readlane(shifted_src, 63);
                    const bool has_visible_key = !edge_tile || written(jb, vis[i]);
                    if (writer && has_visible_key) out_w[i * a.row_stride + jb] = __uint_as_float(max(below, own));
                }
            }
        };
        auto vec2 = [&](int kt) {
            // only tiles that reach past the visible prefix of one of the wave's tokens need per-lane checks
            if (POOL < 0 || kt * kBlock + kBlock > vis_min) vec2_body(kt, std::true_type{});
            else vec2_body(kt, std::false_type{});
        };
        // the block whose window starts in the last tile but would end in the next one
        auto flush_pool = [&]() {
            if (POOL < 0) return;
            const int jb = nkt * (kBlock / 4) - (POOL ? 0 : 1);
#pragma unroll
            for (int i = 0; i < TPW; ++i)
                if (lane == 0 && written(jb, vis[i])) out_w[i * a.row_stride + jb] = __uint_as_float(carry[i]);
        };
        TilePre pf = load_tile(kt_fine, 0, nc, tid);
        stage(0, pf);
        for (int kt = 0; kt < nkt; ++kt) {
            if (kt + 1 < nkt) pf = load_tile(kt_fine, kt + 1, nc, tid);
            if (late && kt > 0) vec2(kt - 1);
            mma(kt, sh_fine, nlse);
            if (!late) vec2(kt);
            if (kt + 1 < nkt) stage(kt + 1, pf);
            else __syncthreads();
        }
        if (late) vec2(nkt - 1);
        flush_pool();
    }
};

template <int NW, int TPW, int POOL, bool DIRECT>
__global__ void __launch_bounds__(NW * 64) block_scores_mfma_kernel(ScoreArgs a, int num_tiles) {
    ScoreKernel<NW, TPW, DIRECT>::template run<POOL>(a, num_tiles);
}

template <int NW, int TPW, int POOL, bool DIRECT>
int launch_scores_mfma(const Launch &L, ScoreArgs a, const int32_t *cu_h) {
    constexpr int T = NW * TPW;
    int64_t tiles = 0, kt_fine = 0, kt_coarse = 0;
    for (int s = 0; s < L.map.batch; ++s) {
        const int len = cu_h[s + 1] - cu_h[s];
        tiles += (len + T - 1) / T;
        kt_fine += (num_cmp(len, a.lc, a.sc) + kBlock - 1) / kBlock;
        if (a.lse_mode) kt_coarse += (num_cmp(len, 4 * a.lc, 4 * a.sc) + kBlock - 1) / kBlock;
    }
    if (tiles == 0 || kt_fine == 0) return INFLLMV2_OK;      // no token sees a compressed key
    if (kt_fine + kt_coarse > 0x7fffffff) return INFLLMV2_ERR_UNSUPPORTED;
    // fp16 key tiles + one shift per tile, in the caller's workspace
    const int hkv = L.p->num_kv_heads;
    const size_t tile_bytes = (size_t)kBlock * SD * sizeof(_Float16);
    const size_t data_bytes = (size_t)hkv * (kt_fine + kt_coarse) * tile_bytes;
    const size_t ws_bytes = data_bytes + (size_t)hkv * (kt_fine + kt_coarse) * sizeof(int32_t);
    void *ws = L.ws;
    if (ws == nullptr || L.ws_bytes < ws_bytes) return INFLLMV2_ERR_WORKSPACE_TOO_SMALL;
    _Float16 *fine = (_Float16 *)ws, *coarse = fine + (size_t)hkv * kt_fine * kBlock * SD;
    int32_t *sh_fine = (int32_t *)((char *)ws + data_bytes), *sh_coarse = sh_fine + (size_t)hkv * kt_fine;
    int ce;
    const float cm = frexpf(a.scale * S_LOG2E, &ce);
    if (!DIRECT)
        hipLaunchKernelGGL(kc_half_kernel, dim3((unsigned)(kt_fine + kt_coarse), hkv), dim3(256), 0, L.stream, a.kc, L.map,
                       a.lc, a.sc, a.dense_below, cm, fine, sh_fine, (int)kt_fine, coarse, sh_coarse, (int)kt_coarse);
    a.fine = HalfTiles{fine, sh_fine, (int32_t)kt_fine};
    a.coarse = HalfTiles{coarse, sh_coarse, (int32_t)kt_coarse};
    const size_t lds = (size_t)2 * S_TILE * sizeof(_Float16);
    dim3 grid((unsigned)tiles, hkv);
    hipLaunchKernelGGL((block_scores_mfma_kernel<NW, TPW, POOL, DIRECT>), grid, dim3(NW * 64), lds, L.stream, a, (int)tiles);
    return hip_status(hipGetLastError());
}

template <int NW, int TPW, bool DIRECT = false>
int launch_scores_pool(const Launch &L, const ScoreArgs &a, const int32_t *cu_h, int pool) {
    if (pool < 0) return launch_scores_mfma<NW, TPW, -1, DIRECT>(L, a, cu_h);
    return pool == 0 ? launch_scores_mfma<NW, TPW, 0, DIRECT>(L, a, cu_h) : launch_scores_mfma<NW, TPW, 1, DIRECT>(L, a, cu_h);
}

bool scores_mfma_params(const infllmv2_params *p, bool pooled) {
    // the tiled kernel pools on chip only for the paper's window (l = 5, s = 4), unshifted or shifted by one, with
    // four compressed keys per selection block (block j's window then starts at key 4j of its tile row)
    const bool pool_ok = !pooled || (p->pool_len == 5 && p->pool_stride == 4 && (p->pool_pad == 0 || p->pool_pad == 1) &&
                                     p->cmp_stride * p->pool_stride == kBlock);
    return p->dtype == INFLLMV2_BF16 && p->head_dim == SD && p->num_q_heads / p->num_kv_heads == SG && pool_ok;
}

}  // namespace

// fp16 copies of the fine (and, with the LSE Approximation, coarse) key tiles plus one shift per tile
size_t scores_ws_bytes(const infllmv2_params *p, const BatchTotals &t, bool pooled) {
    if (!scores_mfma_params(p, pooled)) return 0;
    const int64_t tiles = t.kt_fine + (p->lse_mode ? t.kt_coarse : 0);
    return align256((size_t)p->num_kv_heads * tiles * ((size_t)kBlock * SD * sizeof(_Float16) + sizeof(int32_t)));
}

int launch_block_scores(const Launch &L, const void *q, const float *kc, float *s_shared, int64_t row_stride,
                        const int32_t *cu_h, bool pooled) {
    const bool bf = L.p->dtype == INFLLMV2_BF16;
    const PoolArgs pool{pooled ? 1 : 0, L.p->pool_len, L.p->pool_stride, L.p->pool_pad};
    if (cu_h != nullptr && L.map.ctx == nullptr && scores_mfma_params(L.p, pooled) &&
        (((uintptr_t)q | (uintptr_t)kc) & 15) == 0) {
        ScoreArgs a{(const uint16_t *)q, kc, HalfTiles{}, HalfTiles{}, s_shared, L.map, L.p->num_q_heads, L.p->cmp_len, L.p->cmp_stride,
                    L.p->dense_threshold, L.p->lse_mode, L.p->softmax_scale, row_stride,
                    (L.p->cmp_stride & (L.p->cmp_stride - 1)) == 0 ? __builtin_ctz(L.p->cmp_stride) : -1};
        // Four tokens per wavefront, so that a key fragment read from LDS feeds four products; fewer for short prompts, whose
        // time is what one workgroup takes from its first load to its last store.  Kernel with one / two / four on 2 KV
        // heads: 777 tokens 7.2 / 9.0 / 13.1 us, 1500 tokens 9.9 / 11.2 / 16.6, 2000 tokens 12.2 / 11.8 / 17.2, 3000 tokens
        // 19.9 / 19.8 / 21.3, 4000 tokens 28.2 / 24.8 / 26.0, 4500 tokens 31.8 / 34.1 / 31.5.  With one and two (and the exact
        // normalisation) a workgroup also converts the few key tiles it needs: the kernel then takes as long (777 tokens 7.8 ->
        // 8.0 us, 2000 tokens 12.2 -> 13.4, 4000 tokens 25 -> 29), and a pre-pass of 3.9 to 4.9 us and its launch are gone.
        int64_t tiles8 = 0, tiles16 = 0, tiles16_long = 0;
        for (int s = 0; s < L.map.batch; ++s) {
            const int len = cu_h[s + 1] - cu_h[s];
            tiles8 += (len + 7) / 8;
            tiles16 += (len + 15) / 16;
            if (len > 1750) tiles16_long += (len + 15) / 16;
        }
        if (tiles8 * L.p->num_kv_heads <= 384) {
            if (a.lse_mode == 0) return launch_scores_pool<8, 1, true>(L, a, cu_h, pooled ? pool.pad : -1);
            return launch_scores_pool<8, 1>(L, a, cu_h, pooled ? pool.pad : -1);
        }
        // Just below the line sequences of 1751 to 2048 tokens (two key tiles, nearly full) are better off with four tokens
        // already, if most tiles are theirs.  Calls with two / four: 4 x 2000 on 1 KV head 23.5 / 21.2 us, 2 x 1900 on 2
        // 23.1 / 21.1, 1850 tokens on 4 22.4 / 20.4, 2040 on 4 22.9 / 20.9, with the LSE Approximation 22.9 / 20.0; but 1700
        // tokens on 4 20.3 / 24.3, 1900 beside twenty of 300 on 1 22.9 / 29.5, 16 x 400 on 1 18.8 / 20.2.
        const bool two_tiles = L.max_len <= 2048 && tiles16 * L.p->num_kv_heads > 440 && 2 * tiles16_long > tiles16;
        if (tiles16 * L.p->num_kv_heads <= 512 && !two_tiles) {
            if (a.lse_mode == 0) return launch_scores_pool<8, 2, true>(L, a, cu_h, pooled ? pool.pad : -1);
            // Prompts of up to 2048 tokens have so few coarse key tiles that a workgroup's start is most of what it does: with
            // more workgroups than CUs, two / four tokens per wavefront (calls): 4 x 700 tokens on 2 KV heads 19.8 / 17.4 us,
            // 4 x 1000 20.7 / 17.6, 2 x 1000 on 4 21.0 / 17.7, 4 x 2000 on 1 23.3 / 20.3, one of 600, 1000 tokens on 8
            // 20.4 / 17.0, 20.4 / 17.6, 400 on 16 20.3 / 17.1, 1400 on 4 20.3 / 18.6; but 1100, 1200 tokens on 4 (276 and 300
            // workgroups) 18.1 / 19.0, 19.4 / 20.4, 2 x 3600 on 1 23.8 / 25.7, one of 3800 24.7 / 26.4.
            if (L.max_len > 2048 || tiles16 * L.p->num_kv_heads <= 300)
                return launch_scores_pool<8, 2>(L, a, cu_h, pooled ? pool.pad : -1);
        }
        return launch_scores_pool<8, 4>(L, a, cu_h, pooled ? pool.pad : -1);
    }
    if (L.p->head_dim == 128)
        return bf ? launch_generic<bf16_t, 128>(L, q, kc, s_shared, row_stride, pool)
                  : launch_generic<float, 128>(L, q, kc, s_shared, row_stride, pool);
    return bf ? launch_generic<bf16_t, 64>(L, q, kc, s_shared, row_stride, pool)
              : launch_generic<float, 64>(L, q, kc, s_shared, row_stride, pool);
}

}  // namespace ifv2
