// Stage 4 for short prompts (bf16, G = 16, d_h = 128; sparse, dense and the per-sequence switch as in attn_mfma.hip): calls
// that leave most of the chip idle, or busy for a few intervals only, so that what they cost is the chain of one workgroup.
//
// What shortens that chain against the tile kernel:
//   * tiles of four tokens, each shared by one or two wavefronts (SH) that take the blocks of an interval one each, with a softmax
//     state of their own (merged through LDS at the end);
//   * V is read from its rows by transposing LDS reads, so that there is no V^T pre-pass (a launch of 4.7 us).  They move half
//     as many bytes per clock as reads of a V^T tile, and with SH = 2 they are what an interval's units take longest for (1975
//     clocks, of which the reads need 1850; with the eight copies of a wavefront 2600), but the pre-pass would cost more;
//   * where a token's list can hold every block of the tile's walk, all blocks are walked: their copies start before the lists
//     are read, which then only say who takes part; lists, queries and first blocks are requested together;
//   * heads side by side in the launch, so that the longest tiles of every head start first (500 tokens on 8 KV heads 31.3 -> 25.6 us).
// Measured, call with 64 blocks, tile kernel and pre-pass -> this: 2 KV heads, 60 tokens 10.5 -> 7.5 us, 300 14.3 -> 10.4, 777 23.7 ->
// 19.4, 1000 27.0 -> 24.0; 1 KV head, 1400 tokens 32.0 -> 23.3; 8 KV heads, 700 tokens 51.6 -> 37.5; 500 x 60 tokens 595 -> 269.
// Measured and not built: rings of three or four intervals (no faster: the copies are not what an interval waits for; 4 tokens in 64 KB
// leave room for a second workgroup on the CU), half blocks as a wavefront's share (777 tokens 20.7), tiles of two tokens (29.5; faster
// below 300 tokens by 1 us), two tokens per wavefront with shared operands (half the LDS reads, but a lone wavefront per SIMD issues
// them no faster: 23.1), eight tokens per tile (24).
#include "attn_unit.h"
#include "launch_rules.h"

namespace ifv2 {

namespace {

using namespace attn_unit;

struct ShortArgs {
    const uint16_t *q, *k, *v;
    const int32_t *idx;
    uint16_t *out;
    float *lse;
    RowMap map;
    int hq, topk_total, dense_below;
    float scale;
    int nb_cap;        // words reserved in LDS for the per-block token masks
};

constexpr int T = 4;                                  // tokens of a workgroup
constexpr int kPart = 64 * 4 * 8 + 2 * 64;            // floats of a partial result: O, reference, sum
template <int SH>
constexpr size_t stage_bytes() {                      // two intervals' blocks, and the partial results afterwards
    const size_t stages = (size_t)2 * SH * STAGE_ELEMS * sizeof(uint16_t), parts = (size_t)(SH - 1) * T * kPart * sizeof(float);
    return stages > parts ? stages : parts;
}

// SH wavefronts for each token; an interval is SH blocks, one for each of a token's wavefronts
template <int SH>
__global__ void __launch_bounds__(T * SH * 64) attn_short_kernel(ShortArgs a, int num_tiles) {
    constexpr int NW = T * SH, NTHR = NW * 64;
    static_assert(16 % NW == 0, "sixteen one-KB pieces per tile are dealt round-robin to the waves");
    constexpr uint32_t kTileBytes = TILE_ELEMS * 2, kStageBytes = STAGE_ELEMS * 2;
    extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
    uint32_t *masks = reinterpret_cast<uint32_t *>(smem + stage_bytes<SH>() / sizeof(uint16_t));
    int2 *rec = reinterpret_cast<int2 *>(masks + a.nb_cap);          // union list: (block, token mask) per entry
    __shared__ int s_tile[3], s_ne;

    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t hkv = (uint32_t)a.map.num_kv_heads, nth = blockIdx.x / hkv;
    const int h = (int)(blockIdx.x - nth * hkv);                     // (heads side by side: every one's longest tiles start first)
    int tile;
    const int seq = __builtin_amdgcn_readfirstlane(find_seq_tile(a.map.cu, a.map.batch, T, num_tiles - 1 - (int)nth, tile, s_tile));
    if (seq >= a.map.batch) return;
    const int tok0 = a.map.cu[seq], len = a.map.cu[seq + 1] - tok0;
    const int t0 = __builtin_amdgcn_readfirstlane(tile) * T;         // first token of the tile (position in the sequence)
    const int ntok = min(T, len - t0);
    const int bt = t0 / kBlock, nblk = bt + 1;                       // T divides 64: the tile lies in one block
    const bool dense = a.idx == nullptr || len < a.dense_below;
    const bool every = dense || nblk <= a.topk_total;                // walk all blocks (see above)
    const int row0 = tok0 + t0;
    const int64_t head = (int64_t)tok0 * a.map.kv_tok_stride + (int64_t)h * a.map.kv_head_stride;
    const char *kb = reinterpret_cast<const char *>(a.k + head), *vb = reinterpret_cast<const char *>(a.v + head);
    const uint32_t full = (1u << ntok) - 1u;

    // ---- everything the first interval needs is requested at once: the block lists, the queries, the first blocks
    const int tk = a.topk_total, entries = dense ? 0 : ntok * tk;
    const int32_t *lists = a.idx + ((int64_t)h * a.map.total_rows + row0) * tk;      // (rows of consecutive tokens)
    int mine = -1;
    if (tid < entries) mine = lists[tid];
    // Waves w, w + 4, .. share a SIMD: a token's wavefronts do, so every SIMD has the same share of an interval
    const int m16 = lane & 15, g = lane >> 4;
    const int ti = w % T, share = w / T;
    const int64_t qrow = (int64_t)(row0 + ti) * a.hq + h * G + m16;
    uint4 raw[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
        raw[s] = ti < ntok ? *reinterpret_cast<const uint4 *>(a.q + qrow * D + g * 8 + s * 32) : make_uint4(0, 0, 0, 0);

    // ---- copies: a block is 32 one-KB pieces of four rows, 16 of K and 16 of V, dealt round-robin
    const uint32_t blk_bytes = (uint32_t)a.map.kv_tok_stride * (uint32_t)(kBlock * sizeof(uint16_t));   // < 2^31
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    auto lane_offset = [&](int q, int l, int last_row) -> uint32_t {
        int row, chunk;
        bwd_piece_src(q, l, row, chunk);
        return (uint32_t)(min(row, last_row) * (int)a.map.kv_tok_stride + chunk * 8) * 2u;
    };
    uint32_t off[16 / NW];                                           // of pieces w, w + NW, .. of a whole block
#pragma unroll
    for (int u = 0; u < 16 / NW; ++u) off[u] = lane_offset(w + u * NW, lane, kBlock - 1);
    auto copy_block = [&](int j, uint32_t dst) {
        const char *kj = kb + (uint64_t)j * blk_bytes, *vj = vb + (uint64_t)j * blk_bytes;
        const int last_row = len - j * kBlock - 1;                   // (rows past the end repeat the last one: hidden)
        int l = lane;
        asm volatile("" : "+v"(l));                                  // (not kept in registers over the loop)
#pragma unroll
        for (int u = 0; u < 16 / NW; ++u) {
            const uint32_t o = last_row < kBlock - 1 ? lane_offset(w + u * NW, l, last_row) : off[u];
            async_copy16(kj, o, dst + (uint32_t)(w + u * NW) * 1024u);
            async_copy16(vj, o, dst + kTileBytes + (uint32_t)(w + u * NW) * 1024u);
        }
    };
    int ne = every ? nblk : 0;                                       // blocks in the walk
    auto issue = [&](int i) {                                        // the blocks of interval i into its buffer
#pragma unroll
        for (int x = 0; x < SH; ++x) {
            const int e = SH * i + x;
            if (e >= ne) break;
            const int j = every ? e : __builtin_amdgcn_readfirstlane(rec[e].x);
            copy_block(j, lds0 + (uint32_t)((i & 1) * SH + x) * kStageBytes);
        }
    };
    if (every) issue(0);

    // ---- who selected what: masks[j] has bit ti set if token ti selected block j
    if (!dense) {
        for (int j = tid; j < nblk; j += NTHR) masks[j] = 0u;
        __syncthreads();
        for (int e = tid; e < entries; e += NTHR) {
            const int j = e == tid ? mine : lists[e];
            if (j >= 0 && j <= bt) atomicOr(&masks[j], 1u << (e / tk));
        }
        __syncthreads();
        if (!every) {
            if (w == 0) {
                int base = 0;
                for (int c = 0; c < nblk; c += 64) {
                    const int j = c + lane;
                    const uint32_t mk = j < nblk ? masks[j] : 0u;
                    const uint64_t b = __ballot(mk != 0u);
                    if (mk != 0u) rec[base + __popcll(b & ((1ull << lane) - 1ull))] = make_int2(j, (int)mk);
                    base += __popcll(b);
                }
                if (lane == 0) s_ne = base;
            }
            __syncthreads();
            ne = __builtin_amdgcn_readfirstlane(s_ne);
            issue(0);
        }
    }

    Tok st;
    {
        float cm;
        int ce;
        split_scale(a.scale * LOG2E, cm, ce);
#pragma unroll
        for (int s = 0; s < 4; ++s) st.qf[s] = scale_q(raw[s], ce);
        tok_init(st, __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, cm))));
    }
    const uint32_t rx = bwd_row_bytes(lane), tx = bwd_trans_bytes(lane) + kTileBytes;
    const int ni = (ne + SH - 1) / SH;
    bool took = false;                                               // this wave has had a block
    for (int i = 0; i < ni; ++i) {
        __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);                     // this wave's copies of interval i have landed
        __syncthreads();                                             // everybody's have, and interval i - 1 has been consumed
        // (copies go out after the wave's own S^T products: a CU takes 64 KB of them in some 700 clocks, and a wave that issued
        // its share first would start its unit that much later)
        bool due = i + 1 < ni;
        auto issue_now = [&]() {
            if (due) issue(i + 1);
            due = false;
        };
        const int e = SH * i + share;
        int j = e, mk = e < ne ? (int)full : 0;
        if (!dense && e < ne) {
            const int2 r = every ? make_int2(e, (int)masks[e]) : rec[e];
            j = __builtin_amdgcn_readfirstlane(r.x);
            mk = __builtin_amdgcn_readfirstlane(r.y);
        }
        if (((mk >> ti) & 1) == 0) {
            issue_now();
            continue;
        }
        const uint32_t at = lds0 + (uint32_t)((i & 1) * SH + share) * kStageBytes;
        took = true;
        uint32_t kx = rx, vx = tx;
        asm volatile("" : "+v"(kx), "+v"(vx));        // (operand addresses are formed here, not kept over the loop)
        if (j == bt) unit<true, true>(st, at, kx, vx, lane, t0 + ti - j * kBlock, issue_now);
        else unit<false, true>(st, at, kx, vx, lane, 0, issue_now);
    }
    __syncthreads();

    // ---- merge the shares of a token (the stages are free now), normalise and store
    // (a share whose blocks had no logit but minus infinity counts for nothing beside another's, so its sum is told apart from that of a share without
    // blocks by its sign: with weight 0 it adds nothing, and a token that has nothing else is NaN, like any mean over such logits)
    float *part = reinterpret_cast<float *>(smem);
    const float ref = st.slack > 0.f ? -st.nr : -INFINITY;
    if (share > 0) {
        float *p = part + ((share - 1) * T + ti) * kPart;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) *reinterpret_cast<f32x4 *>(p + (dt * 64 + lane) * 4) = st.o[dt];
        p[64 * 32 + lane] = ref;
        p[64 * 33 + lane] = took && st.l == 0.f ? -1.f : st.l;
    }
    __syncthreads();
    if (share > 0 || ti >= ntok) return;
    float refs[SH], top = ref;
    refs[0] = ref;
#pragma unroll
    for (int s = 1; s < SH; ++s) {
        refs[s] = part[((s - 1) * T + ti) * kPart + 64 * 32 + lane];
        top = fmaxf(top, refs[s]);
    }
    const float base = top == -INFINITY ? 0.f : top;
    float wt = fast_exp2(refs[0] - base), l = st.l * wt;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) st.o[dt] *= wt;
#pragma unroll
    for (int s = 1; s < SH; ++s) {
        const float *p = part + ((s - 1) * T + ti) * kPart;
        wt = fast_exp2(refs[s] - base);
        const float ls = p[64 * 33 + lane];
        took = took || ls != 0.f;
        l += (ls < 0.f ? 0.f : ls) * wt;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) st.o[dt] += *reinterpret_cast<const f32x4 *>(p + (dt * 64 + lane) * 4) * wt;
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const bool none = !(l > 0.f);
    const float inv = !none ? 1.0f / l : took ? NAN : 0.f;
    int lane_end = lane;
    asm volatile("" : "+v"(lane_end));           // the address is formed here, not kept in registers over the loop
    uint16_t *op = a.out + ((int64_t)(row0 + ti) * a.hq + h * G + (lane_end & 15)) * D + (lane_end >> 4) * 4;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
        *reinterpret_cast<uint2 *>(op + dt * 16) = make_uint2(pack_bf16(st.o[dt][0] * inv, st.o[dt][1] * inv), pack_bf16(st.o[dt][2] * inv, st.o[dt][3] * inv));
    if (a.lse != nullptr && g == 0)
        a.lse[(int64_t)(h * G + m16) * a.map.total_rows + row0 + ti] = none && took ? NAN : (__log2f(l) + base) * 0.6931471805599453f;
}

template <int SH>
int launch_short(const Launch &L, ShortArgs a, const int32_t *cu_h) {
    int64_t tiles = 0;
    for (int s = 0; s < L.map.batch; ++s) tiles += (cu_h[s + 1] - cu_h[s] + T - 1) / T;
    const int nb_max = (L.max_len + kBlock - 1) / kBlock;
    a.nb_cap = a.idx ? (nb_max + 3) / 4 * 4 : 0;
    const int list_cap = a.idx && nb_max > a.topk_total ? min(nb_max, T * a.topk_total) : 0;
    const size_t lds = stage_bytes<SH>() + (size_t)a.nb_cap * 4 + (size_t)list_cap * 8;
    if (lds > 160 * 1024 - 256) return INFLLMV2_ERR_UNSUPPORTED;
    void (*kern)(ShortArgs, int) = attn_short_kernel<SH>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return INFLLMV2_ERR_HIP;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles * L.p->num_kv_heads), dim3(T * SH * 64), lds, L.stream, a, (int)tiles);
    return hip_status(hipGetLastError());
}

}  // namespace

// INFLLMV2_ERR_UNSUPPORTED: the tile kernel is the faster one (or takes what this one has no room for)
int launch_attn_short(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, void *out,
                      float *lse, const int32_t *cu_h) {
    ShortArgs a{(const uint16_t *)q, (const uint16_t *)k, (const uint16_t *)v, idx, (uint16_t *)out, lse, L.map,
                L.p->num_q_heads, L.p->topk_total, dense_below, L.p->softmax_scale, 0};
    switch (rules::short_attn_waves(cu_h, L.map.batch, L.max_len, L.p->num_kv_heads, idx != nullptr, L.p->topk_total, dense_below)) {
        case 1: return launch_short<1>(L, a, cu_h);
        case 2: return launch_short<2>(L, a, cu_h);
        default: return INFLLMV2_ERR_UNSUPPORTED;
    }
}

}  // namespace ifv2
