// dK and dV of stage 4 on the matrix cores (bf16, 16 query heads per KV head, d_h = 128); see attn_bwd_mfma.hip for the
// mathematics and the other kernels of the call.
//
// A wavefront -- a workgroup of its own -- owns one 64-key block and the tokens of one chunk that selected it.  The K and V
// rows of the 64 keys (128 registers) and the dK and dV sums (256 accumulator registers) stay in its registers, so a
// token's 8 KB of Q and dO pass through LDS once for 64 keys.  Two tokens at a time: S = Q K^T and dP = dO V^T are products
// of 32 rows (2 tokens x 16 heads) with 32 keys, P and dZ come out with a lane's eight contraction indices of
// dV += P^T dO, dK += dZ^T Q side by side (one token's 16 heads per step), and the rows of dO and Q are read back
// transposed (ds_read_b64_tr_b16) for it: 64 products 32x32x16 per pair of tokens.  The rows go straight from global
// memory to LDS, one buffer computed, the other in flight; nothing waits for another wavefront, and the sums go to memory
// with one float atomic per element at the end.
//
// One wavefront per SIMD (512 registers) means that nobody else fills the gaps, so the vector work is interleaved by
// hand: the exponentials of a 32-key half are issued between the products of the other half.
//
// Which workgroup takes what: the 8 KB per (token, block) are the kernel's traffic (33 GB for 32768 tokens x 64 blocks
// x 2 heads), and far more than the block's own K and V.  A chunk of tokens therefore stays on one XCD (workgroup ids go
// round the eight XCDs) for all blocks that may need it, one block after the other, so that its rows come from that
// XCD's L2 instead of the memory-side cache (44% of them do).
//
// Measured at 32768 tokens, 64 blocks, 2 KV heads: 7.85 -> 5.1 ms, MFMA busy 45% of the time a wavefront runs.  The kernel
// this one replaced (four wavefronts of 16 keys, two tokens per barrier) took 6.2 ms with the order of chunks above.  Four
// wavefronts sharing a block and adding up in LDS: 5.4 ms; without the copies 3.7 ms; all rows L2 hits 4.6 ms; copies
// spread over the products instead of early: 5.8 ms; chunks of 512 / 256 tokens: 5.1 / 5.3 ms.
#include "attn_bwd.h"
#include "attn_unit.h"
#include "launch_rules.h"

namespace ifv2 {

namespace {

using attn_unit::async_copy16;
using attn_unit::bf16x8;
using attn_unit::f32x4;
using attn_unit::lds_address;
using attn_unit::pack_bf16;
using attn_unit::u32x4;

constexpr int D = 128, G = 16;
constexpr float LOG2E = 1.4426950408889634f;
constexpr int MAX_CHUNK = 1024;                        // tokens per workgroup at most (launch_rules.h)
constexpr uint32_t kTokBytes = 2 * G * D * 2;          // a token's Q rows, then its dO rows
constexpr uint32_t kMatBytes = G * D * 2;
constexpr uint32_t kPairBytes = 2 * kTokBytes + 256;   // two tokens, then lse and Delta of their heads
constexpr uint32_t kPairStride = (kPairBytes + 511) / 512 * 512;      // (addresses are formed by exclusive-or)
constexpr int WAIT_VMCNT0 = 0x0F70;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) const bf16x8 lds_b8;
typedef __attribute__((address_space(3))) short4v lds_s4;

__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// 16-byte chunk c of row n (a head) of a token's Q or dO rows lies at chunk c ^ f(n), f(n) = 4 (n % 4) + n / 4: the sixteen
// rows of a row read and the 4 rows x 4 chunks of a transposing read both fall on sixteen different positions.
__device__ inline int swz(int n) { return 4 * (n & 3) + (n >> 2); }

// 4 bytes per lane, global -> LDS (lane l's word at lds + 4 l)
__device__ inline void async_copy4(const float *src, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(src) : "memory", "m0");
}

// elements e and e + 1 of a half's 16: probabilities and dZ, packed.  s holds (q k - lse / scale) and dp holds (dO v - Delta)
// already (the sums were seeded with the subtrahends).
__device__ inline void prob_pair(const f32x16 &s, const f32x16 &dp, int e, float c, uint32_t &pw, uint32_t &zw) {
    const float p0 = exp2_fast(s[e] * c), p1 = exp2_fast(s[e + 1] * c);
    pw = pack_bf16(p0, p1);
    zw = pack_bf16(p0 * dp[e], p1 * dp[e + 1]);
}

// acc += a b with the sum in the accumulator half of the register file.  Written as assembly because the compiler's own
// choice for these 256 registers (next to 230 others) is to spill; the wait states that it would insert stand here:
// a (packed by the vector unit just before) may be read two instructions after it was written, and a sum may be read
// back 18 after the last product (settle).
__device__ inline void accumulate(f32x16 &acc, const u32x4 &a, const bf16x8 &b) {
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ inline void settle(f32x16 &acc) { asm volatile("s_nop 15\n\ts_nop 7" : "+a"(acc)); }

struct State {
    f32x16 k[2][4], v[2][4];       // dK, dV: keys 32 kt + 8 (e / 4) + 4 kg + e % 4, dim 32 dt + lane % 32
};

// one pair of tokens (positions t0, t1) from the LDS buffer at byte address buf; key0: this lane's key of the first half
template <class Copy>
__device__ inline void pair_step(State &acc, const bf16x8 (&kf)[2][8], const bf16x8 (&vf)[2][8], uint32_t buf, int lane,
                                 float c, int key0, int t0, int t1, bool diag, Copy copy) {
    const int kg = lane >> 5, n = lane & 15, L = lane & 15;
    // row operand of step ks: row lane % 32 = (token, head), chunk 2 ks + kg
    const uint32_t ra = buf + (uint32_t)(((lane >> 4) & 1) * kTokBytes + n * 256 + ((kg ^ swz(n)) << 4));
    auto rowq = [&](int ks) -> bf16x8 { return *(lds_b8 *)(uintptr_t)(ra ^ (uint32_t)(32 * ks)); };
    auto rowg = [&](int ks) -> bf16x8 { return *(lds_b8 *)(uintptr_t)((ra ^ (uint32_t)(32 * ks)) + kMatBytes); };
    // transposed operand of token a and dims 32 dt ..: heads 4 kg .. + 3 and 8 + 4 kg .. + 3 of dim 32 dt + lane % 32
    const int head = 4 * kg + (L >> 2);
    const uint32_t ta = buf + (uint32_t)(head * 256 + (((2 * ((lane >> 4) & 1) + ((L & 3) >> 1)) ^ swz(head)) << 4) + (L & 1) * 8);
    auto trans = [&](int a, int dt, uint32_t mat) -> bf16x8 {
        const uint32_t x = (ta ^ (uint32_t)(64 * dt)) + (uint32_t)a * kTokBytes + mat;
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(uintptr_t)x);
        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(uintptr_t)((x ^ 32u) + 2048u));
        const short8v r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, r);
    };
    // Seeds: element e is row 8 (e / 4) + 4 kg + e % 4 of the 32 (token, head) rows.  Minus lse / scale and minus Delta of
    // its token and head, so that the products come out subtracted.
    const uint32_t sa = buf + 2 * kTokBytes + (uint32_t)(kg * 16);
    auto seed = [&](int which) -> f32x16 {
        typedef __attribute__((address_space(3))) const f32x4 lds_f4;
        f32x16 r;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 x = *(lds_f4 *)(uintptr_t)(sa + (uint32_t)((q >> 1) * 128 + which * 64 + (q & 1) * 32));
#pragma unroll
            for (int u = 0; u < 4; ++u) r[4 * q + u] = x[u];
        }
        return r;
    };
    // A key the token does not see (yet: the token then lies in the block itself) gets probability 0 and dP 0.  In the
    // finished products: a seed of minus infinity would not hide a key whose row holds infinities.
    auto hide = [&](f32x16 &x, f32x16 &y, int key) {
        if (!diag) return;                                 // (uniform)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (key > (e < 8 ? t0 : t1)) {
                x[e] = -INFINITY;
                y[e] = 0.f;
            }
    };
    f32x16 s[2], dp[2];
    u32x4 pw[2][2], zw[2][2];       // [half][token]: eight bf16
    // ---- S and dP, 32 keys after 32; operands are requested W1 - 1 steps ahead.  Beside the first half's products the next
    // pair's rows are requested (`copy`), beside the second half's the first half's probabilities are computed.
    constexpr int W1 = 3;
    bf16x8 qa[W1], ga[W1];
    auto fetch1 = [&](int i) {
        qa[i % W1] = rowq(i & 7);
        ga[i % W1] = rowg(i & 7);
    };
    constexpr int W2 = 3;           // the same for the products with transposed operands
    bf16x8 gb[W2], qb[W2];
    auto fetch2 = [&](int i) {
        gb[i % W2] = trans((i >> 2) & 1, i & 3, kMatBytes);
        qb[i % W2] = trans((i >> 2) & 1, i & 3, 0);
    };
    s[0] = seed(0);
    dp[0] = seed(1);
#pragma unroll
    for (int i = 0; i < W1 - 1; ++i) fetch1(i);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int kt = i >> 3, ks = i & 7;
        if (i + W1 - 1 < 16) fetch1(i + W1 - 1);
        else fetch2(i + W1 - 1 - 16);
        if (i == 5) {
            s[1] = seed(0);
            dp[1] = seed(1);
        }
        s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa[i % W1], kf[kt][ks], s[kt], 0, 0, 0);
        dp[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ga[i % W1], vf[kt][ks], dp[kt], 0, 0, 0);
        if (i < 8) {
            copy(2 * i);
            copy(2 * i + 1);
        }
        if (i == 8) hide(s[0], dp[0], key0);
        if (kt == 1) {
            uint32_t p, z;
            prob_pair(s[0], dp[0], 2 * ks, c, p, z);
            pw[0][ks >> 2][ks & 3] = p;
            zw[0][ks >> 2][ks & 3] = z;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // ---- dV, dK, 32 keys after 32; beside the first half's products the other half's probabilities are computed
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int kt = i >> 3, a = (i >> 2) & 1, dt = i & 3;
        if (i + W2 - 1 < 16) fetch2(i + W2 - 1);
        accumulate(acc.v[kt][dt], pw[kt][a], gb[i % W2]);
        accumulate(acc.k[kt][dt], zw[kt][a], qb[i % W2]);
        if (i == 0) hide(s[1], dp[1], key0 + 32);
        if (kt == 0) {
            uint32_t p, z;
            prob_pair(s[1], dp[1], 2 * i, c, p, z);
            pw[1][i >> 2][i & 3] = p;
            zw[1][i >> 2][i & 3] = z;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

__global__ void __launch_bounds__(64, 1) bwd_dkv_mfma_kernel(BwdM a, int chunk, int groups) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * kPairStride];      // two buffers of a pair of tokens
    __shared__ uint16_t s_list[MAX_CHUNK];                             // tokens of the chunk that selected the block
    __shared__ int s_tile[3];
    const int lane = threadIdx.x;
    const int nb = (int)a.nblocks;
    // XCD x (= workgroup id mod 8) takes the (chunk, KV head) groups x, x + 8, ...; the first block, whose list holds every
    // token of a chunk when it is an initial block, of all of them first, then group by group from the last block down
    // (the blocks next to the chunk have the next longest lists).  The groups move on by one XCD from sequence to sequence:
    // those of a batch of short sequences are few and unlike (40 sequences of 777 tokens: eight, between 117 and 2688 entries
    // per sequence; 1148 -> 667 us); and by one more from eight sequences to the next: of one group per sequence every
    // eighth of an XCD's workgroups would have tokens, which an XCD of 32 CUs deals to four of them (1000 x 64 tokens on 1 KV
    // head, whole backward, 1362 -> 1170 us, 400 x 100 656 -> 558).
    const int per_xcd = (groups + 7) >> 3, slot = (int)blockIdx.x >> 3;
    const int ord = slot < per_xcd ? 0 : 1 + (slot - per_xcd) % max(nb - 1, 1);
    int j;
    const int seq = find_seq_tile(a.map.cu, a.map.batch, kBlock, ord == 0 ? 0 : nb - ord, j, s_tile);
    const int grp = (slot < per_xcd ? slot : (slot - per_xcd) / max(nb - 1, 1)) * 8 + (((int)blockIdx.x + seq + (seq >> 3)) & 7);
    if (seq >= a.map.batch || grp >= groups) return;
    const int h = grp % a.map.num_kv_heads, c0 = grp / a.map.num_kv_heads * chunk;
    const int tok0 = a.map.cu[seq], len = a.map.cu[seq + 1] - tok0;
    const int c1 = min(c0 + chunk, len);
    if (c1 <= j * kBlock || c0 >= len) return;
    const bool dense = a.idx == nullptr || len < a.dense_below;

    // ---- tokens of the chunk that selected the block, in token order
    int total = 0;
    if (!dense && a.sel_bits != nullptr) {
        // from the selection bitmap: lane l expands the chunk's bits [l n, (l + 1) n), n = chunk / 64 (at least 1)
        const int words = (len + 31) / 32, n = max(chunk / 64, 1), first = c0 + lane * n;
        const uint32_t *row = a.sel_bits + (int64_t)h * a.sel_words + sel_base(a.map, seq) + (int64_t)j * words;
        // (words of tokens in front of the block are not written)
        const uint32_t word = first < c1 && (first & ~31) >= j * kBlock ? row[first >> 5] : 0u;
        const uint32_t bits = (word >> (first & 31)) & ((1u << n) - 1u);
        const int cnt = __popc(bits);
        int incl = cnt;                                        // inclusive prefix
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o);
            if (lane >= o) incl += up;
        }
        total = __builtin_amdgcn_readlane(incl, 63);
        int base = incl - cnt;
        for (uint32_t rest = bits; rest; rest &= rest - 1) s_list[base++] = (uint16_t)(n * lane + __ffs(rest) - 1);
    } else {
        constexpr int U = 4;                                   // tokens per lane and step (searches overlap)
        for (int r0 = c0; r0 < c1; r0 += 64 * U) {
            bool sel[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = r0 + 64 * u + lane;
                sel[u] = t < c1 && t >= j * kBlock;
                if (sel[u] && !dense) sel[u] = list_has(a.idx + head_row(a.map, h, tok0 + t) * a.topk_total, a.topk_total, j);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t bal = __ballot(sel[u]);
                if (sel[u]) s_list[total + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(r0 + 64 * u + lane - c0);
                total += __popcll(bal);
            }
        }
    }
    if (total == 0) return;                                    // (uniform)
    __syncthreads();
    const int pairs = (total + 1) / 2;

    State acc;
    const f32x16 zero = {0.f};
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) acc.k[kt][dt] = acc.v[kt][dt] = zero;
    {
        // K and V rows of the 64 keys as second operands (rows past the sequence: the last one, never visible)
        bf16x8 kf[2][8], vf[2][8];
        const int key0 = j * kBlock + (lane & 31);
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            const int64_t off = (int64_t)(tok0 + min(key0 + 32 * kt, len - 1)) * a.map.kv_tok_stride +
                                (int64_t)h * a.map.kv_head_stride + (lane >> 5) * 8;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                kf[kt][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(a.k + off + ks * 16));
                vf[kt][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(a.v + off + ks * 16));
            }
        }
        const uint32_t lds_w = __builtin_amdgcn_readfirstlane(lds_address(smem));
        // one 1 KB piece = rows 4 x .. 4 x + 3: lane l fills (row 4 x + l / 16, position l % 16)
        // (swz(4 x + y) = swz(y) ^ x for y < 4)
        const uint32_t voff = (uint32_t)((lane >> 4) * 256 + (((lane & 15) ^ swz(lane >> 4)) << 4));
        auto entry = [&](int i) -> int { return (int)s_list[min(i, total - 1)]; };
        auto uniform = [&](int x) -> int { return c0 + __builtin_amdgcn_readfirstlane(x); };
        // requests a sixteenth of the rows of the pair (ta, tb) into a buffer.  An odd last token's partner is a token that
        // sees no key, with rows of zeros (the copies repeat the last token and are overwritten).
        auto copy_share = [&](int ta, int tb, uint32_t buf, int x) {
            const int64_t row = (int64_t)(tok0 + (x & 8 ? tb : ta)) * a.hq + h * G;
            const uint16_t *src = (x & 4 ? a.dout : a.q) + row * D;
            async_copy16(reinterpret_cast<const char *>(src) + (x & 3) * 1024, voff ^ (uint32_t)((x & 3) << 4),
                         buf + (x & 8 ? kTokBytes : 0u) + (x & 4 ? kMatBytes : 0u) + (x & 3) * 1024u);
            if (x == 15) {
                const int64_t r2 = (int64_t)(tok0 + (lane >> 5 ? tb : ta)) * a.hq + h * G + (lane & 15);
                async_copy4(((lane >> 4) & 1 ? a.ndelta : a.nlse) + r2, buf + 2 * kTokBytes);
            }
        };
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {                   // the zeros are in place before the first product
                settle(acc.k[kt][dt]);
                settle(acc.v[kt][dt]);
            }
        int pi = 0;
        uint32_t cur = lds_w, nxt = lds_w + kPairStride;
        int ta = uniform(entry(0)), tb = uniform(entry(1)), la = entry(2), lb = entry(3);
#pragma unroll
        for (int x = 0; x < 16; ++x) copy_share(ta, tb, cur, x);
        const float c = a.scale * LOG2E;
        while (pi < pairs) {
            const int pn = pi + 1;
            const int na = uniform(la), nbt = uniform(lb);       // (past the end: the last token, not used)
            la = entry(2 * pn + 2);                              // read a pair ahead of their use
            lb = entry(2 * pn + 3);
            __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);           // this pair's rows (and, at first, K and V) are there
            asm volatile("" ::: "memory");
            const bool odd = 2 * pi + 1 == total;
            if (odd) {
                typedef __attribute__((address_space(3))) u32x4 lds_u4;
#pragma unroll
                for (int x = 0; x < 8; ++x) *(lds_u4 *)(uintptr_t)(cur + kTokBytes + x * 1024u + (uint32_t)lane * 16u) = (u32x4)0u;
                asm volatile("" ::: "memory");
            }
            // (the other buffer's last readers were the products of the previous step)
            pair_step(acc, kf, vf, cur, lane, c, key0, ta, odd ? -1 : tb, odd || ta < j * kBlock + kBlock - 1, [&](int x) {
                if (pn < pairs) copy_share(na, nbt, nxt, x);
            });
            asm volatile("" ::: "memory");
            const uint32_t sw = cur;
            cur = nxt;
            nxt = sw;
            pi = pn;
            ta = na;
            tb = nbt;
        }
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                settle(acc.k[kt][dt]);
                settle(acc.v[kt][dt]);
            }
    }
    // ---- the L2's own float adds (no CAS loop); an instruction covers 32 consecutive dims of two rows
    const int64_t base = ((int64_t)h * a.map.total_rows + tok0 + j * kBlock) * D + (lane & 31);
    const int rows = len - j * kBlock;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int key = 32 * kt + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            if (key >= rows) continue;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                unsafeAtomicAdd(a.dk + base + key * D + 32 * dt, acc.k[kt][dt][e] * a.scale);
                unsafeAtomicAdd(a.dv + base + key * D + 32 * dt, acc.v[kt][dt][e]);
            }
        }
}

}  // namespace

int launch_bwd_dkv(const BwdM &a, int chunk, int32_t max_len, hipStream_t stream) {
    const int hkv = a.map.num_kv_heads;
    hipLaunchKernelGGL(bwd_dkv_mfma_kernel, dim3((unsigned)rules::dkv_workgroups(max_len, hkv, a.nblocks, chunk)), dim3(64), 0, stream,
                       a, chunk, (max_len + chunk - 1) / chunk * hkv);
    return hip_status(hipGetLastError());
}

}  // namespace ifv2
