// Matrix-core building blocks of the generic kernels (any G <= 16, d in {64, 128}, fp32 or bf16 data): products whose
// probabilities, weights and sums stay in 32 bits.
//
// A wavefront works on 16 columns.  A column is a (token, head) pair: 16 / G consecutive tokens of one KV head with
// their G heads each, so that a group smaller than 16 does not leave the matrix cores idle and a K/V block that
// neighbouring tokens share is read once for all of them.  Products of two stored rows (Q K^T, dO V^T) run on
// v_mfma_f32_16x16x32_bf16 for bf16 data (the products are exact, the sum is fp32) and on v_mfma_f32_16x16x4_f32
// for fp32 data.  In products with a computed operand (P V, dZ K, P^T dO, dZ^T Q) that operand keeps its 24 bits: see
// weighted_rows.
//
// Layouts, with m = lane % 16 and g = lane / 16.  Row products give a lane the elements (row 4 g + r, column m),
// r = 0..3, and that is exactly what the 16x16x4 instruction wants as its second (or first) operand for the four
// contraction indices 4 g + r: no lane exchange and no LDS between the two products.
#pragma once
#include "common.h"

namespace ifv2 {
namespace gen {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int kCols = 16;
constexpr float kLog2e = 1.4426950408889634f;

__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline bool finite(float x) { return fabsf(x) <= 3.4028234e38f; }

// N consecutive elements at an address that is only known to be aligned to its element (this path serves every
// stride and every pointer the entry points accept; the hardware takes wide global accesses at any alignment)
template <typename E, int N>
struct Unaligned {
    typedef E type __attribute__((ext_vector_type(N), aligned(sizeof(E))));
};
typedef Unaligned<uint16_t, 8>::type u16x8_u;
typedef Unaligned<uint16_t, 4>::type u16x4_u;
typedef Unaligned<float, 4>::type f32x4_u;
typedef Unaligned<float, 8>::type f32x8_u;

// One row (key, token-head or compressed key) as an operand of a row product: lane (m, g) holds a quarter of row m.
// Which elements a lane group takes does not matter as long as both operands agree.
template <typename T, int D> struct RowFrag;
template <int D> struct RowFrag<bf16_t, D> {
    bf16x8 x[D / 32];
    __device__ inline void load(const bf16_t *row, int g) {
#pragma unroll
        for (int s = 0; s < D / 32; ++s)
            x[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8_u *>(row + 32 * s + 8 * g));
    }
    __device__ inline void load_at(const char *base, uint32_t off) {      // lane offset: row and quarter, in bytes
#pragma unroll
        for (int s = 0; s < D / 32; ++s) x[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8_u *>(base + off + 64 * s));
    }
    __device__ inline void load_lds(const bf16_t *row, int g) {   // 16-byte aligned rows
#pragma unroll
        for (int s = 0; s < D / 32; ++s) x[s] = *reinterpret_cast<const bf16x8 *>(row + 32 * s + 8 * g);
    }
};
template <int D> struct RowFrag<float, D> {
    f32x4 x[D / 16];
    __device__ inline void load(const float *row, int g) {
#pragma unroll
        for (int c = 0; c < D / 16; ++c)
            x[c] = __builtin_bit_cast(f32x4, *reinterpret_cast<const f32x4_u *>(row + 16 * c + 4 * g));
    }
    __device__ inline void load_at(const char *base, uint32_t off) {
#pragma unroll
        for (int c = 0; c < D / 16; ++c) x[c] = __builtin_bit_cast(f32x4, *reinterpret_cast<const f32x4_u *>(base + off + 64 * c));
    }
    __device__ inline void load(const bf16_t *row, int g) {       // bf16 data against a float32 operand
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            const u16x4_u r = *reinterpret_cast<const u16x4_u *>(row + 16 * c + 4 * g);
            x[c] = f32x4{bf16_to_float(r[0]), bf16_to_float(r[1]), bf16_to_float(r[2]), bf16_to_float(r[3])};
        }
    }
    __device__ inline void load_lds(const float *row, int g) {
#pragma unroll
        for (int c = 0; c < D / 16; ++c) x[c] = *reinterpret_cast<const f32x4 *>(row + 16 * c + 4 * g);
    }
};

// element r: <row 4 g + r of a, row m of b>
template <int D>
__device__ inline f32x4 row_product(const RowFrag<bf16_t, D> &a, const RowFrag<bf16_t, D> &b) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 32; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.x[s], b.x[s], acc, 0, 0, 0);
    return acc;
}
// (fp32: four partial sums, which halves the rounding error of one long chain and leaves independent products to issue)
template <int D>
__device__ inline f32x4 row_product(const RowFrag<float, D> &a, const RowFrag<float, D> &b) {
    f32x4 acc[4];
#pragma unroll
    for (int c = 0; c < D / 16; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[c][j], b.x[c][j], c ? acc[j] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// One contraction index's row for a product with a computed operand: lane (m, g) holds elements D/16 m .. + D/16 - 1
// of its row, widened to fp32; element j belongs to the j-th 16-wide tile of the result, whose row (column) i is
// therefore element D/16 i + j.
template <typename T, int D>
struct Spread {
    static constexpr int N = D / 16;                              // elements per lane
    static constexpr int W = N * (int)sizeof(T) / 4;              // ... in 32-bit words
    static constexpr int kLdsAlign = W * 4 < 16 ? W * 4 : 16;
    typedef uint32_t Words __attribute__((ext_vector_type(W)));
    typedef uint32_t UWords __attribute__((ext_vector_type(W), aligned(sizeof(T))));
    typedef uint32_t LWords __attribute__((ext_vector_type(W), aligned(kLdsAlign)));
    Words raw;
    __device__ inline void load(const T *row, int m) { raw = *reinterpret_cast<const UWords *>(row + m * N); }
    __device__ inline void load_at(const char *base, uint32_t off) { raw = *reinterpret_cast<const UWords *>(base + off); }
    __device__ inline void load_lds(const T *row, int m) { raw = *reinterpret_cast<const LWords *>(row + m * N); }
    __device__ inline void store_lds(T *row, int m) const { *reinterpret_cast<LWords *>(row + m * N) = raw; }
    __device__ inline void zero() { raw = 0u; }
};

// acc += (computed weights) x (rows v[0..3]) over the sixteen contraction indices 4 g + r: w[r] is this lane's weight of
// index 4 g + r (for result row / column m), v[r] its row.  WEIGHTS_FIRST: the weights are the first operand, i.e.
// acc[j] holds (weight row 4 g + r, element N m + j); otherwise (element N (4 g + r) + j, weight column m).
//
// fp32 rows: 4 N products 16x16x4.
template <bool WEIGHTS_FIRST, int D>
__device__ inline void weighted_rows(f32x4 (&acc)[D / 16], f32x4 w, const Spread<float, D> (&v)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < D / 16; ++j) {
            const float x = __uint_as_float(v[r].raw[j]);
            acc[j] = WEIGHTS_FIRST ? __builtin_amdgcn_mfma_f32_16x16x4f32(w[r], x, acc[j], 0, 0, 0)
                                   : __builtin_amdgcn_mfma_f32_16x16x4f32(x, w[r], acc[j], 0, 0, 0);
        }
}
// the upper (lower) halves of two words, a's first
__device__ inline uint32_t upper_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
__device__ inline uint32_t lower_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }

// The same over the 32 contraction indices of two such groups of rows (weights w0 with rows a, w1 with rows b).  bf16 rows: the
// weights are cut, exactly, into three bf16 pieces of eight significant bits each (truncation, so that nothing rounds), and
// 3 N products 16x16x32 with the rows as stored give the same sum of fp32 weights x bf16 values -- a product of either kind
// adds in fp32 -- in 3/16 of the matrix-core time (a product 16x16x16 occupies the matrix core as long as one over 32).
// CHECKED: the weights may be infinite (an unchecked infinite weight gives NaN, an infinite one is its own first piece).
template <bool WEIGHTS_FIRST, bool CHECKED, int D>
__device__ inline void weighted_rows32(f32x4 (&acc)[D / 16], f32x4 w0, f32x4 w1, const Spread<float, D> (&a)[4],
                                       const Spread<float, D> (&b)[4]) {
    weighted_rows<WEIGHTS_FIRST, D>(acc, w0, a);
    weighted_rows<WEIGHTS_FIRST, D>(acc, w1, b);
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// the next piece of eight weights; what is left stays in w0, w1
template <bool CHECKED>
__device__ inline bf16x8 take_piece32(f32x4 &w0, f32x4 &w1) {
    uint32_t u[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        u[r] = __float_as_uint(w0[r]);
        u[4 + r] = __float_as_uint(w1[r]);
        const float r0 = w0[r] - __uint_as_float(u[r] & 0xffff0000u), r1 = w1[r] - __uint_as_float(u[4 + r] & 0xffff0000u);
        w0[r] = CHECKED && !finite(w0[r]) ? 0.f : r0;
        w1[r] = CHECKED && !finite(w1[r]) ? 0.f : r1;
    }
    return __builtin_bit_cast(bf16x8, (u32x4){upper_halves(u[0], u[1]), upper_halves(u[2], u[3]), upper_halves(u[4], u[5]),
                                              upper_halves(u[6], u[7])});
}
template <bool WEIGHTS_FIRST, bool CHECKED, int D>
__device__ inline void weighted_rows32(f32x4 (&acc)[D / 16], f32x4 w0, f32x4 w1, const Spread<bf16_t, D> (&a)[4],
                                       const Spread<bf16_t, D> (&b)[4]) {
    const bf16x8 p0 = take_piece32<CHECKED>(w0, w1), p1 = take_piece32<CHECKED>(w0, w1), p2 = take_piece32<CHECKED>(w0, w1);
#pragma unroll
    for (int j = 0; j < D / 16; ++j) {
        const int i = j / 2;
        const u32x4 x = j & 1 ? (u32x4){upper_halves(a[0].raw[i], a[1].raw[i]), upper_halves(a[2].raw[i], a[3].raw[i]),
                                        upper_halves(b[0].raw[i], b[1].raw[i]), upper_halves(b[2].raw[i], b[3].raw[i])}
                              : (u32x4){lower_halves(a[0].raw[i], a[1].raw[i]), lower_halves(a[2].raw[i], a[3].raw[i]),
                                        lower_halves(b[0].raw[i], b[1].raw[i]), lower_halves(b[2].raw[i], b[3].raw[i])};
        const bf16x8 row = __builtin_bit_cast(bf16x8, x);
        if (WEIGHTS_FIRST) {
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p2, row, acc[j], 0, 0, 0);
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p1, row, acc[j], 0, 0, 0);
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p0, row, acc[j], 0, 0, 0);
        } else {
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(row, p2, acc[j], 0, 0, 0);
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(row, p1, acc[j], 0, 0, 0);
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(row, p0, acc[j], 0, 0, 0);
        }
    }
}

// K or V rows of one (sequence, KV head): 32 consecutive keys at a time as row fragments or spread rows.  The address of a
// row is a scalar base and a lane offset that stays the same for the whole walk; only the 32 keys that hold the sequence's
// end (rows past it repeat the last one), and token strides of 2^26 bytes and more, form it per lane.
template <typename T, int D>
struct KeyRows {
    const char *base;              // token 0 of the sequence, this head
    int64_t stride;                // bytes from token to token
    int len;
    uint32_t frag_off, spread_off;
    bool narrow;
    __device__ inline KeyRows(const T *p, int64_t tok_stride, int len_, int m, int g)
        : base(reinterpret_cast<const char *>(p)), stride(tok_stride * (int64_t)sizeof(T)), len(len_) {
        narrow = stride < (1 << 26) && stride >= 0;
        frag_off = (uint32_t)((int)stride * m + 16 * g);
        spread_off = (uint32_t)((int)stride * 4 * g + m * (D / 16) * (int)sizeof(T));
    }
    __device__ inline void frags(RowFrag<T, D> (&f)[2], int key0, int m, int g) const {
        if (narrow && key0 + 32 <= len) {
            const char *p = base + (int64_t)key0 * stride;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) f[kt].load_at(p + 16 * kt * stride, frag_off);
        } else {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
                f[kt].load(reinterpret_cast<const T *>(base + (int64_t)min(key0 + 16 * kt + m, len - 1) * stride), g);
        }
    }
    __device__ inline void spread(Spread<T, D> (&v)[2][4], int key0, int m, int g) const {
        if (narrow && key0 + 32 <= len) {
            const char *p = base + (int64_t)key0 * stride;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r) v[kt][r].load_at(p + (16 * kt + r) * stride, spread_off);
        } else {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    v[kt][r].load(reinterpret_cast<const T *>(base + (int64_t)min(key0 + 16 * kt + 4 * g + r, len - 1) * stride), m);
        }
    }
};

// max / sum over the four lane groups (lanes with equal lane % 16), result in every lane
__device__ inline float groups_max(float x) {
    const unsigned u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const unsigned v = __float_as_uint(y);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ inline float groups_sum(float x) {
    const unsigned u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const unsigned v = __float_as_uint(y);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// N consecutive results to memory
template <typename T, int N>
__device__ inline void store_row(T *dst, const float (&x)[N]) {
    if constexpr (sizeof(T) == 2) {
        typename Unaligned<uint16_t, N>::type r;
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = float_to_bf16(x[j]);
        *reinterpret_cast<decltype(r) *>(dst) = r;
    } else {
        typename Unaligned<float, N>::type r;
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = x[j];
        *reinterpret_cast<decltype(r) *>(dst) = r;
    }
}

// The tile of tokens a workgroup works for: kCols / G consecutive tokens of one sequence (decode: one row).
struct Tile {
    int seq, t0, ntok, len;       // first position, tokens (>= 1), sequence length
    int row0;                     // packed row of the first token
    int64_t kv_base;              // element offset of (token 0, head 0) of the sequence in K / V
};
__host__ __device__ inline int tile_tokens(const RowMap &m, int G) { return m.ctx ? 1 : kCols / G; }

// wave 0 looks the tile up (64 sequences per step), every thread gets it; a barrier only if it has to look
// among several sequences.  false: past the last tile
__device__ inline bool find_tile(const RowMap &m, int tile, int tokens, Tile &t, int *s_tile /* 3 ints of LDS */) {
    if (m.ctx) {
        t.seq = tile;
        t.len = m.ctx[tile];
        t.t0 = t.len - 1;
        t.ntok = 1;
        t.row0 = tile;
        t.kv_base = (int64_t)tile * m.kv_batch_stride;
        return true;
    }
    int rem;
    const int seq = find_seq_tile(m.cu, m.batch, tokens, tile, rem, s_tile);
    if (seq >= m.batch) return false;
    const int a = m.cu[seq];
    t.seq = seq;
    t.len = m.cu[seq + 1] - a;
    t.t0 = rem * tokens;
    t.ntok = min(tokens, t.len - t.t0);
    t.row0 = a + t.t0;
    t.kv_base = (int64_t)a * m.kv_tok_stride;
    return true;
}

// The b-th of n workgroups that are all on the chip at once, in an order of falling work: workgroups b and b + 256 share one of the 256 CUs,
// so every second row of 256 goes backwards and long tiles have short ones beside them.
__device__ inline uint32_t back_and_forth(uint32_t b, uint32_t n) {
    const uint32_t row = b & ~255u;
    return b & 256u ? 2 * row + min(255u, n - 1 - row) - b : b;
}

// The union of a tile's block lists, kChunk block numbers at a time: after build() the LDS list holds (block, mask of
// the tokens that take it) in ascending order for the blocks [c0, c0 + kChunk).
constexpr int kChunk = 1024;
struct Union {
    uint32_t masks[kChunk];
    int2 list[kChunk];
    int count;
    // lists: the tile's rows of the block lists (ntok rows of `topk` entries), or nullptr: every block for every token
    __device__ inline void build(const int32_t *lists, int topk, const Tile &t, int c0, int nblk, uint32_t all, int tid,
                                 int nthr) {
        const int n = min(kChunk, nblk - c0);
        if (lists == nullptr) {
            for (int i = tid; i < n; i += nthr) list[i] = make_int2(c0 + i, (int)all);
            if (tid == 0) count = n;
            __syncthreads();
            return;
        }
        for (int i = tid; i < n; i += nthr) masks[i] = 0u;
        __syncthreads();
        for (int e = tid; e < t.ntok * topk; e += nthr) {
            const int ti = e / topk;
            const int j = lists[e];
            if (j >= c0 && j < c0 + n && j <= (t.t0 + ti) / kBlock) atomicOr(&masks[j - c0], 1u << ti);
        }
        __syncthreads();
        if (tid < 64) {
            int base = 0;
            for (int b = 0; b < n; b += 64) {
                const uint32_t mk = b + tid < n ? masks[b + tid] & all : 0u;
                const uint64_t bal = __ballot(mk != 0u);
                if (mk != 0u) list[base + __popcll(bal & ((1ull << tid) - 1ull))] = make_int2(c0 + b + tid, (int)mk);
                base += __popcll(bal);
            }
            if (tid == 0) count = base;
        }
        __syncthreads();
    }
    // half blocks (32 keys) of the list; no token of the tile sees the last one if that starts behind all of them
    __device__ inline int half_blocks(const Tile &t) const {
        return 2 * count - (count > 0 && list[count - 1].x * kBlock + 32 > t.t0 + t.ntok - 1 ? 1 : 0);
    }
};

}  // namespace gen
}  // namespace ifv2
