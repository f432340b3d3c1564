// Rows of 16-bit elements in LDS, 256 bytes each, read both as they are and transposed: K and V of the backward unit and of short prompts
// (attn_unit.h), of the staged generic kernels (attn_staged.hip), Q and dO of the generic dK/dV (attn_bwd.hip).
//
// 16-byte chunk c of row r lies at chunk c ^ swizzle(r): the sixteen rows of an operand read take sixteen positions, and so do the 8 rows x 2
// chunks that half a wave touches in a transposing read.  Row x of product tile kt is row 8 (x / 4) + 4 kt + x % 4, so that the four results of a
// lane (m = lane % 16, g = lane / 16) in two tiles are rows 8 g .. 8 g + 7, as the operand of the second product wants them.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ifv2 {
namespace lds_rows {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 Frag;

constexpr uint32_t kRowBytes = 256;

__device__ inline int swizzle(int r) { return 4 * (r & 3) + 2 * ((r >> 3) & 1) + ((r >> 4) & 1); }
__device__ inline uint32_t offset(int row, int chunk) { return (uint32_t)row * kRowBytes + (uint32_t)((chunk ^ swizzle(row)) << 4); }

// the row of a lane in the row operand of tile 0, and of the piece that it reads transposed (4 x 16: rows 8 g + m / 4, dims 4 (m % 4) ..)
__device__ inline int operand_row(int m) { return 8 * (m >> 2) + (m & 3); }
__device__ inline int piece_row(int m, int g) { return 8 * g + (m >> 2); }
__device__ inline int piece_chunk(int m) { return (m & 3) >> 1; }
__device__ inline uint32_t piece_half(int m) { return (m & 1) * 8; }

// row operand of tile kt, k-step s; at: address of the lane's row of tile 0 at chunk g
__device__ inline Frag operand(uint32_t at, int kt, int s) {
    typedef __attribute__((address_space(3))) const Frag lds_frag;
    return *(lds_frag *)(uintptr_t)((at ^ (uint32_t)(64 * s)) + (uint32_t)(4 * kt) * kRowBytes);
}
// rows 8 g .. 8 g + 7 of the 16 dims at x, one per lane; x: address of the lane's piece
__device__ inline Frag transposed(uint32_t x) {
    typedef short Four __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) Four lds_four;
    const Four lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_four *)(uintptr_t)x);
    const Four hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_four *)(uintptr_t)(x + 4 * kRowBytes));
    return __builtin_bit_cast(Frag, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

}  // namespace lds_rows
}  // namespace ifv2
