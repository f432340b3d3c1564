// Generic attention and dQ of bf16 rows that pass through LDS (attn_staged.hip).
#pragma once
#include "common.h"

namespace ifv2 {

// bf16 prefill calls with rows and strides of 16-byte multiples (whether there are workgroups enough, and not more than a launch holds:
// rules::staged)
bool attn_staged_takes(const Launch &L, const void *k, const void *v);

// tiles: of two column groups, over the whole batch
int launch_attn_staged(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, void *out,
                       float *lse, int64_t tiles);
// delta: <dO, O> per (query head, row)
int launch_dq_staged(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, const float *lse,
                     const float *delta, const void *dout, void *dq, int64_t tiles);

}  // namespace ifv2
