// Generic attention and dQ of bf16 rows that pass through LDS (attn_staged.hip).
#pragma once
#include "common.h"
#include "launch_rules.h"

namespace ifv2 {

// bf16 prefill calls with rows and strides of 16-byte multiples (whether there are workgroups enough, and not more than a launch holds:
// rules::staged)
bool attn_staged_takes(const Launch &L, const void *k, const void *v);

// walks: of the batch's tiles of one column group (rules::walks); cu_h: host cu_seqlens
int launch_attn_staged(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, void *out,
                       float *lse, const int32_t *cu_h, const rules::Walks &walks);
// delta: <dO, O> per (query head, row)
int launch_dq_staged(const Launch &L, const void *q, const void *k, const void *v, const int32_t *idx, int dense_below, const float *lse,
                     const float *delta, const void *dout, void *dq, const int32_t *cu_h, const rules::Walks &walks);

}  // namespace ifv2
