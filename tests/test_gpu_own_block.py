"""The matrix-core attention kernels when a token's list leaves its own block out (any block numbers <= its own are a valid
list), at every tile size of the forward and of dQ (4, 8 and 16 tokens), against the CPU oracle through the C ABI."""
import numpy as np
import pytest
import torch

import synth
from helpers import assert_out_close, prefill_lse_atol, to_dev, to_np
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


def _lists(lens, topk, rng):
    """Random ascending lists of earlier blocks; the own block only in the first block of a sequence (there is no other), in
    every third token of the odd blocks, and in none of the even ones."""
    idx = np.full((1, sum(lens), topk), -1, np.int32)
    row = 0
    for n in lens:
        for t in range(n):
            bt = t // 64
            own = bt == 0 or (bt % 2 == 1 and t % 3 == 0)
            pick = rng.permutation(bt)[:topk - int(own)]
            entries = np.sort(np.append(pick, [bt] if own else [])).astype(np.int32)
            idx[0, row, :len(entries)] = entries
            row += 1
    return idx


@pytest.mark.parametrize("lens", [[700], [1500], [2600], [130, 1, 65, 901]])
def test_lists_without_the_tokens_own_block(m, oracle, lens):  # noqa: F811
    T, topk = sum(lens), 6
    w = synth.make_varlen(lens, 16, 1, 128, seed=2100 + T, dtype="bf16")
    gp, op = _params(m, oracle, "bf16", 16, 1, 128, n_init=1, n_local=1, topk_total=topk)
    idx = _lists(lens, topk, np.random.default_rng(2101))
    q, k, v, idx_d = *(to_dev(w[x], "bf16") for x in ("q", "k", "v")), torch.from_numpy(idx).cuda()
    dout = torch.randn(q.shape, generator=torch.Generator("cuda").manual_seed(5), device="cuda").bfloat16()
    cu = w["cu_seqlens"]
    out, lse = m.sparse_attn_fwd(gp, q, k, v, idx_d, cu)
    grads = m.sparse_attn_bwd(gp, q, k, v, idx_d, out, lse, dout, cu)
    for s in range(len(lens)):
        a, b = int(cu[s]), int(cu[s + 1])
        pos = np.arange(b - a, dtype=np.int32)
        args = w["q"][a:b], pos, w["k"][0, a:b], w["v"][0, a:b], idx[0, a:b]
        O, L = oracle.sparse_attn(*args, op)
        assert_out_close(to_np(out)[a:b], O, "bf16")
        assert np.abs(to_np(lse)[:, a:b].T - L).max() <= prefill_lse_atol("bf16")
        want = oracle.attn_bwd(*args, to_np(dout)[a:b], op)
        got = to_np(grads[0])[a:b], to_np(grads[1])[0, a:b], to_np(grads[2])[0, a:b]
        for name, x, ref in zip(("dq", "dk", "dv"), got, want):
            # the bar of the backward tests: 2e-2 of the gradient's largest value
            assert np.abs(x - ref).max() <= 2e-2 * max(np.abs(ref).max(), 0.1), (name, s)
