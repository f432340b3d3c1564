"""Prompts short enough for the smaller tiles of the matrix-core kernels: 4- and 8-token attention tiles, score tiles with one
and two tokens per wavefront, at their first and last lengths, ragged, packed and switched, against the CPU oracle."""
import numpy as np
import pytest

import synth
from helpers import assert_out_close, to_dev, to_np
from test_gpu_parity import _check_backward, _params, _run_prefill_case, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,threshold", [([511], 0), ([512], 0), ([513], 0), ([1021], 0), ([1024], 0), ([1025], 0), ([2048], 0),
                                            ([2049], 0),
                                            ([3, 130, 1, 250], 100), ([65, 301, 70, 480], 128)])
def test_small_tiles(m, oracle, lens, threshold):  # noqa: F811
    w = synth.make_varlen(lens, 32, 2, 128, seed=1200 + len(lens) + lens[0], dtype="bf16")
    rows = np.arange(sum(lens)) if sum(lens) < 1200 else np.unique(np.concatenate([np.arange(0, sum(lens), 7), np.arange(sum(lens) - 70, sum(lens))]))
    for kw in (dict(), dict(lse_mode=1, pool_pad=1)):
        gp, op = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=1, topk_total=4, dense_threshold=threshold, **kw)
        _run_prefill_case(m, oracle, w, gp, op, "bf16", rows=rows)
        _run_prefill_case(m, oracle, w, gp, op, "bf16", rows=rows, fused_pool=True)
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    out, _ = m.dense_attn_fwd(gp, q, k, v, w["cu_seqlens"])
    a, b = int(w["cu_seqlens"][-2]), int(w["cu_seqlens"][-1])
    pos = np.unique(np.concatenate([np.arange(0, b - a, 13), [b - a - 1]])).astype(np.int32)
    O, _ = oracle.dense_attn(w["q"][a + pos, :16], pos, w["k"][0, a:b], w["v"][0, a:b], op)
    assert_out_close(to_np(out)[a + pos, :16], O, "bf16", "dense")


@pytest.mark.parametrize("n,topk", [(1009, 32), (1024, 12), (2039, 20), (2048, 40)])
def test_union_lists_long_enough_to_be_paired(m, oracle, n, topk):  # noqa: F811
    """One KV head, where the small tiles reach 1024 (4 tokens) and 2048 (8): a wavefront then has at least four list entries
    to pair.  Budgets that every token shares in full, and that neighbouring tokens fill differently."""
    w = synth.make_prefill(n, 16, 1, 128, seed=1300 + n, dtype="bf16")
    gp, op = _params(m, oracle, "bf16", 16, 1, 128, n_init=1, n_local=2, topk_total=topk)
    _run_prefill_case(m, oracle, w, gp, op, "bf16")
    _check_backward(m, oracle, w, gp, op, "bf16")
