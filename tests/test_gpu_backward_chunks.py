"""The matrix-core backward at sizes that take each length of the dK / dV kernel's token chunks (32 .. 512 tokens; 1024 in
the full-size test), with list lengths of both parities and a ragged end, and each tile of the dQ kernel (4, 8, 16 tokens;
one list entry per interval), against the CPU oracle through the C ABI."""
import numpy as np
import pytest
import torch

import synth
from helpers import to_dev, to_np
from test_gpu_parity import _check_backward, _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1, 2, 66, 191], [1024], [1025], [1999], [3333], [4601], [6400], [9001], [12001]])
def test_token_chunks_of_the_dkv_kernel(m, oracle, lens):  # noqa: F811
    w = synth.make_varlen(lens, 16, 1, 128, seed=700 + len(lens), dtype="bf16")
    gp, op = _params(m, oracle, "bf16", 16, 1, 128, n_init=1, n_local=1, topk_total=3)
    _check_backward(m, oracle, w, gp, op, "bf16")
    if lens[0] in (1024, 3333):
        _check_backward(m, oracle, w, gp, op, "bf16", sel_bitmap_max_bytes=0)


def test_dq_with_one_entry_per_interval(m, oracle):  # noqa: F811
    """A union list too long for two entries per interval (136 blocks, more than 2046 blocks): dQ of sampled rows for given
    random lists.  Bar as in the backward tests: 2e-2 of the gradient's largest value."""
    n, K = 131136, 136
    w = synth.make_prefill(n, 16, 1, 128, seed=790, dtype="bf16")
    gp, op = _params(m, oracle, "bf16", 16, 1, 128, n_init=1, n_local=1, topk_total=K)
    rng = np.random.default_rng(791)
    idx = np.full((1, n, K), -1, np.int32)
    bt = np.arange(n) // 64
    # ascending distinct blocks: a random start and random gaps, the token's own block last
    step = np.maximum(bt // K, 1)
    body = np.minimum(rng.integers(0, step)[:, None] + step[:, None] * np.arange(K - 1)[None], bt[:, None])
    idx[0, :, :K - 1] = np.where(body < bt[:, None], body, -1)
    cnt = (idx[0] >= 0).sum(1)
    idx[0, np.arange(n), cnt] = bt
    q, k, v, idx_d = to_dev(w["q"], "bf16"), to_dev(w["k"], "bf16"), to_dev(w["v"], "bf16"), torch.from_numpy(idx).cuda()
    dout = torch.randn(q.shape, generator=torch.Generator("cuda").manual_seed(5), device="cuda").bfloat16()
    out, lse = m.sparse_attn_fwd(gp, q, k, v, idx_d, [0, n])
    dq, _, _ = m.sparse_attn_bwd(gp, q, k, v, idx_d, out, lse, dout, [0, n])
    rows = np.unique(np.concatenate([rng.integers(0, n, 40), np.arange(n - 20, n), np.arange(0, 130, 13)]))
    rows_d = torch.from_numpy(rows).cuda()
    dQ, _, _ = oracle.attn_bwd(w["q"][rows], rows.astype(np.int32), w["k"][0], w["v"][0], idx[0, rows], to_np(dout[rows_d]), op)
    assert np.abs(to_np(dq[rows_d]) - dQ).max() <= 2e-2 * max(np.abs(dQ).max(), 0.1)


@pytest.mark.parametrize("heads", [(16, 1), (32, 2)])
def test_more_sequences_than_xcds(m, oracle, heads):  # noqa: F811
    """Eleven sequences: the (chunk, head) groups move on by one of the eight XCDs with every sequence."""
    lens = [70, 129, 1, 64, 200, 33, 65, 130, 40, 300, 90]
    w = synth.make_varlen(lens, *heads, 128, seed=730, dtype="bf16")
    gp, op = _params(m, oracle, "bf16", *heads, 128, n_init=1, n_local=1, topk_total=3, dense_threshold=80)
    _check_backward(m, oracle, w, gp, op, "bf16")


@pytest.mark.parametrize("dense", [True, False])
def test_token_strides_past_32_bits_per_block(m, oracle, dense):  # noqa: F811
    """K and V rows 2^24 elements apart (a block then spans 2^31 bytes), a partial last block: the same gradients as from
    contiguous rows, up to the order of fp32 additions and, in dQ, one step of its bf16 rounding."""
    n, S = 333, 1 << 24
    w = synth.make_prefill(n, 32, 2, 128, seed=720, dtype="bf16")
    gp, _ = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=1, topk_total=3)
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    buf = torch.empty(n * S, dtype=torch.bfloat16, device="cuda")
    kw, vw = (buf.as_strided(k.shape, (128, S, 1), at).copy_(x) for x, at in ((k, 0), (v, 4096)))
    idx = None if dense else m.sparse_prefill(gp, q, k, v, [0, n])["block_idx"]
    out, lse = m.dense_attn_fwd(gp, q, k, v, [0, n]) if dense else m.sparse_attn_fwd(gp, q, k, v, idx, [0, n])
    dout = torch.randn(q.shape, generator=torch.Generator("cuda").manual_seed(5), device="cuda").bfloat16()
    want = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, [0, n])
    got = m.sparse_attn_bwd(gp, q, kw, vw, idx, out, lse, dout, [0, n])
    for name, a, b, rtol in zip(("dq", "dk", "dv"), got, want, (2.0 ** -7, 0.0, 0.0)):
        a, b = to_np(a), to_np(b)
        assert (np.abs(a - b) <= rtol * np.abs(b) + 1e-5 * np.abs(b).max()).all(), name
