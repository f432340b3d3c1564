"""Decode steps whose attend workgroups take several blocks per wavefront, and whose rows are pooled where they are picked from: batches
around the lines between the forms, budgets that leave the last round incomplete, dense sequences with more blocks than a
workgroup takes; against the CPU oracle, and the forms against each other."""
import numpy as np
import pytest
import torch

import synth
from helpers import assert_out_close, to_np
from test_gpu_parity import _check_decode, _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


# pairs x ceil(entries / 8) against 256 decides between one block and several; 256 / pairs workgroups for each pair then
@pytest.mark.parametrize("batch,topk,n_local,threshold", [(18, 64, 8, 0), (19, 64, 8, 0), (20, 33, 1, 0), (40, 96, 32, 0), (43, 64, 8, 5200),
                                                          (64, 26, 2, 0), (129, 64, 8, 0)])
def test_rounds(m, oracle, batch, topk, n_local, threshold):  # noqa: F811
    top = 5300 if batch < 100 else 4400
    ctx = [1 + (7919 * i + 5111) % top for i in range(batch - 1)] + [top]
    w = synth.make_decode(ctx, 32, 2, 128, seed=90 + batch, dtype="bf16", max_len=top)
    gp, op = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=n_local, topk_total=topk, dense_threshold=threshold)
    assert _check_decode(m, oracle, w, ctx, gp, op, "bf16") > 0


@pytest.mark.parametrize("n", [16415, 16416])              # 1024 and 1025 compressed keys
@pytest.mark.parametrize("batch", [1, 3])
def test_rows_pooled_by_the_attend_workgroups(m, oracle, n, batch):  # noqa: F811
    ctx = [n - 1311 * i for i in range(batch)]
    w = synth.make_decode(ctx, 16, 1, 128, seed=n + batch, dtype="bf16", max_len=n)
    for kw in (dict(), dict(pool_pad=1)):
        gp, op = _params(m, oracle, "bf16", 16, 1, 128, n_init=1, n_local=8, topk_total=64, **kw)
        assert _check_decode(m, oracle, w, ctx, gp, op, "bf16") > 0


def test_forms_agree(m):  # noqa: F811
    """520 pairs (pooled by a kernel in front) and the same sequences in calls of 130 and 10 (pooled by the selection kernel, by the
    attend workgroups): the same lists, and outputs that differ by the order of their sums only."""
    B, n = 260, 4200
    torch.manual_seed(7)
    q, k = torch.randn(B, 32, 128).cuda().bfloat16(), torch.randn(B, 2, n, 128, device="cuda").bfloat16()
    v = torch.randn(B, 2, n, 128, device="cuda").bfloat16()
    ctx = [int(x) for x in np.random.default_rng(3).integers(300, n + 1, B)]
    gp = m.Params.make("bf16", 32, 2, 128, n_init=1, n_local=4, topk_total=32)
    kc = torch.zeros((B, 2, m.num_cmp(gp, n), 128), device="cuda")
    m.compress_k_append(gp, k, kc, [0] * B, ctx)
    want = m.sparse_decode(gp, q, k, v, kc, ctx)
    for part in (130, 10):
        for b in range(0, B, part):
            s = slice(b, b + part)
            out, lse, idx = m.sparse_decode(gp, q[s], k[s], v[s], kc[s], ctx[s])
            assert torch.equal(idx, want[2][s])
            assert_out_close(to_np(out), to_np(want[0][s]), "bf16")
            assert (lse - want[1][s]).abs().max() < 1e-5           # (see test_gpu_decode_splits.py)


def test_rounds_of_dense_sequences(m):  # noqa: F811
    """400 pairs, one workgroup each by their number, with dense sequences of 65 to 67 blocks: more than sixteen rounds of four wavefronts hold, so that
    the limit decides; against calls of 10 sequences, where every wavefront takes one block."""
    B, n = 200, 4400
    torch.manual_seed(9)
    q, k = torch.randn(B, 32, 128).cuda().bfloat16(), torch.randn(B, 2, n, 128, device="cuda").bfloat16()
    v = torch.randn(B, 2, n, 128, device="cuda").bfloat16()
    ctx = [int(x) for x in np.random.default_rng(4).integers(4100, n + 1, B)]
    gp = m.Params.make("bf16", 32, 2, 128, n_init=1, n_local=4, topk_total=32, dense_threshold=4270)
    kc = torch.zeros((B, 2, m.num_cmp(gp, n), 128), device="cuda")
    m.compress_k_append(gp, k, kc, [0] * B, ctx)
    want = m.sparse_decode(gp, q, k, v, kc, ctx)
    for b in range(0, B, 10):
        s = slice(b, b + 10)
        out, lse, idx = m.sparse_decode(gp, q[s], k[s], v[s], kc[s], ctx[s])
        assert torch.equal(idx, want[2][s])
        assert_out_close(to_np(out), to_np(want[0][s]), "bf16")
        assert (lse - want[1][s]).abs().max() < 1e-5


def test_lists_do_not_depend_on_the_batch(m):  # noqa: F811
    """Rows of up to 20 chunk partials, pooled by a kernel of their own (520 and 20 pairs), by the selection kernel (260) and by the attend
    workgroups (200 and 120 pairs): the normaliser and the sums are added in one order, so the lists are the same."""
    B, n = 260, 40000
    torch.manual_seed(11)
    q, k = torch.randn(B, 32, 128).cuda().bfloat16(), torch.empty(B, 2, n, 128, device="cuda", dtype=torch.bfloat16).normal_()
    ctx = [int(x) for x in np.random.default_rng(5).integers(20000, n + 1, B)]
    gp = m.Params.make("bf16", 32, 2, 128, n_init=1, n_local=8, topk_total=16)
    kc = torch.zeros((B, 2, m.num_cmp(gp, n), 128), device="cuda")
    m.compress_k_append(gp, k, kc, [0] * B, ctx)
    want = m.sparse_decode(gp, q, k, k, kc, ctx)[2]
    for part in (130, 100, 10):
        for b in range(0, B, part):
            s = slice(b, b + part)
            assert torch.equal(m.sparse_decode(gp, q[s], k[s], k[s], kc[s], ctx[s])[2], want[s]), (part, b)
