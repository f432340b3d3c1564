"""Attention of short prompts (four-token tiles, one or two wavefronts per token, all blocks walked or the lists' union): lengths
around its tiles, blocks and rules, ragged and packed batches, odd strides of K and V, lists with and without the own block, rows
that are not finite, against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth
from helpers import assert_out_close, to_dev, to_np
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


def _lists(rng, lens, hkv, topk, drop_own=False):
    """Ascending random block lists, -1 padded; every block where the budget allows."""
    idx = np.full((hkv, sum(lens), topk), -1, np.int32)
    t0 = 0
    for n in lens:
        for t in range(n):
            own = t // 64
            for h in range(hkv):
                have = np.arange(own + (0 if drop_own and own > 0 else 1))
                if len(have) > topk:
                    have = np.sort(rng.choice(have, topk, replace=False))
                idx[h, t0 + t, :len(have)] = have
        t0 += n
    return idx


def _check(m, oracle, w, gp, op, idx, lens, hkv, q, k, v):  # noqa: F811
    cu = w["cu_seqlens"]
    if idx is None:
        out, lse = m.dense_attn_fwd(gp, q, k, v, cu)
    else:
        out, lse = m.sparse_attn_fwd(gp, q, k, v, torch.from_numpy(idx).cuda(), cu)
    out, lse = to_np(out), to_np(lse)
    for s, n in enumerate(lens):
        a, b = int(cu[s]), int(cu[s + 1])
        pos = np.arange(n, dtype=np.int32)
        for h in range(hkv):
            Q = w["q"][a:b, 16 * h:16 * h + 16]
            if idx is None or n < gp.dense_threshold:
                O, L = oracle.dense_attn(Q, pos, w["k"][h, a:b], w["v"][h, a:b], op)
            else:
                O, L = oracle.sparse_attn(Q, pos, w["k"][h, a:b], w["v"][h, a:b], idx[h, a:b], op)
            assert_out_close(out[a:b, 16 * h:16 * h + 16], O, "bf16", f"sequence {s} head {h}")
            assert np.abs(lse[16 * h:16 * h + 16, a:b].T - L).max() <= 2e-3     # the forward bar of the log-sum-exp


# (W = workgroups of the call: 1 and 2 wavefronts per token lie on either side of 256, 400 and 512, the tile kernel behind)
@pytest.mark.parametrize("lens,hkv,topk,threshold", [
    ([1], 1, 8, 0), ([3], 2, 8, 0), ([5], 1, 1, 0), ([63], 2, 8, 0), ([64], 1, 8, 0), ([65], 2, 2, 0), ([130], 2, 1, 0),
    ([512], 2, 8, 0), ([516], 2, 4, 0), ([257], 4, 3, 0), ([600], 1, 10, 0), ([640], 2, 12, 0), ([777], 2, 5, 0), ([1025], 1, 20, 0),
    ([65, 1, 200, 64], 2, 3, 0), ([7] * 70, 2, 4, 0), ([300, 20, 333], 4, 4, 100), ([600, 129], 4, 12, 0), ([1000, 3], 2, 16, 0)])
def test_lengths_and_lists(m, oracle, lens, hkv, topk, threshold):  # noqa: F811
    w = synth.make_varlen(lens, 16 * hkv, hkv, 128, seed=4100 + sum(lens), dtype="bf16")
    gp, op = _params(m, oracle, "bf16", 16 * hkv, hkv, 128, n_init=0, n_local=1, topk_total=topk, dense_threshold=threshold)
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    rng = np.random.default_rng(sum(lens) + topk)
    for drop_own in (False, True):
        idx = _lists(rng, lens, hkv, topk, drop_own)
        _check(m, oracle, w, gp, op, idx, lens, hkv, q, k, v)
    _check(m, oracle, w, gp, op, None, lens, hkv, q, k, v)
    # K and V with gaps between tokens and heads
    wide = lambda x: torch.nn.functional.pad(x, (0, 8, 0, 3))[:, :x.shape[1], :128]
    _check(m, oracle, w, gp, op, idx, lens, hkv, q, wide(k), wide(v))


@pytest.mark.parametrize("n", [130, 640])
def test_rows_that_are_not_finite(m, n):  # noqa: F811
    """An infinite V row, or a K row of minus infinity, of the last token: what it does not reach stays as it is, also the
    tokens of the same block (they do not see it, and the rows past the end repeat it)."""
    torch.manual_seed(n)
    q, k, v = torch.randn(n, 32, 128).abs().cuda().bfloat16(), torch.randn(2, n, 128).cuda().bfloat16(), torch.randn(2, n, 128).cuda().bfloat16()
    gp = m.Params.make("bf16", 32, 2, 128)
    want, lse = m.dense_attn_fwd(gp, q, k, v, [0, n])
    v2 = v.clone()
    v2[0, n - 1] = float("inf")
    out, lse2 = m.dense_attn_fwd(gp, q, k, v2, [0, n])
    assert torch.equal(out[:n - 1], want[:n - 1]) and torch.equal(out[:, 16:], want[:, 16:]) and torch.equal(lse, lse2)
    assert torch.isinf(out[n - 1, :16]).all()
    k2 = k.clone()
    k2[0, 32:64] = float("-inf")                                  # half a block whose logits are all minus infinity
    out, lse2 = m.dense_attn_fwd(gp, q, k2, v, [0, n])
    keep = torch.cat([k[:1, :32], k[:1, 64:]], 1).float(), torch.cat([v[:1, :32], v[:1, 64:]], 1).float()
    z = (q[n - 1, :16].float() @ keep[0][0].t().contiguous()) * 128 ** -0.5
    assert (torch.softmax(z, 1) @ keep[1][0] - out[n - 1, :16].float()).abs().max() <= 2e-2      # the forward bar
    assert (torch.logsumexp(z, 1) - lse2[:16, n - 1]).abs().max() <= 2e-3


@pytest.mark.parametrize("hkv,n", [(1, 40), (2, 130), (4, 300), (2, 777), (2, 1500)])
def test_logits_that_are_all_minus_infinity(m, hkv, n):  # noqa: F811
    """A token that sees nothing but logits of minus infinity has no mean, NaN; one whose list is empty has nothing, 0 and minus infinity.
    (One and two wavefronts per token, and the tile kernel.)"""
    torch.manual_seed(n)
    q, v = torch.randn(n, 16 * hkv, 128).abs().cuda().bfloat16(), torch.randn(hkv, n, 128).cuda().bfloat16()
    k = torch.randn(hkv, n, 128).cuda().bfloat16()
    gp = m.Params.make("bf16", 16 * hkv, hkv, 128, n_init=0, n_local=1, topk_total=2)
    k[:, :min(n, 64)] = float("-inf")
    idx = torch.full((hkv, n, 2), -1, dtype=torch.int32, device="cuda")
    idx[:, :, 0] = 0                                              # block 0 alone: minus infinity throughout
    idx[:, n // 2:, 0] = -1                                       # nothing
    out, lse = m.sparse_attn_fwd(gp, q, k, v, idx, [0, n])
    assert out[:n // 2].isnan().all() and lse[:, :n // 2].isnan().all()
    assert (out[n // 2:] == 0).all() and (lse[:, n // 2:] == float("-inf")).all()
    out, lse = m.dense_attn_fwd(gp, q, k, v, [0, n])
    assert out[:min(n, 64)].isnan().all() and lse[:, :min(n, 64)].isnan().all()
    if n <= 777:                                                  # (the tile kernel's tokens meet block 0 first and keep its NaN)
        assert out[64:].isfinite().all() and lse[:, 64:].isfinite().all()
