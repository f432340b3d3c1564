"""Generic bf16 attention and dQ with rows that pass through LDS: batches large enough for them, lengths around half blocks, blocks and
tiles, every kind of group, lists and dense calls, strided and unaligned rows, and logits that move a column's reference late; against
the CPU oracle."""
import numpy as np
import pytest
import torch

import synth
import test_gpu_generic_groups as groups
from helpers import assert_out_close, to_dev, to_np
from test_gpu_parity import _check_backward, _params, _run_prefill_case, m  # noqa: F401

pytestmark = pytest.mark.gpu

EDGES = [97, 127, 128, 129, 159, 160, 161, 191, 193, 223, 225, 255, 256, 257]


@pytest.mark.parametrize("hq,hkv,d,lens,topk,threshold", [
    (8, 2, 128, EDGES, 3, 0), (8, 2, 64, EDGES, 3, 190), (16, 8, 128, [129, 97, 161, 225, 257], 2, 0),     # four and eight tokens per group
    (9, 3, 128, EDGES[:12], 4, 0), (9, 3, 64, EDGES[:12], 4, 160),                                    # G = 3: five tokens, 15 columns
    (56, 8, 128, [197, 230], 3, 0), (12, 1, 64, EDGES[8:], 3, 0), (16, 1, 64, [300, 257, 500], 3, 0),   # two tokens and one per group
    (8, 8, 128, EDGES[:9] + [511], 3, 0), (8, 8, 64, [1300], 5, 0),                                   # G = 1: 32 tokens per tile
    (8, 2, 128, [1985], 40, 0),                                                                       # walks of up to 62 half blocks
])
def test_lengths_and_groups(m, oracle, hq, hkv, d, lens, topk, threshold):  # noqa: F811
    w = synth.make_varlen(lens, hq, hkv, d, seed=7400 + hq + sum(lens) + d, dtype="bf16")
    gp, op = _params(m, oracle, "bf16", hq, hkv, d, n_init=1, n_local=1, topk_total=topk, dense_threshold=threshold)
    T = sum(lens)
    rows = np.unique(np.concatenate([np.arange(0, T, 11), np.arange(max(0, T - 70), T)]))
    _run_prefill_case(m, oracle, w, gp, op, "bf16", rows=rows)
    _check_backward(m, oracle, w, gp, op, "bf16")
    _check_backward(m, oracle, w, gp, op, "bf16", dense_all=True)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("how", ["heads apart", "tokens apart", "off by one element", "odd token stride"])
def test_strides_and_alignments(m, d, how):  # noqa: F811
    """The same values wherever the rows lie: 16-byte strides take the same kernel, others the one without LDS rows; either way each
    result is within a bf16 rounding of the same sum."""
    hq, hkv, n = 8, 2, 1500
    w = synth.make_prefill(n, hq, hkv, d, seed=7500 + d, dtype="bf16")
    gp = m.Params.make("bf16", hq, hkv, d, n_init=1, n_local=1, topk_total=5)
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    idx = m.sparse_prefill(gp, q, k, v, [0, n])["block_idx"]
    dout = torch.randn(q.shape, generator=torch.Generator().manual_seed(7)).cuda().bfloat16()

    def placed(x):
        if how == "heads apart":
            y = torch.zeros(hkv, n + 24, d, dtype=x.dtype, device="cuda")[:, :n]
        elif how == "tokens apart":
            y = torch.zeros(hkv, n, d + 40, dtype=x.dtype, device="cuda")[:, :, :d]
        elif how == "off by one element":
            y = torch.zeros(hkv * n * d + 1, dtype=x.dtype, device="cuda")[1:].view(hkv, n, d)
        else:
            y = torch.zeros(hkv, n, d + 3, dtype=x.dtype, device="cuda")[:, :, :d]
        return y.copy_(x)

    want, lse = m.sparse_attn_fwd(gp, q, k, v, idx, [0, n])
    want_dq, _, _ = m.sparse_attn_bwd(gp, q, k, v, idx, want, lse, dout, [0, n])
    k2, v2 = placed(k), placed(v)
    out, lse2 = m.sparse_attn_fwd(gp, q, k2, v2, idx, [0, n])
    dq, _, _ = m.sparse_attn_bwd(gp, q, k2, v2, idx, want, lse, dout, [0, n])
    assert_out_close(to_np(out), to_np(want), "bf16", "out")
    assert (lse2 - lse).abs().max() <= 2e-6 * lse.abs().max()             # fp32 sums in another order
    assert (dq.float() - want_dq.float()).norm() <= 2.0 ** -8 * want_dq.float().norm()


@pytest.mark.parametrize("size", [3.0, 40.0, 400.0])
@pytest.mark.parametrize("d", [64, 128])
def test_references_that_move_late(m, d, size):  # noqa: F811
    """Keys whose logits grow along the sequence, from block to block by less and by more than a kept reference may fall behind, up to
    logits of thousands."""
    hq, hkv, n = 8, 2, 1500
    g = torch.Generator().manual_seed(7600 + d)
    q = torch.randn(n, hq, d, generator=g).abs().bfloat16()
    k = (torch.randn(hkv, n, d, generator=g).abs() * torch.linspace(0.1, 1.0, n)[None, :, None] * size).bfloat16()
    v = torch.randn(hkv, n, d, generator=g).bfloat16()
    gp = m.Params.make("bf16", hq, hkv, d, n_init=1, n_local=1, topk_total=4)
    out, lse = m.dense_attn_fwd(gp, q.cuda(), k.cuda(), v.cuda(), [0, n])
    hidden = torch.triu(torch.ones(n, n, dtype=torch.bool), 1)
    for h in range(hq):
        s = q[:, h].double() @ k[h // 4].double().T * gp.softmax_scale
        top = s.abs().masked_fill(hidden, 0).amax(-1)
        s.masked_fill_(hidden, float("-inf"))
        # a logit is a sum of at most 128 exact products in fp32, off by at most 2^-20 of its size here, where all terms are positive
        assert ((lse[h].double().cpu() - torch.logsumexp(s, -1)).abs() <= 2.0 ** -20 * top + 1e-5).all()
        assert_out_close(to_np(out[:, h]), (torch.softmax(s, -1) @ v[h // 4].double()).numpy(), "bf16", f"head {h}")


def test_infinite_rows(m, oracle):  # noqa: F811
    groups.test_infinite_rows_stay_with_the_tokens_that_see_them(m, oracle, "bf16", 1500)


@pytest.mark.parametrize("d,hq,hkv", [(64, 4, 1), (128, 8, 2)])
def test_walks_of_more_than_one_list(m, d, hq, hkv):  # noqa: F811
    """More than 1024 blocks: a tile's list is built again and the wavefronts' buffers start again.  Sampled rows of attention and dQ against float64."""
    n, topk, G = 65536 + 700, 6, hq // hkv
    g = torch.Generator(device="cuda").manual_seed(7700 + d)
    rnd = lambda *shape: torch.randn(*shape, generator=g, device="cuda").bfloat16()
    q, k, v, dout = rnd(n, hq, d), rnd(hkv, n, d), rnd(hkv, n, d), rnd(n, hq, d)
    own = torch.arange(n, device="cuda") // 64
    idx = (torch.rand(hkv, n, topk, generator=g, device="cuda") * (own[None, :, None] + 1)).int()        # anywhere up to the own block
    idx[..., 0] = own.int()
    idx = idx.sort(-1).values
    dup = torch.zeros_like(idx, dtype=torch.bool)
    dup[..., 1:] = idx[..., 1:] == idx[..., :-1]
    idx[dup] = 1 << 20
    idx = idx.sort(-1).values
    idx[idx == 1 << 20] = -1
    gp = m.Params.make("bf16", hq, hkv, d, n_init=0, n_local=1, topk_total=topk)
    for lists in (idx, None):
        if lists is None and d == 128:
            continue                                       # (every block of 66236 tokens: once is enough)
        out, lse = m.sparse_attn_fwd(gp, q, k, v, lists, [0, n]) if lists is not None else m.dense_attn_fwd(gp, q, k, v, [0, n])
        dq = m.sparse_attn_bwd(gp, q, k, v, lists, out, lse, dout, [0, n])[0]
        worst = 0.0
        for t in list(range(65520, 65560)) + list(range(n - 9, n)) + list(range(5, n, 2717)):
            for h in range(hkv):
                if lists is None:
                    keys = torch.arange(t + 1, device="cuda")
                else:
                    have = lists[h, t][lists[h, t] >= 0].long()
                    keys = (have[:, None] * 64 + torch.arange(64, device="cuda")).flatten()
                    keys = keys[keys <= t]
                K, V, s = k[h, keys].double(), v[h, keys].double(), slice(h * G, h * G + G)
                z = q[t, s].double() @ K.t().contiguous() * gp.softmax_scale
                assert (torch.logsumexp(z, 1) - lse[s, t].double()).abs().max() <= 2e-3
                O = torch.softmax(z, 1) @ V
                assert (O - out[t, s].double()).abs().max() <= 2e-2                                   # the forward bar
                dO = dout[t, s].double()
                dz = (z - lse[s, t, None].double()).exp() * (dO @ V.t().contiguous() - (dO * out[t, s].double()).sum(1, keepdim=True))
                want = gp.softmax_scale * dz @ K
                # a bf16 rounding, and fp32 products and sums of terms that cancel
                worst = max(worst, float((want - dq[t, s].double()).abs().max() / max(float(want.abs().max()), 0.1)))
        assert worst <= 2.0 ** -7, worst
