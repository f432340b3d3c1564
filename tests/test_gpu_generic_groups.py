"""The generic attention and gradient kernels with one and two column groups per wavefront: the token counts on both sides of
each rule, tiles that end ragged, groups that do not divide 16, packed and switched sequences, strided rows and infinities in
rows that only some of a tile's tokens see; against the CPU oracle."""
import sys

import numpy as np
import pytest
import torch

import synth
import test_gpu_parity
from helpers import assert_out_close, to_dev, to_np
from test_gpu_parity import _check_backward, _params, _run_prefill_case, m  # noqa: F401

pytestmark = pytest.mark.gpu

# Forms of the calls below, held on the host by test_launch_rules_host.py: dtype, heads, KV heads, d, lengths, blocks, threshold; whether attention and dQ of rows of
# 16-byte multiples pass through LDS; and the generic form, which serves the rest and all rows that lie otherwise: column groups and rows requested ahead of
# attention, the same of dQ.
GENERIC_FORMS = [
    ("bf16", 8, 2, 128, [555], 4, 0, (0, 0), (1, 1, 1, 1)), ("bf16", 8, 2, 128, [565], 4, 0, (0, 0), (1, 1, 2, 1)),
    ("bf16", 8, 2, 128, [755], 4, 0, (0, 1), (1, 1, 2, 1)), ("bf16", 8, 2, 128, [769], 4, 0, (0, 1), (2, 1, 2, 1)),
    ("bf16", 8, 2, 64, [3, 700, 66], 4, 67, (0, 1), (1, 1, 2, 1)), ("bf16", 24, 8, 64, [131, 120], 4, 67, (0, 1), (1, 0, 2, 1)),
    ("bf16", 8, 8, 128, [777], 4, 0, (0, 1), (2, 1, 2, 1)), ("bf16", 40, 8, 128, [400], 4, 0, (1, 1), (2, 0, 2, 1)),
    ("bf16", 40, 8, 64, [801], 4, 0, (1, 1), (2, 0, 2, 1)), ("bf16", 40, 8, 64, [31, 32, 200, 1], 4, 67, (0, 1), (1, 0, 2, 1)),
    ("bf16", 8, 8, 64, [40, 65, 33] * 16, 4, 67, (0, 1), (1, 0, 1, 0)), ("bf16", 48, 4, 128, [101, 17], 4, 67, (0, 0), (1, 0, 1, 0)),
    ("bf16", 40, 8, 128, [96, 33, 5, 64, 65, 130], 4, 67, (0, 0), (1, 0, 1, 0)), ("bf16", 40, 8, 64, [400, 430], 4, 67, (1, 1), (2, 0, 2, 1)),
    ("fp32", 8, 2, 64, [705], 4, 0, (0, 0), (1, 0, 2, 1)), ("fp32", 8, 2, 128, [1195], 4, 0, (0, 0), (1, 0, 1, 1)),
    ("fp32", 8, 2, 128, [1000, 210], 4, 67, (0, 0), (1, 0, 1, 1)), ("fp32", 24, 4, 128, [331], 4, 0, (0, 0), (1, 0, 1, 1)),
    ("fp32", 40, 8, 128, [100, 33, 5], 4, 67, (0, 0), (1, 0, 1, 1)), ("fp32", 40, 8, 64, [130, 31], 4, 67, (0, 0), (1, 0, 2, 1)),
    # rows that are not finite
    ("bf16", 40, 8, 128, [96, 130, 65, 100], 3, 0, (0, 1), (1, 0, 1, 0)), ("bf16", 8, 2, 128, [1100], 3, 0, (0, 1), (2, 1, 2, 1)),
    ("bf16", 8, 2, 128, [400], 3, 0, (0, 0), (1, 1, 1, 1)), ("bf16", 40, 8, 128, [400, 430], 3, 0, (1, 1), (2, 0, 2, 1)),
    ("fp32", 8, 2, 128, [300], 3, 0, (0, 0), (1, 1, 1, 1)), ("fp32", 40, 8, 64, [130, 100, 97], 3, 0, (0, 0), (1, 0, 2, 1)),
    ("bf16", 8, 8, 128, [800], 3, 0, (0, 1), (2, 1, 2, 1)),
]


def _off_by_one(a, dtype):
    """The same values one element behind an aligned place: no row is a 16-byte multiple."""
    x = to_dev(a, dtype)
    return torch.zeros(x.numel() + 1, dtype=x.dtype, device="cuda")[1:].view(x.shape).copy_(x)


@pytest.mark.parametrize("dtype,hq,hkv,d,lens", [
    ("bf16", 8, 2, 128, [555]), ("bf16", 8, 2, 128, [565]), ("bf16", 8, 2, 128, [755]), ("bf16", 8, 2, 128, [769]),
    ("bf16", 8, 2, 64, [3, 700, 66]), ("bf16", 24, 8, 64, [131, 120]),        # G = 3: five tokens per group, 15 columns
    ("bf16", 8, 8, 128, [777]),                                               # G = 1: 32 tokens per tile
    ("fp32", 8, 2, 64, [705]), ("fp32", 8, 2, 128, [1195]), ("fp32", 8, 2, 128, [1000, 210]),
    ("fp32", 24, 4, 128, [331]),                                              # G = 6: two tokens per group, 12 columns
    ("bf16", 48, 4, 128, [101, 17]),                                          # G = 12: one token per group
    # many workgroups, rows not requested ahead: one group and two; walks that end in the first half of a block
    ("bf16", 40, 8, 128, [96, 33, 5, 64, 65, 130]), ("bf16", 40, 8, 64, [31, 32, 200, 1]), ("bf16", 40, 8, 128, [400]),
    ("bf16", 40, 8, 64, [801]), ("fp32", 40, 8, 128, [100, 33, 5]), ("fp32", 40, 8, 64, [130, 31]),
    # (no sequence of 3 tokens among these: Delta = <dO, O> of a bf16 O is off by 2^-9 |O| sqrt(64 / 3) = 0.006, dQ by scale |K|
    # times that = 6e-4, and with three tokens the largest dQ is 0.3: 2e-3 of it on average, as much as the comparison allows)
    ("bf16", 8, 8, 64, [40, 65, 33] * 16),
])
def test_both_sides_of_the_rules(m, oracle, dtype, hq, hkv, d, lens):  # noqa: F811
    w = synth.make_varlen(lens, hq, hkv, d, seed=2800 + sum(lens) + d, dtype=dtype)
    gp, op = _params(m, oracle, dtype, hq, hkv, d, n_init=1, n_local=1, topk_total=4, dense_threshold=67 if len(lens) > 1 else 0)
    T = sum(lens)
    rows = np.unique(np.concatenate([np.arange(0, T, 7), np.arange(max(0, T - 70), T)]))
    _run_prefill_case(m, oracle, w, gp, op, dtype, rows=rows)
    _check_backward(m, oracle, w, gp, op, dtype)


@pytest.mark.parametrize("dtype,n", [("bf16", 400), ("bf16", 1100), ("fp32", 1300)])
def test_infinite_rows_stay_with_the_tokens_that_see_them(m, oracle, dtype, n):  # noqa: F811
    """A V row of infinities in the second half of a block: the tokens before it in the same block are computed again without
    it, and give what they give when the row is finite."""
    hq, hkv, d = 8, 2, 128
    w = synth.make_prefill(n, hq, hkv, d, seed=2900 + n, dtype=dtype)
    gp, op = _params(m, oracle, dtype, hq, hkv, d, n_init=1, n_local=1, topk_total=3)
    q, k, v = (to_dev(w[x], dtype) for x in ("q", "k", "v"))
    idx = m.sparse_prefill(gp, q, k, v, [0, n])["block_idx"]
    clean, _ = m.sparse_attn_fwd(gp, q, k, v, idx, [0, n])
    hit = 64 * (n // 128) + 41
    v[:, hit] = float("inf")
    out, lse = m.sparse_attn_fwd(gp, q, k, v, idx, [0, n])
    idx_h = to_np(idx)
    for h in range(hkv):
        sees = np.array([t >= hit and hit // 64 in idx_h[h, t] for t in range(n)])
        o, c = to_np(out)[:, 4 * h:4 * h + 4], to_np(clean)[:, 4 * h:4 * h + 4]
        assert not np.isfinite(o[sees]).any() and sees.any()
        assert_out_close(o[~sees], c[~sees], dtype, "tokens that do not see the row")
    assert torch.isfinite(lse).all()


# (which form each takes, also of the tests below: GENERIC_FORMS)
@pytest.mark.parametrize("dtype,hq,hkv,d,lens", [
    ("bf16", 40, 8, 128, [96, 130, 65, 100]), ("bf16", 8, 2, 128, [1100]), ("bf16", 8, 2, 128, [400]), ("bf16", 40, 8, 128, [400, 430]),
    ("fp32", 8, 2, 128, [300]), ("fp32", 40, 8, 64, [130, 100, 97]), ("bf16", 8, 8, 128, [800]),
])
@pytest.mark.parametrize("bad", ["nan", "inf", "one inf"])
def test_key_rows_that_are_not_finite(m, oracle, dtype, hq, hkv, d, lens, bad):  # noqa: F811
    """A K row of NaN, of infinities or with one infinity, in the second half of a block: tokens that do not see it, in the same
    tiles as tokens that do, keep output, log-sum-exp and dQ."""
    T, G = sum(lens), hq // hkv
    w = synth.make_varlen(lens, hq, hkv, d, seed=2970 + T, dtype=dtype)
    gp, _ = _params(m, oracle, dtype, hq, hkv, d, n_init=1, n_local=1, topk_total=3)
    q, k, v = (to_dev(w[x], dtype) for x in ("q", "k", "v"))
    cu = w["cu_seqlens"]
    idx = m.sparse_prefill(gp, q, k, v, cu)["block_idx"]
    clean, lse = m.sparse_attn_fwd(gp, q, k, v, idx, cu)
    torch.manual_seed(T)
    dout = torch.randn_like(q)
    want = m.sparse_attn_bwd(gp, q, k, v, idx, clean, lse, dout, cu)[0]
    sees = torch.zeros(hkv, T, dtype=torch.bool, device="cuda")
    for a, n in zip(cu[:-1].tolist(), lens):
        hit = min(64 * (n // 128) + 41, n - 2)
        k[:, a + hit] = float("nan") if bad == "nan" else k[:, a + hit]
        if bad == "inf":
            k[:, a + hit] = float("inf")
        if bad == "one inf":
            k[:, a + hit, 5] = float("inf")
        sees[:, a + hit:a + n] = (idx[:, a + hit:a + n] == hit // 64).any(-1)
    assert sees.any() and not sees.all()
    out, lse2 = m.sparse_attn_fwd(gp, q, k, v, idx, cu)
    got = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse2, dout, cu)[0]
    for h in range(hkv):
        heads, rest = slice(h * G, h * G + G), ~sees[h]
        if bad == "nan":
            assert not torch.isfinite(out[sees[h], heads]).any()
        assert_out_close(to_np(out[rest, heads]), to_np(clean[rest, heads]), dtype, "out")
        assert (lse2[heads][:, rest] - lse[heads][:, rest]).abs().max() <= 1e-5
        # the same sums in another order, of another (rounded) output: a rounding of dQ
        scale = max(float(want.float().abs().max()), 0.1)
        assert (got[rest, heads].float() - want[rest, heads].float()).abs().max() <= (2.0**-7 if dtype == "bf16" else 1e-5) * scale


@pytest.mark.parametrize("hq,hkv,d,lens", [(40, 8, 128, [400]), (40, 8, 64, [801]), (40, 8, 64, [400, 430]), (8, 2, 128, [769]), (8, 2, 64, [3, 700, 66]),
                                           (24, 8, 64, [131, 120]), (8, 8, 128, [777]), (8, 8, 64, [40, 65, 33] * 16)])
def test_both_sides_of_the_rules_unaligned(m, oracle, monkeypatch, hq, hkv, d, lens):  # noqa: F811
    """The generic two-group forms, and those whose aligned calls pass their rows through LDS."""
    monkeypatch.setattr(test_gpu_parity, "to_dev", _off_by_one)
    test_both_sides_of_the_rules(m, oracle, "bf16", hq, hkv, d, lens)


@pytest.mark.parametrize("hq,hkv,d,lens", [(40, 8, 128, [96, 130, 65, 100]), (8, 2, 128, [1100]), (40, 8, 128, [400, 430]), (8, 8, 128, [800])])
@pytest.mark.parametrize("bad", ["nan", "inf", "one inf"])
def test_key_rows_that_are_not_finite_unaligned(m, oracle, monkeypatch, hq, hkv, d, lens, bad):  # noqa: F811
    aligned = to_dev
    monkeypatch.setattr(sys.modules[__name__], "to_dev", lambda a, dtype: torch.zeros(aligned(a, dtype).numel() + 1, dtype=torch.bfloat16, device="cuda")[1:].view(
        a.shape).copy_(aligned(a, dtype)))
    test_key_rows_that_are_not_finite(m, oracle, "bf16", hq, hkv, d, lens, bad)


def test_strided_rows(m, oracle):  # noqa: F811
    """Rows 192 elements apart, and 2^25 elements apart (64-bit row distances), against rows side by side."""
    n, hq, hkv, d = 780, 8, 2, 128
    w = synth.make_prefill(n, hq, hkv, d, seed=2950, dtype="bf16")
    gp, _ = _params(m, oracle, "bf16", hq, hkv, d, n_init=1, n_local=1, topk_total=4)
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    idx = m.sparse_prefill(gp, q, k, v, [0, n])["block_idx"]
    out, lse = m.sparse_attn_fwd(gp, q, k, v, idx, [0, n])
    dout = torch.flip(out, (0,)).contiguous()
    want = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, [0, n])
    for stride in (192, 1 << 25):
        buf = torch.empty(n * stride + 2048 if stride > 1000 else 0, dtype=torch.bfloat16, device="cuda")     # (only the rows are touched)
        ks, vs = (torch.as_strided(buf, (hkv, n, d), (d if stride > 1000 else n * stride, stride, 1), o) for o in (0, 1024)) \
            if stride > 1000 else (torch.zeros(hkv, n, stride, dtype=torch.bfloat16, device="cuda")[:, :, :d] for _ in range(2))
        ks.copy_(k)
        vs.copy_(v)
        o2, l2 = m.sparse_attn_fwd(gp, q, ks, vs, idx, [0, n])
        assert torch.equal(out, o2) and torch.equal(lse, l2)
        got = m.sparse_attn_bwd(gp, q, ks, vs, idx, out, lse, dout, [0, n])
        assert torch.equal(got[0], want[0])
        for x, y in zip(got[1:], want[1:]):
            # (the order of the float adds differs from run to run)
            assert (x - y).abs().max() <= 2e-5 * float(y.abs().max())
        del buf, ks, vs
        torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype,hq,hkv,d,lens", [
    ("bf16", 8, 2, 128, [33]), ("bf16", 8, 2, 128, [31, 300, 32, 1]), ("fp32", 8, 2, 128, [289]), ("bf16", 8, 2, 64, [97, 160]),
    ("fp32", 8, 2, 64, [350]), ("bf16", 8, 8, 128, [500]), ("bf16", 16, 16, 128, [700, 65]),
    ("bf16", 40, 8, 64, [64, 130, 65] * 8), ("bf16", 16, 8, 64, [129, 63, 64] * 9),       # one group of 16 rows per step
])
def test_token_chunks_of_dkv(m, oracle, dtype, hq, hkv, d, lens):  # noqa: F811
    """Chunks from 32 to 256 tokens, with ends inside and at the edge of a chunk."""
    w = synth.make_varlen(lens, hq, hkv, d, seed=2950 + sum(lens) + d, dtype=dtype)
    gp, op = _params(m, oracle, dtype, hq, hkv, d, n_init=1, n_local=1, topk_total=4)
    _check_backward(m, oracle, w, gp, op, dtype)
