"""Selection bitmap from lists longer than a wavefront (65 and more entries), ragged ends, dense sequences in between, and
gradients cleared by the call itself: the same as without the bitmap, into buffers full of NaN."""
import pytest
import torch

import synth
from helpers import to_dev
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,topk,threshold", [([4700], 70, 0), ([5000, 31, 4400], 65, 0), ([300, 4800, 257], 130, 280), ([33], 66, 0),
                                                 ([17, 70, 64, 200] * 50, 16, 65)])       # sequences looked for 64 at a time
def test_long_lists(m, oracle, lens, topk, threshold):  # noqa: F811
    w = synth.make_varlen(lens, 32, 2, 128, seed=2700 + topk, dtype="bf16")
    gp, _ = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=2, topk_total=topk, dense_threshold=threshold)
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    r = m.sparse_prefill(gp, q, k, v, w["cu_seqlens"])
    torch.manual_seed(topk)
    dout = torch.randn_like(q)
    got = []
    for most in (512 << 20, 0):
        dk, dv = (torch.full((2, sum(lens), 128), float("nan"), device="cuda") for _ in range(2))
        got.append(m.sparse_attn_bwd(gp, q, k, v, r["block_idx"], r["out"], r["lse"], dout, w["cu_seqlens"], dk=dk, dv=dv,
                                     sel_bitmap_max_bytes=most))
    for x, y in zip(*got):
        assert torch.isfinite(x).all()
        # (the order of the float adds of dK and dV differs from run to run)
        assert (x.float() - y.float()).abs().max() <= 2e-5 * max(float(y.float().abs().max()), 0.1)


def test_many_sequences_beside_a_long_one(m, oracle):  # noqa: F811
    """60000 sequences of one token beside one of 100000: the token chunks of the dK/dV launch, which every sequence gets as the
    longest needs them, have to be long ones for its thread count to stay under the limit.  Every token selects its own block."""
    hq, hkv, n, ones = 128, 8, 100000, 60000
    gp, _ = _params(m, oracle, "bf16", hq, hkv, 128, n_init=1, n_local=1, topk_total=2)
    torch.manual_seed(5)
    rows = n + ones
    q, dout = (torch.randn(rows, hq, 128, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    k, v = (torch.randn(hkv, rows, 128, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    si = m.SeqInfo([0, n] + list(range(n + 1, rows + 1)))
    idx = torch.full((hkv, rows, 2), -1, dtype=torch.int32, device="cuda")
    idx[:, :n, 0] = (torch.arange(n, device="cuda") // 64).int()
    idx[:, n:, 0] = 0
    out, lse = m.sparse_attn_fwd(gp, q, k, v, idx, si)
    _, dk, dv = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, si, sel_bitmap_max_bytes=0)
    # one key: P = 1, so dV is the group's sum of dO (sixteen fp32 adds; P and dO of |dO| < 6 as bf16) and dZ = 0 up to rounding
    want = dout[n:].float().view(ones, hkv, 16, 128).sum(2).transpose(0, 1)
    assert (dv[:, n:] - want).abs().max() <= 16 * 6 * 2.0**-9
    assert dk[:, n:].abs().max() <= 16 * 6 * 2.0**-9
    # the long sequence's last block: 32 tokens that attend to nothing else
    s = slice(n - n % 64, n)
    rq, rk, rv = q[s].float(), k[:, s].float().requires_grad_(), v[:, s].float().requires_grad_()
    c = n % 64
    z = torch.stack([rq.view(c, hkv, 16, 128)[:, h].reshape(c * 16, 128) @ rk[h].T for h in range(hkv)]) / 128**0.5
    seen = torch.arange(c, device="cuda")[None, :] <= torch.arange(c, device="cuda").repeat_interleave(16)[:, None]
    p = z.masked_fill(~seen, float("-inf")).softmax(-1)
    o = torch.stack([p[h] @ rv[h] for h in range(hkv)]).view(hkv, c, 16, 128).transpose(0, 1).reshape(c, hq, 128)
    (o * dout[s].float()).sum().backward()
    for got, ref in ((dk[:, s], rk.grad), (dv[:, s], rv.grad)):
        assert (got - ref).abs().max() <= 0.02 * ref.abs().max()      # bf16 probabilities and dZ, as the other tests
