"""Selection bitmap from lists longer than a wavefront (65 and more entries), ragged ends, dense sequences in between, and
gradients cleared by the call itself: the same as without the bitmap, into buffers full of NaN."""
import pytest
import torch

import synth
from helpers import to_dev
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,topk,threshold", [([4700], 70, 0), ([5000, 31, 4400], 65, 0), ([300, 4800, 257], 130, 280), ([33], 66, 0)])
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
