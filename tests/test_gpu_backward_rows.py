"""dK and dV of bf16 rows in the generic backward (32 rows per step) and the numbering of its workgroups: lengths around steps, blocks
and chunks, every kind of group, packed and switched batches, lists and dense calls, against the CPU oracle."""
import pytest
import torch

import synth
from helpers import to_dev
from test_gpu_parity import _check_backward, _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (8, 2, 64), (1, 1, 128), (3, 1, 64), (10, 2, 128), (16, 1, 64), (7, 1, 128)])
@pytest.mark.parametrize("lens,topk,threshold", [([1], 3, 0), ([8, 31, 33], 3, 0), ([63, 64, 65, 96], 2, 64), ([127, 129, 300], 2, 0)])
def test_lengths_and_groups(m, oracle, hq, hkv, d, lens, topk, threshold):  # noqa: F811
    """(Sequences of a few tokens are compared below: their dQ is the difference of nearly equal terms, and Delta = <dO, O> of the
    bf16-rounded O is off by up to 3.5 x 2^-9 / sqrt(3) sqrt(d) |dO| |O| = 0.03, which times scale and a key is a tenth of the 0.1 at
    which the comparison's scale stops.)"""
    w = synth.make_varlen(lens, hq, hkv, d, seed=7000 + hq + sum(lens), dtype="bf16")
    gp, op = _params(m, oracle, "bf16", hq, hkv, d, n_init=1, n_local=1, topk_total=topk, dense_threshold=threshold)
    _check_backward(m, oracle, w, gp, op, "bf16")
    _check_backward(m, oracle, w, gp, op, "bf16", dense_all=True)


@pytest.mark.parametrize("dtype,hq,hkv,lens", [("bf16", 4, 1, [1100]), ("bf16", 8, 8, [700, 9]), ("bf16", 4, 2, [1985]), ("fp32", 4, 1, [900]),
                                               ("fp32", 4, 4, [513, 130])])
def test_chunks_of_64_tokens_and_more(m, oracle, dtype, hq, hkv, lens):  # noqa: F811
    w = synth.make_varlen(lens, hq, hkv, 128, seed=7100 + sum(lens), dtype=dtype)
    for topk in (5, 80):                                   # lists searched, and too long to be read whole
        gp, op = _params(m, oracle, dtype, hq, hkv, 128, n_init=1, n_local=1, topk_total=topk)
        _check_backward(m, oracle, w, gp, op, dtype)


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (8, 2, 64), (3, 1, 128), (16, 1, 64), (8, 8, 64), (6, 3, 64)])
@pytest.mark.parametrize("lens", [[4] * 400, [2, 3, 1, 5] * 40, [9] * 30, [333], [16, 1, 15, 9] * 30, [8, 7] * 120])
def test_the_same_values_as_fp32(m, hq, hkv, d, lens):  # noqa: F811
    """The fp32 kernels fed the bf16 call's inputs, outputs and Delta: dK and dV differ by fp32 roundings of sums over up to 333 x G rows."""
    w = synth.make_varlen(lens, hq, hkv, d, seed=7200 + len(lens) + hq, dtype="bf16")
    cu, f32 = w["cu_seqlens"], lambda x: x.float()
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    dout = torch.randn(q.shape, generator=torch.Generator().manual_seed(5)).cuda().bfloat16()
    kw = dict(n_init=1, n_local=1, topk_total=3)
    p16, p32 = m.Params.make("bf16", hq, hkv, d, **kw), m.Params.make("fp32", hq, hkv, d, **kw)
    r = m.sparse_prefill(p16, q, k, v, cu)
    for idx in (r["block_idx"], None):
        out, lse = (r["out"], r["lse"]) if idx is not None else m.dense_attn_fwd(p16, q, k, v, cu)
        _, dk, dv = m.sparse_attn_bwd(p16, q, k, v, idx, out, lse, dout, cu)
        _, dk32, dv32 = m.sparse_attn_bwd(p32, f32(q), f32(k), f32(v), idx, f32(out), lse, f32(dout), cu)
        for got, want in ((dk, dk32), (dv, dv32)):
            assert (got - want).abs().max() <= 1e-5 * max(float(want.abs().max()), 1.0)
