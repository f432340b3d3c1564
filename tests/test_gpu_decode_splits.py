"""Decode steps with few sequences: the selected blocks spread over as many workgroups as the merge takes at once, over fewer
where the caller's scratch holds no more partials, and refused below that; against the CPU oracle."""
import pytest
import torch

import synth
from helpers import assert_out_close, to_dev, to_np
from test_gpu_parity import _check_decode, _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 2, 9, 12])          # 2 to 24 pairs: 11 splits, 11, 11, 10
@pytest.mark.parametrize("n_local,topk", [(8, 64), (2, 12), (24, 64)])
def test_few_sequences(m, oracle, batch, n_local, topk):  # noqa: F811
    ctx = [8200 - 611 * i for i in range(batch)]
    w = synth.make_decode(ctx, 32, 2, 128, seed=70 + batch, dtype="bf16", max_len=8200)
    gp, op = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=n_local, topk_total=topk)
    assert _check_decode(m, oracle, w, ctx, gp, op, "bf16") > 0
    q, k, v = to_dev(w["q"], "bf16"), to_dev(w["k_cache"], "bf16"), to_dev(w["v_cache"], "bf16")
    kc = torch.zeros((batch, 2, oracle.num_cmp(8200, op), 128), device="cuda")
    m.compress_k_append(gp, k, kc, [0] * batch, ctx)
    need = m.decode_workspace_bytes(gp, batch, max(ctx))
    buf = torch.zeros(need + 256, dtype=torch.uint8, device="cuda")
    out, lse, idx = m.sparse_decode(gp, q, k, v, kc, ctx, workspace=buf[:need])
    tried = 0
    for size in range(need - 256, 0, -(need // 40) // 256 * 256):
        buf[size:] = 0x5A
        try:
            got = m.sparse_decode(gp, q, k, v, kc, ctx, workspace=buf[:size])
        except m.InfllmV2Error as e:
            assert e.status == -3
            break
        tried += 1
        assert (buf[size:] == 0x5A).all() and torch.equal(idx, got[2])
        assert_out_close(to_np(got[0]), to_np(out), "bf16")
        # the same keys in sums of other lengths: a few fp32 roundings of log2 of ~1000 summands, around lse < 16
        assert (got[1] - lse).abs().max() < 1e-5
    else:
        pytest.fail("no size was refused")
    # 55 blocks: 7 splits at least, 11 at most; the other budgets and 24 pairs have one form
    assert (tried > 0) == ((n_local, topk) == (8, 64) and batch <= 9)
