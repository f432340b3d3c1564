"""The matrix-core backward when a key row holds infinities: gradients of the tokens that do not see it stay what they are with a finite row, at every tile size of dQ."""
import pytest
import torch

import synth
from helpers import to_dev
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu

LENS = [203, 1500, 2600]          # 4, 8 and 16 tokens per dQ tile (one KV head)


def _setup(m, oracle, n, dense):
    w = synth.make_prefill(n, 16, 1, 128, seed=2200 + n, dtype="bf16")
    gp, _ = _params(m, oracle, "bf16", 16, 1, 128, n_init=1, n_local=2, topk_total=4)
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    idx = None if dense else m.sparse_prefill(gp, q, k, v, [0, n])["block_idx"]
    out, lse = m.dense_attn_fwd(gp, q, k, v, [0, n]) if dense else m.sparse_attn_fwd(gp, q, k, v, idx, [0, n])
    dout = torch.randn(q.shape, generator=torch.Generator("cuda").manual_seed(3), device="cuda").bfloat16()
    return gp, q, k, v, idx, out, lse, dout


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("n", LENS)
def test_dq_of_tokens_that_do_not_see_the_key(m, oracle, n, dense):  # noqa: F811
    """Key u = 120 of block 1 (and its value row) holds an infinity: the 56 tokens in front of it in its block do not see it."""
    gp, q, k, v, idx, out, lse, dout = _setup(m, oracle, n, dense)
    want, _, _ = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, [0, n])
    u = 120
    k[0, u, 5], v[0, u, 7] = float("inf"), float("-inf")
    got, _, _ = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, [0, n])
    t = torch.arange(n, device="cuda")
    sees = t >= u if dense else (t >= u) & (idx[0] == u // 64).any(1)
    assert bool(torch.equal(got[~sees], want[~sees]))
    assert not torch.isfinite(got[sees]).all()
