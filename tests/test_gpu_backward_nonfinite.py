"""The matrix-core backward when a key row holds infinities: gradients of the tokens and keys that have nothing to do with
that key stay what they are with a finite row, at every tile size of dQ and with odd and even token counts of dK / dV."""
import pytest
import torch

import synth
from helpers import to_dev, to_np
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu

LENS = [203, 1500, 2600]          # 4, 8 and 16 tokens per dQ tile (one KV head)


def _setup(m, oracle, n, dense, sign_from=None):
    w = synth.make_prefill(n, 16, 1, 128, seed=2200 + n, dtype="bf16")
    gp, _ = _params(m, oracle, "bf16", 16, 1, 128, n_init=1, n_local=2, topk_total=4)
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    if sign_from is not None:     # channel 3: logits towards +inf before that token, -inf from it on (key channel -inf)
        q[:, :, 3] = torch.where(torch.arange(n, device="cuda")[:, None] < sign_from, -1.0, 1.0)
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


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("n", LENS)
def test_dk_dv_of_a_key_whose_logits_are_minus_infinity(m, oracle, n, dense):  # noqa: F811
    """A key that no token gives any weight (logits of -inf where it is visible, +inf where it is not) has zero gradients, and
    the other keys' do not change."""
    u = n - 40 if n == 203 else 120       # (203: the last block, an odd number of tokens)
    gp, q, k, v, idx, out, lse, dout = _setup(m, oracle, n, dense, sign_from=u)
    _, dk0, dv0 = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, [0, n])
    k[0, u, 3] = float("-inf")
    _, dk, dv = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, [0, n])
    others = torch.arange(n, device="cuda") != u
    for got, want in ((dk, dk0), (dv, dv0)):
        assert not got[0, u].any(), to_np(got[0, u, :8])
        assert (got[0, others] - want[0, others]).abs().max().item() <= 1e-5 * want.abs().max().item()   # order of the adds
