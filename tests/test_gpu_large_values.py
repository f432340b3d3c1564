"""Values next to the largest that bf16 holds: sums that are finite relative to the largest logit so far stay finite, whatever the softmax
reference of a kernel is."""
import pytest
import torch

from test_gpu_parity import m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n", [(64, 1500), (128, 1500), (128, 2100)])
def test_a_reference_that_lags_behind(m, d, n):  # noqa: F811
    """Four keys in the first four half blocks, one of them 7.48 binary orders above those far behind: less than a lazily moved reference
    may lag.  All other weights are nothing, so relative to the largest logit they sum up to 4 and sums of V = 2^122 stay below 2^125;
    179 V would be 2^129.5."""
    hq, hkv, hit = 8, 2, 700
    gp = m.Params.make("bf16", hq, hkv, d, softmax_scale=1.0)
    q, k = torch.zeros(n, hq, d, device="cuda", dtype=torch.bfloat16), torch.zeros(hkv, n, d, device="cuda", dtype=torch.bfloat16)
    q[..., 0] = 1.0
    k[..., 0] = -30.0
    k[:, [0, 32, 64, 96], 0] = 0.0
    k[:, hit, 0] = 5.1875
    v = torch.full((hkv, n, d), 2.0 ** 122, device="cuda", dtype=torch.bfloat16)
    out, lse = m.dense_attn_fwd(gp, q, k, v, [0, n])
    # every row is a mean of equal values: 2^122 up to the rounding of its weights' sum
    assert torch.isfinite(out).all() and (out.float() / 2.0 ** 122 - 1).abs().max() <= 2.0 ** -7
    assert (lse.double() - torch.logcumsumexp(k[0, :, 0].double(), 0)).abs().max() <= 2e-3


def test_decode_blocks_of_falling_logits(m):  # noqa: F811
    """Sixteen blocks per wavefront whose largest logits fall by 0.45 binary orders each.  A reference that follows them down would stand
    0.45 x 15 = 6.7 orders below the first and bring V = 2^122 to 2^128.7; relative to the largest the weights sum up to at most
    4 x 3.7 x 2."""
    hq, hkv, d, batch, n = 32, 2, 128, 128, 8190
    gp = m.Params.make("bf16", hq, hkv, d, n_init=1, n_local=8, topk_total=64, dense_threshold=8192, softmax_scale=1.0)
    q, k = torch.zeros(batch, hq, d, device="cuda", dtype=torch.bfloat16), torch.zeros(batch, hkv, n, d, device="cuda", dtype=torch.bfloat16)
    q[..., 0] = 1.0
    k[..., 0] = -30.0
    for block in range(n // 64):
        k[:, :, 64 * block + block % 64, 0] = -0.45 * 0.6931 * (block % 64 // 4)
    v = torch.full((batch, hkv, n, d), 2.0 ** 122, device="cuda", dtype=torch.bfloat16)
    kc = torch.zeros(batch, hkv, m.num_cmp(gp, n), d, device="cuda")
    m.compress_k_append(gp, k, kc, [0] * batch, [n] * batch)
    out, lse, _ = m.sparse_decode(gp, q, k, v, kc, [n] * batch)
    assert torch.isfinite(out).all() and (out.float() / 2.0 ** 122 - 1).abs().max() <= 2.0 ** -7
    assert (lse.double() - torch.logsumexp(k[0, 0, :, 0].double(), 0)).abs().max() <= 2e-3
