"""Short prompts, whose score kernel converts the compressed keys itself: the same scores as from the pre-pass (the prompt packed
behind a long one takes it), for ragged lengths, several sequences, and keys so large that single tiles need an exponent of
their own, infinities among them."""
import pytest
import torch

from test_gpu_parity import m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[31], [32], [777], [1055], [1536], [1537], [4090], [65, 1300, 40]])
@pytest.mark.parametrize("pooled,pad", [(False, 0), (True, 0), (True, 1)])
@pytest.mark.parametrize("large", ["", "all", "one tile", "infinite"])
def test_same_scores_as_from_the_pre_pass(m, lens, pooled, pad, large):  # noqa: F811
    torch.manual_seed(sum(lens) + pad)
    n, far = sum(lens), 9000
    q = torch.randn(n + far, 32, 128, device="cuda").bfloat16()
    k = torch.randn(2, n + far, 128, device="cuda").bfloat16()
    if large == "all":
        k[:, :n] *= 2.0 ** 17
        q[:n] *= 2.0 ** -15
    if large in ("one tile", "infinite"):
        at = max(lens) - max(lens) // 3
        k[:, at:at + 40] *= 2.0 ** 18
        q[:n] *= 2.0 ** -15
    if large == "infinite":
        k[0, at] = float("inf")
    p = m.Params.make("bf16", 32, 2, 128, n_init=1, n_local=1, topk_total=4, pool_pad=pad)

    def scores(qs, ks, lengths):
        cu = [0]
        for x in lengths:
            cu.append(cu[-1] + x)
        kc, cu_c = m.compress_k(p, ks.contiguous(), cu)
        width = 141 if pooled else 564
        out = torch.zeros(2, cu[-1], width, device="cuda")
        (m.block_scores_pooled if pooled else m.block_scores)(p, qs, kc, cu, cu_c, out=out)
        return out
    got = scores(q[:n], k[:, :n], lens)
    want = scores(torch.cat([q[n:], q[:n]]), torch.cat([k[:, n:], k[:, :n]], 1), [far] + lens)[:, far:]
    v = torch.cat([torch.clamp((torch.arange(x) - 31) // 16 + 1, min=0) for x in lens]).cuda()
    if not pooled:      # entries behind a token's visible keys are unspecified
        see = torch.arange(got.shape[2], device="cuda")[None] < v[:, None]
        got, want = got * see, want * see
    assert torch.equal(got.isnan(), want.isnan())
    got, want = got.nan_to_num(7.0), want.nan_to_num(7.0)
    # the same products in another order of the tokens: the exponentials' sums of a row may round differently
    assert (got - want).abs().max() <= 2e-5 and ((got - want).abs() <= 1e-5 * want.abs() + 1e-12).all()
