"""Compressed keys appended for sequences that grew by different amounts in one call: none, one, a few and many new rows per
sequence, so that a workgroup holds rows of one or of several (sequence, head) pairs.  The sums are taken in the order of
infllmv2_compress_k, so the rows are the same bit for bit, and rows outside [nc(prev), nc(ctx)) stay as they were."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hkv,d", [("bf16", 2, 128), ("fp32", 1, 64), ("bf16", 3, 64), ("fp32", 2, 128)])
@pytest.mark.parametrize("window", [(32, 16), (7, 3), (64, 16)])
def test_sequences_that_grew_differently(dtype, hkv, d, window):
    import paper_2509_24663_amd as m
    p = m.Params.make(dtype, 4 * hkv, hkv, d, cmp_len=window[0], cmp_stride=window[1])
    gen = torch.Generator("cuda").manual_seed(window[0] + d)
    for prev, ctx in (([999], [1008]), ([0, 500, 77, 600], [1, 500, 160, 1203]), ([0], [40]), ([31] * 5, [33, 64, 31, 400, 47])):
        cap, nc = max(ctx), [[m.num_cmp(p, n) for n in x] for x in (prev, ctx)]
        k = torch.randn((len(ctx), hkv, cap, d), generator=gen, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        kc = torch.full((len(ctx), hkv, max(max(nc[1]), 1), d), -7.0, device="cuda")
        m.compress_k_append(p, k, kc, prev, ctx)
        for b, n in enumerate(ctx):
            want = torch.full_like(kc[b], -7.0)
            if nc[1][b] > nc[0][b]:
                rows, _ = m.compress_k(p, k[b, :, :n].contiguous(), [0, n])
                want[:, nc[0][b]:nc[1][b]] = rows[:, nc[0][b]:nc[1][b]]
            assert torch.equal(kc[b], want), (prev, ctx, b)
