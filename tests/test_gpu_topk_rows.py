"""Selection from pooled scores at the row lengths where the kernel changes its code (quarters of the longest row's 64-block
chunks) and where live blocks end inside, at and past a chunk, against a plain sort."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _expected(row, pos, p):
    """init + local blocks and the largest others, equal scores to the smaller block; row: defined scores, others 0."""
    bt = pos // 64
    forced = set(range(min(p.n_init, bt + 1))) | set(range(max(0, bt - p.n_local + 1), bt + 1))
    rest = [j for j in range(bt + 1) if j not in forced]
    want = min(p.topk_total - p.n_init - p.n_local, len(rest))
    order = sorted(rest, key=lambda j: (-float(row[j]), j))[:want]
    got = sorted(forced | set(order))
    return got + [-1] * (p.topk_total - len(got))


@pytest.mark.parametrize("blocks,n_init,topk,pad,cmp", [
    (70, 1, 9, 0, (32, 16)), (130, 1, 20, 1, (64, 16)), (256, 30, 64, 3, (32, 16)), (300, 1, 64, 0, (32, 16)), (512, 0, 20, 1, (32, 16)), (700, 70, 140, 0, (32, 16)), (1024, 2, 96, 0, (64, 16)),
    (1500, 1, 16, 3, (32, 16)), (2048, 1, 64, 0, (32, 16))])
def test_pooled_rows_of_every_length_class(blocks, n_init, topk, pad, cmp):
    import paper_2509_24663_amd as m
    n = blocks * 64 - 7
    p = m.Params.make("bf16", 16, 1, 128, n_init=n_init, n_local=2, topk_total=topk, pool_pad=pad, cmp_len=cmp[0], cmp_stride=cmp[1])
    gen = torch.Generator("cuda").manual_seed(blocks)
    s = torch.rand((1, n, blocks), generator=gen, device="cuda")
    s = torch.where(s < 0.3, (s * 40).floor() / 40, s)                   # ties among a part of them
    idx = m.topk_pooled(p, s, [0, n])[0]
    chunks = (blocks + 63) // 64
    cap = 4 if chunks <= 4 else 8 if chunks <= 8 else 16 if chunks <= 16 else 32
    edges = [e for q in range(1, 5) for e in (q * cap // 4 * 4096 + d for d in (-65, -64, -1, 0, 1, 63, 64))]
    rows = sorted({r for r in edges + [0, 31, 64 * topk, n - 1, n // 3, n // 2 + 17] if 0 <= r < n})
    got, sc = idx[rows].cpu().numpy(), s[0, rows].cpu().numpy()
    for i, t in enumerate(rows):
        v = 0 if t < cmp[0] - 1 else (t - cmp[0] + 1) // cmp[1] + 1
        row = np.array([sc[i, j] if max(4 * j - pad, 0) < v else 0.0 for j in range(blocks)])
        assert got[i].tolist() == _expected(row, t, p), (blocks, t)
