"""The selection bitmap of the matrix-core backward: lengths around its tiles (256 tokens, 32-token words, 64-key blocks),
several sequences, one that attends densely; the words a tile does not write hold ones beforehand, so a reader that looked
at them would take tokens in front of its block.  The reference is the same call without the bitmap (compared with the
oracle in the other backward tests): the same tokens, so equal up to the order in which the float atomics arrive."""
import numpy as np
import pytest
import torch

import synth
from helpers import to_dev
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1, 255, 256, 257, 64], [31, 2047, 65, 512], [4129, 33]])
def test_bitmap_in_a_workspace_full_of_ones(m, oracle, lens):  # noqa: F811
    K, T = 5, sum(lens)
    w = synth.make_varlen(lens, 32, 2, 128, seed=900 + len(lens), dtype="bf16")
    gp, _ = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=1, topk_total=K, dense_threshold=40)
    cu = [0] + np.cumsum(lens).tolist()
    rng = np.random.default_rng(901)
    idx = np.full((2, T, K), -1, np.int32)
    for s, n in enumerate(lens):
        for h in range(2):
            for t in range(n):
                bt = t // 64
                pick = rng.permutation(bt)[:K - 1]
                row = np.sort(np.append(pick, bt))
                idx[h, cu[s] + t, :len(row)] = row
    q, k, v = (to_dev(w[x], "bf16") for x in ("q", "k", "v"))
    idx_d = torch.from_numpy(idx).cuda()
    dout = torch.randn(q.shape, generator=torch.Generator("cuda").manual_seed(5), device="cuda").bfloat16()
    out, lse = m.sparse_attn_fwd(gp, q, k, v, idx_d, cu)
    want = m.sparse_attn_bwd(gp, q, k, v, idx_d, out, lse, dout, cu, sel_bitmap_max_bytes=0)
    need = m.workspace_bytes(m.OP_SPARSE_ATTN_BWD, gp, len(lens), T, max(lens))
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    got = m.sparse_attn_bwd(gp, q, k, v, idx_d, out, lse, dout, cu, workspace=ws)
    assert torch.equal(got[0], want[0])
    for a, b in zip(got[1:], want[1:]):
        assert (a - b).abs().max().item() <= 1e-5 * b.abs().max().item()      # order of float additions
