"""Which entries of the pooled scores the matrix-core kernel writes: every block up to the token's own whose clipped window holds
a visible key, and nothing else, also behind the buffer, for compressed windows of one stride to several and both paddings
it serves.  Values: the maximum over the window of what the unpooled call stores."""
import numpy as np
import pytest
import torch

import synth
from helpers import to_dev, to_np
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("window", [(16, 16), (17, 16), (32, 16), (64, 16)])
@pytest.mark.parametrize("lens", [[640, 64, 1, 128], [2048], [5 * 1024]])       # 1, 2 and 4 tokens per wavefront
def test_entries_written(m, oracle, lens, window, pad):  # noqa: F811
    w = synth.make_varlen(lens, 32, 2, 128, seed=2500 + lens[0], dtype="bf16")
    gp, op = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=1, topk_total=4, cmp_len=window[0], cmp_stride=window[1],
                     pool_pad=pad)
    q, k = to_dev(w["q"], "bf16"), to_dev(w["k"], "bf16")
    cu, T, width = w["cu_seqlens"], sum(lens), max(lens) // 64
    kc, cu_c = m.compress_k(gp, k, cu)
    buf = torch.full((2 * T * width + 64,), -5.0, device="cuda")
    m.block_scores_pooled(gp, q, kc, cu, cu_c, out=buf[:-64].view(2, T, width))
    assert (buf[-64:] == -5.0).all()
    got, single = to_np(buf[:-64].view(2, T, width)), to_np(m.block_scores(gp, q, kc, cu, cu_c))
    for s, n in enumerate(lens):
        for t in range(n):
            row, v = int(cu[s]) + t, oracle.visible_cmp(t, op)
            want = np.full((2, width), -5.0, np.float32)
            for j in range(t // 64 + 1):
                lo, hi = max(4 * j - pad, 0), min(4 * j - pad + 5, v)
                if lo < v:
                    want[:, j] = single[:, row, lo:hi].max(1)
            if t % 5 == 0 or t % 64 > 60:
                assert np.array_equal(got[:, row], want), (s, t)
