"""The matrix-core score kernel where its tiles change (one, two and four tokens per wavefront: 1536 and 4096 tokens on two KV
heads), ragged and packed, and with compression strides that are no power of two, against the CPU oracle."""
import numpy as np
import pytest

import synth
from helpers import to_dev, to_np
from test_gpu_parity import _params, m  # noqa: F401

pytestmark = pytest.mark.gpu

# Relative error of a score = absolute error of a logit and of its row's log-sum-exp.  A compressed key is rounded to fp16
# (2^-12 / sqrt(3) rms), so a logit is off by scale * sqrt(sum q^2 k^2) times that: with q^2 ~ 1.25, k^2 ~ 0.25 + 1/24 (windows
# of 24 keys) and 128 dimensions 8.5e-5 rms.  Five times that for the largest of ~1e6 logits, and as much again for a
# normaliser that hangs on one or two coarse keys.
RTOL = 10 * 8.5e-5


@pytest.mark.parametrize("lens", [[1535], [1536], [1537], [4095], [4096], [4097], [37, 1200, 1, 290], [2300, 33, 1800],
                                  [700, 701, 31, 699, 703], [1801, 1850], [1750, 33, 1801], [1751, 600, 610, 640], [2048, 2047]])
@pytest.mark.parametrize("window", [(32, 16), (24, 12), (25, 5)])
@pytest.mark.parametrize("lse_mode", [0, 1])
def test_scores(m, oracle, lens, window, lse_mode):  # noqa: F811
    if lse_mode and window[0] % window[1]:
        pytest.skip("the coarse keys need windows of whole strides")
    w = synth.make_varlen(lens, 32, 2, 128, seed=2600 + lens[0] + window[1], dtype="bf16")
    gp, op = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=1, topk_total=4, cmp_len=window[0], cmp_stride=window[1],
                     lse_mode=lse_mode)
    q, k = to_dev(w["q"], "bf16"), to_dev(w["k"], "bf16")
    cu = w["cu_seqlens"]
    kc, cu_c = m.compress_k(gp, k, cu)
    got = to_np(m.block_scores(gp, q, kc, cu, cu_c))
    for s, n in enumerate(lens):
        a = int(cu[s])
        pos = np.unique(np.concatenate([np.arange(0, n, 61), np.arange(max(0, n - 40), n), np.arange(min(n, 40))])).astype(np.int32)
        for h in range(2):
            kch = oracle.compress_k(w["k"][h, a:a + n], op)
            want = oracle.block_scores(w["q"][a + pos, h * 16:h * 16 + 16], pos, kch, op,
                                       kc2=oracle.compress_k(w["k"][h, a:a + n], op, level=2) if lse_mode else None)
            for i, t in enumerate(pos):
                v = oracle.visible_cmp(int(t), op)
                x, y = got[h, a + t, :v], want[i, :v]
                assert (np.abs(x - y) <= 1e-7 + RTOL * np.abs(y)).all(), (s, h, t)
