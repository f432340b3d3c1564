"""dK / dV of the matrix-core backward at sizes that take each length of its token chunks (64 .. 512 tokens; 1024 in the
full-size test), with list lengths of both parities and a ragged end, against the CPU oracle through the C ABI."""
import pytest

import synth
from test_gpu_parity import _check_backward, _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1, 2, 66, 191], [3333], [4601], [6400], [9001]])
def test_token_chunks_of_the_dkv_kernel(m, oracle, lens):  # noqa: F811
    w = synth.make_varlen(lens, 16, 1, 128, seed=700 + len(lens), dtype="bf16")
    gp, op = _params(m, oracle, "bf16", 16, 1, 128, n_init=1, n_local=1, topk_total=3)
    _check_backward(m, oracle, w, gp, op, "bf16")
    if lens[0] == 3333:
        _check_backward(m, oracle, w, gp, op, "bf16", sel_bitmap_max_bytes=0)
