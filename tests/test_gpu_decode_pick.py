"""Decode batches large enough for the selection to run as a kernel of its own: with and without the caller's list buffer,
dense and sparse sequences mixed, rows that keep everything, and a budget without a top-k part, against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth
from helpers import to_dev
from test_gpu_parity import _check_decode, _params, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("topk,n_local,threshold", [(64, 8, 1500), (70, 8, 0), (9, 8, 3000)])
def test_selection_as_its_own_kernel(m, oracle, topk, n_local, threshold):  # noqa: F811
    rng = np.random.default_rng(40 + topk)
    ctx = [int(x) for x in rng.integers(1, 6000, 21)] + [64, 4097, 7001]
    w = synth.make_decode(ctx, 32, 2, 128, seed=50 + topk, dtype="bf16", max_len=7040)
    gp, op = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=n_local, topk_total=topk, dense_threshold=threshold)
    assert _check_decode(m, oracle, w, ctx, gp, op, "bf16") > 0
    q, k, v = to_dev(w["q"], "bf16"), to_dev(w["k_cache"], "bf16"), to_dev(w["v_cache"], "bf16")
    kc = torch.zeros((len(ctx), 2, oracle.num_cmp(7040, op), 128), device="cuda")
    m.compress_k_append(gp, k, kc, [0] * len(ctx), ctx)
    out, lse, _ = m.sparse_decode(gp, q, k, v, kc, ctx)
    out2, lse2, none = m.sparse_decode(gp, q, k, v, kc, ctx, return_idx=False)
    assert none is None and torch.equal(out, out2) and torch.equal(lse, lse2)


@pytest.mark.parametrize("kw", [dict(lse_mode=1), dict(pool_len=60, pool_stride=40, pool_pad=3)])
def test_budget_without_a_top_k_part_outside_the_staged_form(m, oracle, kw):  # noqa: F811
    """The LSE Approximation and pooling windows too large for the staged form select in a kernel of their own, whose list
    must hold the forced blocks only, and nothing may be written behind it."""
    ctx = [5000, 700, 64, 1, 4097]
    w = synth.make_decode(ctx, 32, 2, 128, seed=61, dtype="bf16", max_len=5008)
    gp, op = _params(m, oracle, "bf16", 32, 2, 128, n_init=1, n_local=2, topk_total=3, **kw)
    assert _check_decode(m, oracle, w, ctx, gp, op, "bf16") == 2 * len(ctx)
    q, k, v = to_dev(w["q"], "bf16"), to_dev(w["k_cache"], "bf16"), to_dev(w["v_cache"], "bf16")
    kc = torch.zeros((len(ctx), 2, oracle.num_cmp(5008, op), 128), device="cuda")
    m.compress_k_append(gp, k, kc, [0] * len(ctx), ctx)
    n = len(ctx) * 2 * 3
    buf = torch.full((n + 4096,), -77, dtype=torch.int32, device="cuda")
    m.sparse_decode(gp, q, k, v, kc, ctx, idx=buf[:n].view(len(ctx), 2, 3))
    assert (buf[n:] == -77).all() and buf[:3].tolist() == [0, 77, 78]
