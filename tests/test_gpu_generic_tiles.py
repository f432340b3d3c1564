"""The generic kernels (any group size, d 64 / 128, fp32 or bf16, any alignment) where their token tiles, block chunks
and key chunks can go wrong, against the CPU oracle through the C ABI."""
import numpy as np
import pytest
import torch

import synth
from helpers import assert_out_close, to_dev, to_np
from test_gpu_parity import _check_backward, _check_decode, _params, _run_prefill_case, m  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hq,hkv,d", [
    ("fp32", 2, 2, 64),        # G = 1: sixteen tokens per tile
    ("fp32", 3, 1, 128),       # G = 3: five tokens, one column unused, tiles straddle blocks
    ("bf16", 10, 2, 64),       # G = 5
    ("bf16", 6, 1, 128),       # G = 6: two tokens, four columns unused
    ("fp32", 12, 1, 64),       # G = 12: one token
    ("bf16", 16, 1, 64),       # G = 16, d 64
])
def test_group_sizes_ragged_and_switched(m, oracle, dtype, hq, hkv, d):  # noqa: F811
    """Sequences shorter than a tile, one token past a tile, one past a block, and on both sides of the switch."""
    w = synth.make_varlen([1, 17, 65, 130, 451], hq, hkv, d, seed=900 + hq + d, dtype=dtype)
    gp, op = _params(m, oracle, dtype, hq, hkv, d, n_init=1, n_local=1, topk_total=3, dense_threshold=100)
    _run_prefill_case(m, oracle, w, gp, op, dtype)
    _run_prefill_case(m, oracle, w, gp, op, dtype, fused_pool=True)
    _check_backward(m, oracle, w, gp, op, dtype)


def test_addresses_aligned_to_one_element_only(m, oracle):  # noqa: F811
    """bf16 rows of the paper's head shape that start at odd elements (row stride 129, buffers shifted by one) cannot
    take the tile kernels' 16-byte path; the generic kernels serve them."""
    n, hq, hkv, d = 333, 32, 2, 128
    w = synth.make_prefill(n, hq, hkv, d, seed=951, dtype="bf16")
    gp, op = _params(m, oracle, "bf16", hq, hkv, d, n_init=1, n_local=1, topk_total=3)

    def shifted(x, pad):
        x = to_dev(x, "bf16")
        buf = torch.zeros(x.shape[:-1] + (d + pad,), dtype=x.dtype, device="cuda") if pad else \
            torch.zeros(x.numel() + 1, dtype=x.dtype, device="cuda")
        view = buf[..., 1:] if pad else buf[1:].view(x.shape)
        view.copy_(x)
        return view
    q, k, v = shifted(w["q"], 0), shifted(w["k"], 1), shifted(w["v"], 1)
    assert q.data_ptr() % 16 == 2 and k.stride(1) == 129
    idx = m.sparse_prefill(gp, *(to_dev(w[x], "bf16") for x in ("q", "k", "v")), [0, n])["block_idx"]
    out, lse = m.sparse_attn_fwd(gp, q, k, v, idx, [0, n])
    dout = shifted(synth.round_to_bf16(np.random.default_rng(5).standard_normal((n, hq, d)).astype(np.float32)), 0)
    dq, dk, dv = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, [0, n])
    pos, G, idx_h = np.arange(n, dtype=np.int32), hq // hkv, to_np(idx)
    for h in range(hkv):
        Qh, sl = w["q"][:, h * G:(h + 1) * G], slice(h * G, (h + 1) * G)
        O, L = oracle.sparse_attn(Qh, pos, w["k"][h], w["v"][h], idx_h[h], op)
        assert_out_close(to_np(out)[:, sl], O, "bf16", "unaligned out")
        np.testing.assert_allclose(to_np(lse)[sl].T, L, atol=2e-3)
        grads = oracle.attn_bwd(Qh, pos, w["k"][h], w["v"][h], idx_h[h], to_np(dout)[:, sl], op)
        for name, got, ref in (("dq", to_np(dq)[:, sl], grads[0]), ("dk", to_np(dk)[h], grads[1]), ("dv", to_np(dv)[h], grads[2])):
            # the forward bar of bf16 data, relative to the gradient's largest value (Delta comes from the bf16 O)
            assert np.abs(got - ref).max() <= 2e-2 * np.abs(ref).max(), name


@pytest.mark.parametrize("dense", [True, False])
def test_values_a_token_does_not_see_stay_out_of_its_result(m, oracle, dense):  # noqa: F811
    """A tile's tokens share products: an infinity or a NaN in a row that only some of them see must reach those only."""
    n, hq, hkv, d = 203, 4, 1, 64
    w = synth.make_prefill(n, hq, hkv, d, seed=961, dtype="fp32")
    gp, _ = _params(m, oracle, "fp32", hq, hkv, d, n_init=1, n_local=1, topk_total=2)
    q, k, v = (to_dev(w[x], "fp32") for x in ("q", "k", "v"))
    idx = None if dense else m.sparse_prefill(gp, q, k, v, [0, n])["block_idx"]
    run = lambda kk, vv: (m.dense_attn_fwd(gp, q, kk, vv, [0, n]) if dense else  # noqa: E731
                          m.sparse_attn_fwd(gp, q, kk, vv, idx, [0, n]))
    out, lse = run(k, v)
    dout = torch.randn(q.shape, generator=torch.Generator("cuda").manual_seed(3), device="cuda")
    dq, _, _ = m.sparse_attn_bwd(gp, q, k, v, idx, out, lse, dout, [0, n])
    # rows 70 (block 1) and 201 (the last block): who sees them
    t = np.arange(n)
    sees70 = (t >= 70) if dense else (t >= 70) & (to_np(idx)[0] == 1).any(1)
    sees201 = t >= 201
    bad_v = v.clone()
    bad_v[0, 70, 3], bad_v[0, 201, 5] = float("inf"), float("nan")
    out_b, lse_b = run(k, bad_v)
    clean = torch.from_numpy(~(sees70 | sees201)).cuda()
    torch.testing.assert_close(out_b[clean], out[clean], rtol=1e-5, atol=1e-5)      # (computed again, other order)
    torch.testing.assert_close(lse_b, lse, rtol=1e-6, atol=1e-6)
    assert not torch.isfinite(out_b[torch.from_numpy(sees70).cuda(), :, 3]).any()
    assert torch.isnan(out_b[201:, :, 5]).all()
    bad_k = k.clone()
    bad_k[0, 70, 3], bad_k[0, 201, 5] = float("inf"), float("nan")
    dq_b, _, _ = m.sparse_attn_bwd(gp, q, bad_k, v, idx, out, lse, dout, [0, n])
    torch.testing.assert_close(dq_b[clean], dq[clean], rtol=1e-4, atol=1e-5)
    assert not torch.isfinite(dq_b[201:]).all()


def test_more_blocks_than_one_chunk_of_the_union(m, oracle):  # noqa: F811
    """A dense decode row over 1094 blocks (the union is handled 1024 block numbers at a time)."""
    ctx = [70000, 65537]
    w = synth.make_decode(ctx, 4, 1, 64, seed=971, dtype="fp32")
    gp, op = _params(m, oracle, "fp32", 4, 1, 64, n_init=1, n_local=2, topk_total=8, dense_threshold=69000)
    assert _check_decode(m, oracle, w, ctx, gp, op, "fp32") == 1


@pytest.mark.parametrize("pool", [(300, 70, 5), (256, 256, 0), (257, 3, 2), (5, 4, 200), (1, 300, 0), (2, 255, 1)])
def test_pooling_windows_around_the_key_chunk(m, oracle, pool):  # noqa: F811
    """Pooling windows longer than, as long as and far from a 256-key chunk of the fused scores."""
    w = synth.make_prefill(4500, 2, 1, 64, seed=980 + pool[0], dtype="fp32")
    gp, op = _params(m, oracle, "fp32", 2, 1, 64, n_init=1, n_local=2, topk_total=5, pool_len=pool[0], pool_stride=pool[1],
                     pool_pad=pool[2])
    rows = np.unique(np.concatenate([np.arange(0, 4500, 41), np.arange(4400, 4500)]))
    _run_prefill_case(m, oracle, w, gp, op, "fp32", rows=rows, fused_pool=True)
