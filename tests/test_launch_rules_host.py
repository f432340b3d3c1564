"""Which form of a kernel a call takes (csrc/launch_rules.h), compiled for the host: rules that depend on a batch's lengths."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "launch_rules.h"
using namespace ifv2::rules;
extern "C" void generic(int bf16, int d, int hkv, int tokens, const int *cu, int batch, int sparse, int topk, int below, int *r) {
    const Walks x = walks(cu, batch, tokens, sparse, topk, below);
    const GenericForm f = generic_form(bf16, d, hkv, x), g = generic_dq_form(bf16, d, hkv, x);
    r[0] = f.groups;
    r[1] = f.ahead;
    r[2] = g.groups;
    r[3] = g.ahead;
}
extern "C" int fp32_ahead(int d, int hkv, int tokens, const int *cu, int batch, int sparse, int topk, int below) {
    const Walks x = walks(cu, batch, tokens, sparse, topk, below);
    return fp32_rows_ahead(d, hkv, x.one * hkv, x);
}
extern "C" int back(const int *cu, int batch, int tokens, int tiles, int hkv, int sparse, int topk, int below, int resident, int side) {
    const double far = cu ? walks(cu, batch, tokens, sparse, topk, below).half_blocks : 0;
    return back_and_forth(cu, batch, tokens, tiles, hkv, sparse, topk, below, far, resident, side);
}
extern "C" int staged_form(int bwd, int d, int hkv, int tokens, const int *cu, int batch, int sparse, int topk, int below) {
    const Walks x = walks(cu, batch, tokens, sparse, topk, below);
    return staged(bwd, d, x.two * hkv, x);
}
extern "C" int short_waves(const int *cu, int batch, int max_len, int hkv, int sparse, int topk, int below) {
    return short_attn_waves(cu, batch, max_len, hkv, sparse, topk, below);
}
extern "C" void splits(long long pairs, int entries, int waves, int *r) {
    const DecodeSplits d = decode_splits(pairs, entries, waves);
    r[0] = d.bpw;
    r[1] = d.nsplit;
}
extern "C" int short_steps(int d, int G, int max_len, long long blocks) { return dkv_short_steps(d, G, max_len, blocks); }
extern "C" int tile(const int *cu, int batch, int max_len, int hkv, int sparse, int topk, int below, int bwd) {
    return attn_tile_tokens(cu, batch, max_len, hkv, sparse, topk, below, bwd);
}
extern "C" long long busy(int len, int c) {
    return c == 32 ? dkv_busy<0>(len) : c == 64 ? dkv_busy<1>(len) : c == 128 ? dkv_busy<2>(len) : c == 256 ? dkv_busy<3>(len)
           : c == 512 ? dkv_busy<4>(len) : dkv_busy<5>(len);
}
extern "C" int chunk(const int *cu, int batch, int max_len, int hkv, long long nblocks, int sparse, int topk, int below, long long most) {
    return dkv_chunk({cu, batch, max_len, hkv, nblocks, sparse != 0, topk, below}, most);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src = d / "rules.cpp"
    src.write_text(HARNESS)
    lib = d / "rules.so"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2509_24663_amd", "csrc"),
                           "-o", str(lib), str(src)])
    return ctypes.CDLL(str(lib))


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return (ctypes.c_int * len(cu))(*cu)


def _generic(rules, bf16, d, hq, hkv, lens, topk=16, sparse=1, below=0):
    r = (ctypes.c_int * 4)()
    rules.generic(bf16, d, hkv, 16 // (hq // hkv), _cu(lens), len(lens), sparse, topk, below, r)
    return tuple(r)


def test_many_short_sequences_take_one_column_group(rules):
    """Tiles that end with their sequence have nothing for a second group: the number of sequences alone must not choose it."""
    for lens in ([4] * 500, [1] * 2000, [10] * 200, [33] * 242, [100] * 40):
        for bf16, d in ((1, 128), (1, 64), (0, 128), (0, 64)):
            f = _generic(rules, bf16, d, 8, 2, lens)
            assert f[:2] == (1, 0) and (lens[0] > 33 or f[2:] == (1, not bf16 and d == 128)), (lens[:1], bf16, d)
    # a long sequence keeps the form it has alone
    assert _generic(rules, 1, 128, 8, 2, [1985]) == (2, 1, 2, 1)
    assert _generic(rules, 1, 128, 8, 2, [1985, 3, 5]) == (2, 1, 2, 1)
    assert _generic(rules, 0, 64, 4, 1, [2048], topk=8) == (1, 1, 2, 1)
    assert _generic(rules, 1, 128, 8, 2, [6000]) == (2, 0, 2, 1)
    assert _generic(rules, 0, 128, 8, 2, [600]) == (1, 1, 1, 1)
    assert _generic(rules, 1, 128, 8, 2, []) == (1, 1, 1, 1)


def _back(rules, lens, tokens, hkv, resident, topk=16, sparse=1, below=0, side=0):
    tiles = sum(-(-n // tokens) for n in lens) if side else sum(lens) // tokens + len(lens)      # (the staged form launches no empty ones)
    return tiles, rules.back(_cu(lens), len(lens), tokens, tiles, hkv, sparse, topk, below, resident, side)


def test_order_of_generic_attention_workgroups(rules):
    """Back and forth while all workgroups are on the chip; for packed batches only where the fullest CU then has less to do."""
    assert _back(rules, [1020], 4, 1, 768)[1] == 0 and _back(rules, [1024], 4, 1, 768)[1] == 1        # 256 and 257 workgroups
    assert _back(rules, [3068], 4, 1, 768)[1] == 1 and _back(rules, [3072], 4, 1, 768)[1] == 0        # 768 and 769
    assert _back(rules, [1024], 4, 1, 256)[1] == 0 and _back(rules, [2000], 4, 1, 2048)[1] == 0
    assert rules.back(None, 300, 1, 300, 2, 1, 16, 0, 768, 0) == 1 and rules.back(None, 2, 1, 1 << 30, 4, 1, 16, 0, 768, 0) == 0   # (2^32 workgroups)
    assert _back(rules, [2463, 2040, 68], 8, 1, 768, sparse=0)[1] == 1
    assert _back(rules, [2490] + [1] * 100, 8, 1, 768, sparse=0)[1] == 0 and _back(rules, [2675] + [100] * 10, 8, 1, 768)[1] == 0
    import random
    rng, seen = random.Random(3), set()
    assert _back(rules, [2389, 434, 509], 32, 4, 512, side=1)[1] == 0 and _back(rules, [3000], 8, 1, 512, side=1)[1] == 1
    for i in range(500):
        tokens, hkv, side = rng.choice([1, 2, 4, 8, 16, 32]), rng.choice([1, 2, 3, 8]), i % 2
        lens = [rng.choice([0, 1, rng.randint(1, 90), rng.randint(100, 3000)]) for _ in range(rng.randint(2, 40))]
        topk, sparse, below = rng.choice([1, 4, 16]), rng.randint(0, 1), rng.choice([0, 500])
        tiles, got = _back(rules, lens, tokens, hkv, 768, topk, sparse, below, side)
        n = tiles * hkv
        if not 256 < n <= 768:
            assert not got
            continue
        count = [-(-L // tokens) for L in lens]
        far = sum(c * min((L + 32) / 64, 2 * topk if sparse and L >= below else 1e9) for c, L in zip(count, lens)) / sum(count)
        if far < 4:                                                  # (not counted)
            assert got
            continue
        work = []
        for L in lens:
            most = 2 * topk if sparse and L >= below else 1 << 30
            work += [4 + min((min(t + tokens, L) + 31) // 32, most) for t in range(0, L, tokens)]
        work = [0] * (tiles - len(work)) + work[::-1]
        order = [w for w in work for _ in range(hkv)]                # heads side by side
        one = order if side else [work[b % tiles] for b in range(n)]
        rows = [order[i:i + 256] for i in range(0, n, 256)]
        two = sum((r[::-1] if i % 2 else r for i, r in enumerate(rows)), [])
        fullest = [max(sum(x[c::256]) for c in range(256)) for x in (one, two)]
        assert got == (fullest[1] < fullest[0]), (lens, tokens, hkv)
        seen.add((side, got))
    assert len(seen) == 4


@pytest.mark.parametrize("d,G,max_len,blocks,want", [(64, 4, 4, 601, 1), (64, 4, 4, 600, 0), (64, 4, 5, 4000, 0), (64, 1, 16, 700, 1), (64, 1, 17, 4000, 0),
                                                     (64, 2, 8, 700, 1), (64, 16, 4, 700, 1), (128, 1, 1, 4000, 0)])
def test_dkv_in_steps_of_16_rows(rules, d, G, max_len, blocks, want):
    assert rules.short_steps(d, G, max_len, ctypes.c_longlong(blocks)) == want


def _chunk(rules, lens, hkv=2, sparse=0, topk=16, below=0, most=0xffffffff // 64):
    nblocks = sum((n + 63) // 64 for n in lens)
    return rules.chunk(_cu(lens), len(lens), max(lens), hkv, ctypes.c_longlong(nblocks), sparse, topk, below, ctypes.c_longlong(most))


def test_matrix_core_dkv_workgroups_are_counted_exactly(rules):
    rules.busy.restype = ctypes.c_longlong
    for c in (32, 64, 128, 256, 512, 1024):
        for n in list(range(0, 700)) + [1023, 1024, 1025, 4095, 4100, 262144]:
            want = sum((min(i + c, n) - 1) // 64 + 1 for i in range(0, n, c))
            assert rules.busy(n, c) == want, (n, c)


def test_matrix_core_dkv_chunks(rules):
    # chunks longer than every sequence are the same work: never better than the shortest of them
    for lens in ([300] * 100, [100] * 400, [64] * 1000, [200] * 8, [500] * 30):
        for hkv in (1, 2, 4, 8):
            for sparse in (0, 1):
                c = _chunk(rules, lens, hkv, sparse)
                assert c < 2 * lens[0], (lens[0], hkv, c)
    for lens, hkv, good in (([300] * 100, 2, (64, 128)), ([300] * 100, 4, (128,)), ([500] * 30, 8, (64, 128, 256)), ([65] * 300, 1, (32,)),
                            ([500], 2, (32,)), ([1000] * 10, 2, (256,)), ([200] * 8, 1, (32,))):
        assert _chunk(rules, lens, hkv) in good, (lens[0], hkv)
    assert _chunk(rules, [32768], 2, sparse=1, topk=64) == 1024 and _chunk(rules, [8000], 2, sparse=1, topk=64) == 256
    # a launch's limit: chunks that are too many are left out, and 0 says that none is few enough
    assert _chunk(rules, [100000] + [1] * 60000, 8, most=8 * 98 * (1563 + 60000)) == 1024
    assert _chunk(rules, [100000] + [1] * 60000, 8, most=8 * 98 * (1563 + 60000) - 1) == 0


def test_attention_tiles(rules):
    def tile(lens, hkv=2, sparse=1, topk=64, below=0, bwd=0):
        return rules.tile(_cu(lens), len(lens), max(lens, default=0), hkv, sparse, topk, below, bwd)
    assert [tile([n]) for n in (1, 512, 513, 1024, 1025, 2048, 2049)] == [4, 4, 8, 8, 8, 8, 16]
    assert [tile([n], 1) for n in (1024, 1025, 2048, 2049, 4096, 4097)] == [4, 8, 8, 8, 8, 16]
    assert [tile([n], 8) for n in (128, 129, 256, 257, 2000)] == [4, 8, 8, 16, 16]
    # a short sequence beside a long one changes nothing; two alike do
    assert tile([1400, 10]) == tile([10, 1400]) == tile([1400]) == 8 and tile([1024, 1024]) == tile([1200, 800]) == 16
    # lists with small budgets: the gradient keeps the small tiles, dense calls and sequences under the threshold too
    for n, hkv, topk, want in ((4096, 1, 16, 16), (2800, 1, 12, 8), (3600, 1, 8, 16), (2040, 2, 12, 16), (1400, 2, 12, 8), (2040, 2, 64, 8)):
        assert tile([n], hkv, topk=topk) == want, (n, hkv, topk)
        assert tile([n], hkv, topk=topk, bwd=1) == tile([n], hkv, sparse=0, topk=topk) == tile([n], hkv, topk=topk, below=n + 1) == 8
    assert tile([]) == 4


@pytest.mark.parametrize("d,hq,hkv,lens,topk,ahead", [
    (64, 4, 1, [1000], 8, 1), (64, 4, 1, [1200], 16, 1), (64, 4, 1, [1201], 16, 0), (64, 4, 1, [1025], 4, 0), (64, 8, 2, [1000], 8, 0),
    (64, 4, 1, [300], 8, 0), (128, 8, 2, [1000], 8, 1), (128, 8, 2, [1024], 8, 1), (128, 8, 2, [1025], 8, 1), (128, 8, 2, [1000, 50], 16, 1),
    (128, 8, 2, [1300], 8, 0), (128, 4, 1, [1985], 16, 1), (128, 4, 1, [2100], 4, 0), (128, 4, 1, [1255, 347], 16, 1), (128, 4, 4, [4000], 16, 1), (128, 4, 4, [1600], 16, 0), (128, 8, 8, [1000], 16, 0),
    (128, 16, 4, [1000], 16, 1), (128, 16, 4, [1000], 4, 0), (128, 4, 1, [150], 8, 0), (128, 4, 1, [], 8, 0),
    (128, 3, 3, [1968], 16, 1), (128, 3, 3, [1969], 16, 0), (128, 6, 3, [834], 16, 1), (128, 6, 3, [834], 4, 0), (128, 4, 4, [1290], 16, 0)])
def test_fp32_rows_ahead_only_where_a_cu_has_one_workgroup_to_run(rules, d, hq, hkv, lens, topk, ahead):
    assert rules.fp32_ahead(d, hkv, 16 // (hq // hkv), _cu(lens), len(lens), 1, topk, 0) == ahead


@pytest.mark.parametrize("bwd,d,hq,hkv,lens,want", [
    (0, 128, 8, 2, [1352], 0), (0, 128, 8, 2, [1353], 1), (0, 128, 8, 2, [4] * 400, 0), (0, 64, 8, 2, [1200], 0), (0, 64, 8, 2, [1201], 1),
    (0, 64, 8, 2, [4] * 400, 0), (0, 64, 8, 2, [300] * 6, 0), (0, 64, 8, 2, [300] * 8, 1), (1, 128, 8, 2, [592], 0), (1, 128, 8, 2, [593], 1), (1, 128, 8, 2, [30] * 100, 0),
    (1, 64, 8, 2, [30] * 100, 1), (1, 64, 8, 2, [592], 0), (1, 64, 4, 1, [], 0),
    (0, 128, 4, 1, [189] * 16, 0), (0, 128, 4, 1, [238] * 12, 0), (0, 128, 16, 4, [200] * 4, 1), (0, 128, 6, 3, [309] * 6, 1)])
def test_rows_through_lds_for_large_calls(rules, bwd, d, hq, hkv, lens, want):
    assert rules.staged_form(bwd, d, hkv, 16 // (hq // hkv), _cu(lens), len(lens), 1, 16, 0) == want


@pytest.mark.parametrize("hkv,lens,topk,want", [(2, [512], 16, 2), (2, [513], 16, 2), (2, [640], 16, 2), (2, [500, 13], 16, 1), (2, [300] * 4, 16, 1),
                                                (4, [260], 16, 1), (2, [600], 4, 1), (3, [500], 16, 1)])
def test_wavefronts_per_token_of_short_prompts(rules, hkv, lens, topk, want):
    assert rules.short_waves(_cu(lens), len(lens), max(lens), hkv, 1, topk, 0) == want


def test_no_more_workgroups_than_a_launch_holds(rules):
    """Tiles and heads side by side in x, 256 threads each: fewer than 2^32 threads, or the kernels with heads in y serve the call."""
    for bwd in (0, 1):
        for n, want in ((55924, 1), (55925, 0)):                      # sequences of 150 tiles on 2 KV heads: 16777200 and 16777500 workgroups
            assert rules.staged_form(bwd, 64, 2, 1, _cu([300] * n), n, 0, 16, 0) == want
    for n, want in ((8388607, 1), (8388608, 0)):
        cu = (ctypes.c_int * (n + 1))(*range(n + 1))
        assert rules.short_waves(cu, n, 1, 2, 0, 16, 0) == want


@pytest.mark.parametrize("bwd,d,hq,hkv,lens,topk,want", [
    (0, 128, 4, 1, [3000] + [4] * 300, 4, 0), (0, 128, 4, 1, [3000] + [4] * 300, 16, 1), (0, 128, 4, 4, [1000] + [4] * 300, 16, 0),
    (0, 128, 8, 2, [1000] + [1] * 200, 4, 0), (0, 128, 8, 2, [1000] + [1] * 200, 16, 1), (0, 64, 4, 1, [1000] + [1] * 200, 16, 0),
    (0, 64, 8, 2, [1000] + [1] * 200, 4, 0), (0, 64, 8, 2, [1000] + [1] * 200, 16, 1), (0, 64, 8, 2, [3000] + [1] * 500, 4, 1),
    (1, 64, 8, 8, [1] * 500, 16, 0), (1, 64, 8, 8, [16] * 500, 16, 1), (1, 64, 8, 2, [1] * 2000, 16, 0), (1, 64, 8, 2, [4] * 2000, 16, 1),
    (1, 64, 8, 1, [1] * 2000, 16, 1)])
def test_rows_through_lds_not_for_empty_second_groups(rules, bwd, d, hq, hkv, lens, topk, want):
    assert rules.staged_form(bwd, d, hkv, 16 // (hq // hkv), _cu(lens), len(lens), 1, topk, 0) == want


def _splits(rules, pairs, entries, waves=4):
    r = (ctypes.c_int * 2)()
    rules.splits(ctypes.c_longlong(pairs), entries, waves, r)
    return tuple(r)


def test_decode_splits_hold_every_block(rules):
    """Every entry has a place, in at most sixteen rounds of the workgroup's wavefronts, and no more splits than four blocks each would make."""
    for pairs in list(range(1, 600)) + [1000, 4000, 65535]:
        for entries in list(range(0, 70)) + [127, 128, 129, 500, 1024, 4096]:
            bpw, ns = _splits(rules, pairs, entries)
            assert bpw % 4 == 0 and 4 <= bpw <= 16 * 4 and ns * bpw >= entries and 1 <= ns <= max((entries + 3) // 4, 1), (pairs, entries)


def test_decode_splits_fill_the_chip(rules):
    """Steps in microseconds, with one workgroup per pair / with this: 130 pairs 113 / 106, 264 207 / 186, 320 221 / 208."""
    assert [_splits(rules, p, 55)[1] for p in (43, 64, 96, 128, 130, 160, 192, 256, 264, 320, 400, 512, 600)] == [5, 4, 2, 2, 3, 3, 1, 1, 3, 3, 1, 1, 2]
    assert _splits(rules, 512, 128) == (64, 2) and _splits(rules, 300, 128) == (32, 4) and _splits(rules, 128, 0) == (4, 1)


def _cases():
    import test_gpu_generic_groups as g
    return g.GENERIC_FORMS


@pytest.mark.parametrize("dtype,hq,hkv,d,lens,topk,below,lds,form", _cases())
def test_forms_that_the_gpu_tests_count_on(rules, dtype, hq, hkv, d, lens, topk, below, lds, form):
    """A rule that moves one of these calls to another form leaves the form it had without a test."""
    bf16, tokens = dtype == "bf16", 16 // (hq // hkv)
    got = _generic(rules, bf16, d, hq, hkv, lens, topk, 1, below)
    if not bf16:
        got = (1, rules.fp32_ahead(d, hkv, tokens, _cu(lens), len(lens), 1, topk, below)) + got[2:]
    assert got == form
    assert tuple(bf16 and rules.staged_form(b, d, hkv, tokens, _cu(lens), len(lens), 1, topk, below) for b in (0, 1)) == lds
