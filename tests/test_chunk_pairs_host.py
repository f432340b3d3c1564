"""The numbering of (token chunk, KV block) pairs that the dK/dV workgroups go by (csrc/chunk_pairs.h), and the rule for the chunk's
size, compiled for the host."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#define __device__
#include "chunk_pairs.h"
#include "launch_rules.h"
extern "C" int pairs(int n, int shift) { return ifv2::sequence_pairs(n, shift); }
extern "C" void at(int nth, int shift, int *r) { ifv2::pair_at(nth, shift, r[0], r[1]); }
extern "C" int shift(int bf16, int d, int G, const int *cu, int batch, int max_len, int hkv, long long nblocks, int sparse, int topk, int below,
                     long long *pairs) {
    int64_t n;
    const int s = ifv2::rules::generic_dkv_shift(bf16, d, G, {cu, batch, max_len, hkv, nblocks, sparse != 0, topk, below}, n);
    *pairs = n;
    return s;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("chunk_pairs")
    (d / "h.cpp").write_text(HARNESS)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2509_24663_amd", "csrc"),
                           "-o", str(d / "h.so"), str(d / "h.cpp")])
    return ctypes.CDLL(str(d / "h.so"))


@pytest.mark.parametrize("shift", [5, 6, 7, 8])
def test_every_pair_once(lib, shift):
    r = (ctypes.c_int * 2)()
    for n in list(range(1, 300)) + [511, 512, 513, 1985, 4100]:
        c = 1 << shift
        want = [(i, j) for i in range((n + c - 1) // c) for j in range((min((i + 1) * c, n) - 1) // 64 + 1)]
        assert lib.pairs(n, shift) == len(want), n
        for k in range(len(want)) if n < 300 or n > 4000 else ():
            lib.at(k, shift, r)
            assert (r[0], r[1]) == want[k], (n, k)


@pytest.mark.parametrize("shift,n", [(5, 1 << 20), (6, 1 << 20), (7, 1 << 20), (8, 65535 * 64)])
def test_long_sequences(lib, shift, n):
    """Both ends of the numbering and places in between, where a float's square root is off."""
    r, c, total = (ctypes.c_int * 2)(), 1 << shift, lib.pairs(n, shift)
    assert 0 < total < 1 << 31
    for k in [0, 1, total - 1, total - 2] + [total // 97 * i for i in range(97)]:
        lib.at(k, shift, r)
        assert 0 <= r[0] < (n + c - 1) // c and 0 <= r[1] <= (min((r[0] + 1) * c, n) - 1) // 64
        lib.at(k + 1, shift, r2 := (ctypes.c_int * 2)())
        assert k + 1 >= total or (r2[0], r2[1]) == ((r[0], r[1] + 1) if r[1] < (min((r[0] + 1) * c, n) - 1) // 64 else (r[0] + 1, 0))


def _shift(lib, lens, bf16=1, d=128, G=4, hkv=2, sparse=1, topk=16, below=0):
    cu, pairs = [0], ctypes.c_longlong()
    for n in lens:
        cu.append(cu[-1] + n)
    s = lib.shift(bf16, d, G, (ctypes.c_int * len(cu))(*cu), len(lens), max(lens), hkv, ctypes.c_longlong(sum((n + 63) // 64 for n in lens)),
                  sparse, topk, below, ctypes.byref(pairs))
    assert pairs.value == sum(lib.pairs(n, s) for n in lens)
    return 1 << s


def test_chunks(lib):
    assert [_shift(lib, [n]) for n in (300, 1000, 1985, 3000)] == [32, 64, 128, 256]
    assert _shift(lib, [300], 0) == 32 and _shift(lib, [4000] * 8) == 256 and _shift(lib, [65535 * 64], topk=64) == 256
    # why every block is selected does not matter
    for lens in ([300], [1985], [700] * 4):
        assert _shift(lib, lens, topk=64) == _shift(lib, lens, sparse=0) == _shift(lib, lens, below=max(lens) + 1)


@pytest.mark.parametrize("bf16,d,G,hkv,lens,topk,want", [
    (0, 128, 1, 4, [1000], 16, 128), (0, 128, 1, 4, [1000, 50], 16, 128), (0, 128, 4, 1, [1600], 16, 64), (0, 128, 1, 4, [1600], 64, 256),
    (1, 128, 4, 2, [1000], 4, 64), (1, 128, 4, 2, [1000, 50], 4, 64), (1, 128, 4, 1, [1000, 1000], 4, 64), (1, 64, 4, 2, [1985], 16, 128),
    (1, 64, 2, 3, [800], 64, 64), (1, 64, 2, 3, [800], 4, 64), (1, 64, 8, 1, [265, 1167, 2164], 16, 64), (1, 128, 14, 1, [1094, 1374, 285, 401], 16, 64), (1, 128, 1, 4, [1985], 16, 256)])
def test_chunks_of_small_groups_and_budgets(lib, bf16, d, G, hkv, lens, topk, want):
    """Whole backward with the chunk of this rule / with half or twice of it, the rule before: fp32, d 128, 4 heads on 4, 1000 tokens 105 / 118 us, 1600
    193 / 205; 4 heads on 1, 1600 tokens 167 / 179; bf16, d 128, 8 heads on 2, 4 blocks, 1000 tokens 48 / 63."""
    assert _shift(lib, lens, bf16, d, G, hkv, topk=topk) == want
