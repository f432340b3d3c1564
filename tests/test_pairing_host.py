"""The pairing of a tile's union list (csrc/pair_entries.h), compiled for the host with a wavefront of 64 threads that meet at
every ballot and lane read: the list keeps every entry exactly once, in an order that follows from the list alone."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <pthread.h>
#include <stdint.h>
#include <algorithm>
#include <thread>
#include <vector>
using std::max;
#define __device__
struct int2 { int x, y; };
static int2 make_int2(int x, int y) { return int2{x, y}; }
static pthread_barrier_t meet;
static uint32_t slot[64];
static thread_local int self;
static void put(uint32_t v) { slot[self] = v; pthread_barrier_wait(&meet); }
static void done() { pthread_barrier_wait(&meet); }
static uint64_t __ballot(bool p) {
    put(p);
    uint64_t b = 0;
    for (int l = 0; l < 64; ++l) b |= (uint64_t)slot[l] << l;
    done();
    return b;
}
static int __builtin_amdgcn_readlane(int v, int l) { put((uint32_t)v); const int r = (int)slot[l]; done(); return r; }
static int __ffsll(long long x) { return __builtin_ffsll(x); }
static int __popc(uint32_t x) { return __builtin_popcount(x); }
#include "pair_entries.h"
template <int NW> static void run(int2 *rec, int body) {
    pthread_barrier_init(&meet, nullptr, 64);
    for (int w = 0; w < NW; ++w) {
        std::vector<std::thread> lanes;
        for (int l = 0; l < 64; ++l)
            lanes.emplace_back([=] { self = l; ifv2::pair_entries<NW>(rec, body, w, l); });
        for (auto &t : lanes) t.join();
    }
    pthread_barrier_destroy(&meet);
}
extern "C" void pair(int nw, int *rec, int body) {
    if (nw == 4) run<4>((int2 *)rec, body);
    else if (nw == 8) run<8>((int2 *)rec, body);
    else run<16>((int2 *)rec, body);
}
"""


@pytest.fixture(scope="module")
def pair(tmp_path_factory):
    d = tmp_path_factory.mktemp("pairing")
    (d / "harness.cpp").write_text(HARNESS)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-w", "-shared", "-fPIC", "-pthread", "-I",
                           os.path.join(ROOT, "paper_2509_24663_amd", "csrc"), "-o", str(d / "h.so"), str(d / "harness.cpp")])
    lib = ctypes.CDLL(str(d / "h.so"))

    def call(nw, masks):
        """The list (block numbers 0 ..) after the pairing; the last entry is not part of it."""
        rec = np.stack([np.arange(len(masks)), masks], 1).astype(np.int32)
        lib.pair(nw, rec.ctypes.data_as(ctypes.c_void_p), len(masks) - 1)
        return rec
    return call


def _paired(nw, masks):
    """The rule in plain words: inside each wave's range the first entry left is joined to the one that adds the least to what
    it costs alone; an entry costs as many units as its busiest SIMD has, waves w, w + 4, ... sharing one."""
    loads = np.array([[bin(int(mk) & (0x1111 << sd) & 0xffff).count("1") for sd in range(4)] for mk in masks])
    order = list(range(len(masks)))
    pairs = (len(masks) - 1) // 2
    for w in range(nw):
        lo, hi = 2 * (pairs * w // nw), 2 * (pairs * (w + 1) // nw)
        if 4 <= hi - lo <= 64:
            left, out = list(range(lo, hi)), []
            while left:
                first = left.pop(0)
                second = min(left, key=lambda e: ((loads[first] + loads[e]).max() - loads[e].max(), e))
                left.remove(second)
                out += [first, second]
            order[lo:hi] = out
    return order


@pytest.mark.parametrize("nw", [4, 8, 16])
def test_every_entry_once_in_the_order_of_the_rule(pair, nw):
    rng = np.random.default_rng(nw)
    full = (1 << nw) - 1
    for n in (1, 2, nw * 4, nw * 4 + 1, nw * 5 + 2, nw * 13 + 1):
        for masks in (np.full(n, full), rng.integers(1, full + 1, n), 1 << rng.integers(0, nw, n)):
            rec = pair(nw, masks)
            assert sorted(rec[:, 0].tolist()) == list(range(n)) and (rec[:, 1] == masks[rec[:, 0]]).all()
            assert rec[:, 0].tolist() == _paired(nw, masks), n


def test_no_kernel_asks_where_its_waves_run():
    csrc = os.path.join(ROOT, "paper_2509_24663_amd", "csrc")
    assert [f for f in sorted(os.listdir(csrc)) if "s_getreg" in open(os.path.join(csrc, f)).read()] == []
