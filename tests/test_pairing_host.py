"""The pairing of a tile's union list (csrc/pair_entries.h), compiled for the host with a wavefront of 64 threads that meet at
every ballot and lane read: the list keeps every entry exactly once, wherever the hardware puts the waves."""
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
template <int NW> static void run(int2 *rec, int body, const uint32_t *simd_waves) {
    pthread_barrier_init(&meet, nullptr, 64);
    for (int w = 0; w < NW; ++w) {
        std::vector<std::thread> lanes;
        for (int l = 0; l < 64; ++l)
            lanes.emplace_back([=] { self = l; ifv2::pair_entries<NW>(rec, body, w, l, simd_waves); });
        for (auto &t : lanes) t.join();
    }
    pthread_barrier_destroy(&meet);
}
extern "C" void pair(int nw, int *rec, int body, const uint32_t *simd_waves) {
    if (nw == 4) run<4>((int2 *)rec, body, simd_waves);
    else if (nw == 8) run<8>((int2 *)rec, body, simd_waves);
    else run<16>((int2 *)rec, body, simd_waves);
}
"""


@pytest.fixture(scope="module")
def pair(tmp_path_factory):
    d = tmp_path_factory.mktemp("pairing")
    (d / "harness.cpp").write_text(HARNESS)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-w", "-shared", "-fPIC", "-pthread", "-I",
                           os.path.join(ROOT, "paper_2509_24663_amd", "csrc"), "-o", str(d / "h.so"), str(d / "harness.cpp")])
    lib = ctypes.CDLL(str(d / "h.so"))

    def call(nw, masks, simd_of_wave):
        """The list (block numbers 0 ..) after the pairing; the last entry is not part of it."""
        table = np.zeros(4, np.uint32)
        for w, sd in enumerate(simd_of_wave):
            table[sd] |= np.uint32(1 << w)
        rec = np.stack([np.arange(len(masks)), masks], 1).astype(np.int32)
        lib.pair(nw, rec.ctypes.data_as(ctypes.c_void_p), len(masks) - 1, table.ctypes.data_as(ctypes.c_void_p))
        return rec
    return call


PLACEMENTS = {4: [[0, 1, 2, 3], [0, 0, 1, 2], [3, 3, 3, 3]],
              8: [[0, 1, 2, 3] * 2, [0, 0, 0, 1, 1, 2, 2, 3], [2] * 8],
              16: [[0, 1, 3, 2] * 4, [0] * 6 + [1] * 4 + [2] * 4 + [3] * 2, [1] * 16]}


@pytest.mark.parametrize("nw", [4, 8, 16])
def test_every_entry_stays_in_the_list_once(pair, nw):
    rng = np.random.default_rng(nw)
    full = (1 << nw) - 1
    for n in (1, 2, nw * 4, nw * 4 + 1, nw * 5 + 2):
        for masks in (np.full(n, full), rng.integers(1, full + 1, n)):
            for simd_of_wave in PLACEMENTS[nw]:
                rec = pair(nw, masks, simd_of_wave)
                assert sorted(rec[:, 0].tolist()) == list(range(n)), (n, simd_of_wave, rec[:, 0].tolist())
                assert rec[-1, 0] == n - 1 and (rec[:, 1] == masks[rec[:, 0]]).all()
