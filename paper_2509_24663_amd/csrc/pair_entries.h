// The order in which a tile's union list is walked (attn_mfma.hip).  Apart from the kernel so that it can be run on the
// host as well: everything here is lane arithmetic, ballots and lane reads.
#pragma once

namespace ifv2 {

// An interval holds two consecutive entries of the union list, and between its barriers a SIMD works through
// the units of the waves it hosts, so an interval lasts about as long as its busiest SIMD.  The list (all of
// it but the last entry, which stays there) is therefore re-paired: each wave takes a contiguous, even
// sized range of entries and repeatedly joins its first remaining entry to the one that raises the pair's
// busiest SIMD the least.  Partners stay a few entries apart, so the walk remains nearly ascending
// (neighbouring tiles then touch the same blocks at about the same time, which the L2 likes).
// Waves w, w + 4, w + 8, ... are taken to share a SIMD: that is how a workgroup's waves are dealt out (checked for 4, 8 and 16
// waves on idle and full chips).  The hardware's own record of it is not asked, because the order of a token's blocks, and
// with it the last bits of its result, must not depend on where the waves happened to run.
// rec: (block, token mask) per entry; body: entries in front of the last one.
template <int NW>
__device__ inline void pair_entries(int2 *rec, int body, int w, int lane) {
    const int pairs = body / 2;
    const int lo = 2 * (pairs * w / NW), hi = 2 * (pairs * (w + 1) / NW);
    const int n = hi - lo;
    if (n < 4 || n > 64) return;                        // nothing to choose / more entries than lanes: left as is
    bool live = lane < n;
    const int2 r = live ? rec[lo + lane] : make_int2(0, 0);
    uint32_t loads = 0u;                                // consumers per SIMD, one byte each
#pragma unroll
    for (int sd = 0; sd < 4; ++sd) loads |= (uint32_t)__popc((uint32_t)r.y & (0x1111u << sd)) << (8 * sd);
    auto max_byte = [](uint32_t x) -> int {
        return (int)max(max(x & 0xffu, (x >> 8) & 0xffu), max((x >> 16) & 0xffu, x >> 24));
    };
    const int own_max = max_byte(loads);
    for (int pos = lo; pos < hi; pos += 2) {
        // first: the live entry with the smallest block number, which keeps the walk close to ascending
        const int first = __ffsll((long long)__ballot(live)) - 1;
        const uint32_t lf = (uint32_t)__builtin_amdgcn_readlane((int)loads, first);
        if (lane == first) { rec[pos] = r; live = false; }
        // second: the live entry whose company costs the least beyond what it would cost alone (at most what the first one
        // costs; n is even, so there is one)
        const int extra = max_byte(lf + loads) - own_max;
        uint64_t least = 0u;
        for (int c = 0; c <= NW && least == 0u; ++c) least = __ballot(live && extra == c);
        const int second = __ffsll((long long)least) - 1;
        if (lane == second) { rec[pos + 1] = r; live = false; }
    }
}

}  // namespace ifv2
