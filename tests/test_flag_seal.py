"""The seal of the polled flag words, on the host: stale words never match it.

A set of words that reached memory in parts mixes words of two sets.  For sets
as consecutive runs give them, every choice of stale words (2^14 of them) has
another seal than the new set; and words that changed by the same bits, which
an exclusive or of the words alone cannot tell, do too.
"""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROG = r"""
#include <cstdint>
#include <cstdio>
#include "md_seal.h"
constexpr int N = 14;
static uint64_t seal(const uint64_t* w, uint64_t seq)
{
    uint64_t x = md::seal_mix(seq, N);
    for (int k = 0; k < N; ++k) x ^= md::seal_mix(w[k], k);
    return x;
}
int main()
{
    long bad = 0, sets = 0;
    // a run of 4 steps, then one of 5 that stopped: words 12 and 13 change by the same bit
    uint64_t was[N] = {262144, 1216, 0, 0, 0, 0, 0, 0x3F80000000000000ull, 0, 0, 0, 812, 4, 0};
    uint64_t now[N] = {262144, 1216, 0, 0, 0, 0, 0, 0x3F90000000000000ull, 0, 0, 0, 812, 5, 1};
    // after a rebuild: totals, stride and stage change, too
    uint64_t reb[N] = {262656, 1728, 0, 0, 0, 0, 0, 0, 0, 0, 0, 300, 5, 0};
    uint64_t* from[2] = {was, now};
    uint64_t* to[2] = {now, reb};
    for (int p = 0; p < 2; ++p)
        for (int m = 1; m < 1 << N; ++m) {
            uint64_t torn[N];
            bool differs = false;
            for (int k = 0; k < N; ++k) {
                torn[k] = m >> k & 1 ? from[p][k] : to[p][k];
                differs |= torn[k] != to[p][k];
            }
            if (!differs) continue;
            ++sets;
            bad += seal(torn, 7) == seal(to[p], 7);
        }
    // any two words changed by the same bits
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < i; ++j)
            for (int b = 0; b < 64; ++b) {
                uint64_t w[N];
                for (int k = 0; k < N; ++k) w[k] = now[k];
                w[i] ^= 1ull << b;
                w[j] ^= 1ull << b;
                ++sets;
                bad += seal(w, 7) == seal(now, 7);
            }
    bad += seal(now, 7) == seal(now, 8);
    std::printf("%ld %ld\n", sets, bad);
}
"""


def test_no_torn_set_matches_the_seal(tmp_path):
    src, exe = tmp_path / "seal.cpp", tmp_path / "seal"
    src.write_text(PROG)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1012_2677_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    sets, bad = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert sets > 10000 and bad == 0
