"""A row's packed counts and the places they name in the harmonic table, on the CPU.

The two functions are compiled here as host code from the kernels' own header.  Whatever word a row
holds (counts in range, a range of -1 rows, a word that no kernel wrote), its three places lie in
[0, n]; counts in range come back as they went in."""

import os
import subprocess

from paper_1902_06828_amd import build as B

MAIN = r"""
#include <cstdio>
#include "engine.h"
using namespace mte;
int main() {
    const int ns[] = {1, 2, 9995, 1 << 20, kListMaxN};
    for (int n : ns) {
        const int in[] = {0, 1, n / 2, n - 1, n};
        for (int a : in)
            for (int b : in)
                for (int c : in) {
                    const Counts r = unpack_counts(pack_counts(a, b, c), n < kListMaxN ? n : n - 1);
                    const int top = n < kListMaxN ? n : n - 1;      // a field holds up to 2^21 - 1
                    if (a > top || b > top || c > top) continue;
                    if ((int)r.xz != a || (int)r.yz != b || (int)r.z != c) return std::printf("lost %d %d %d\n", a, b, c), 1;
                }
        // a range without the row itself, in each field: the others stay
        const Counts x = unpack_counts(pack_counts(-1, 1, 0), n), y = unpack_counts(pack_counts(1, -1, 0), n),
                     z = unpack_counts(pack_counts(0, 1, -1), n);
        if (x.xz != 0 || x.yz != 1 || x.z != 0 || y.xz != 1 || y.yz != 0 || y.z != 0 || z.xz != 0 || z.yz != 1 || z.z != 0)
            return std::printf("-1 spreads, n = %d\n", n), 1;
        uint64_t w = 0x9E3779B97F4A7C15ull;
        for (int t = 0; t < 100000; ++t, w = w * 6364136223846793005ull + 1442695040888963407ull) {
            const Counts r = unpack_counts(t == 0 ? ~0ull : w, n);
            if (r.xz > (uint32_t)n || r.yz > (uint32_t)n || r.z > (uint32_t)n) return std::printf("outside, n = %d\n", n), 1;
        }
    }
    return 0;
}
"""


def test_places_stay_in_the_table(tmp_path):
    src, exe = tmp_path / "words.cpp", tmp_path / "words"
    src.write_text(MAIN)
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    subprocess.run([B.CLANGXX, "-std=c++17", "-O1", "-I", B.CSRC, str(src), "-o", str(exe)], check=True, env=env)
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env)
    assert r.returncode == 0, r.stdout
