"""The tiles of the 4-cycle apex lists over every graph size the header accepts
(no GPU): tiles cover the ids, and the packed sizes of a tile hold for every
mix of the three classes, a whole tile of one class included."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "list_tiles.h"
using namespace gpm;
static int bad(const char *what, long long n, int k) {
    std::printf("%s: n = %lld, class %d\n", what, n, k);
    return 1;
}
int main() {
    const long long most = INT32_MAX - 1;
    for (long long n = 1; n <= most; n = n < 100000 ? n + 1 : n + n / 997 + 1) {
        for (long long m : {n, most - n + 1}) {
            const int64_t t = list_tile((int32_t)m);
            if (t < 1 || t % kListTile) return bad("step", m, 0);
            if ((m + t - 1) / t > kListTiles) return bad("tiles", m, 0);
            for (int k = 0; k < 3; k++) {
                // the sizes of a whole tile of class k, and of one that misses
                // an id to each of the others
                const uint64_t all = (uint64_t)t * one_of_class(k);
                uint64_t mix = (uint64_t)(t - 2) * one_of_class(k);
                for (int q = 0; q < 3; q++) mix += q == k ? 0 : one_of_class(q);
                for (int q = 0; q < 3; q++) {
                    if (ids_of_class(all, q) != (q == k ? (uint32_t)t : 0u)) return bad("all", m, k);
                    if (ids_of_class(mix, q) != (q == k ? (uint32_t)t - 2u : 1u)) return bad("mix", m, k);
                }
            }
        }
    }
    return 0;
}
"""


def test_tiles_of_every_accepted_size(tmp_path):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2011_03135_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
