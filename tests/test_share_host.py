"""Dealing out pieces to workgroups in 32 bits (dfk_share.h), compiled for the host, against Python's integers."""
import os
import random
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include <cstdio>
#include "dfk_share.h"
int main() {
    unsigned n, S, s; int i;
    while (scanf("%u %u %u %d", &n, &S, &s, &i) == 4) {
        int lo, hi;
        dfk::share_of(n, S, s, lo, hi);
        printf("%d %d %d\\n", lo, hi, dfk::share_with((int)n, (int)S, i));
    }
}
"""


def test_shares_in_32_bits(tmp_path):
    exe = str(tmp_path / "share")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2602_11808_amd", "csrc"), "-x", "c++", "-", "-o", exe],
                   input=SRC, text=True, check=True)
    rng = random.Random(3)
    edge = [1, 2, 3, 7, 8, 255, 256, 257, 512, 65534, 65535, 65536, 65537, 1 << 20, (1 << 28) - 1]
    rows = [(n, S, s) for n in edge for S in edge if S <= min(n, 65535) for s in {0, 1, S // 2, S - 1} if s < S]
    rows += [(n, S, rng.randrange(S)) for n, S in ((n, rng.randint(1, min(n, 65535))) for n in (int(2 ** rng.uniform(0, 28)) for _ in range(4000)))]
    rows = [(n, S, s, rng.randrange(n)) for n, S, s in rows]
    out = subprocess.run([exe], input="".join("%d %d %d %d\n" % r for r in rows), capture_output=True, text=True, check=True).stdout.split("\n")
    for (n, S, s, i), line in zip(rows, out):
        lo, hi, at = map(int, line.split())
        assert (lo, hi) == (n * s // S, n * (s + 1) // S), (n, S, s)
        assert n * at // S <= i < n * (at + 1) // S, (n, S, i, at)
