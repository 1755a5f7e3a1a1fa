"""What the 256-token pair launches of a configuration (dfk_big_plan.h), compiled for the host: both sides of every line of its rules."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include <cstdio>
#include "dfk_big_plan.h"
int main() {
    int what, m, ff, splits, k2c, wdt, summed;
    while (scanf("%d %d %d %d %d %d %d", &what, &m, &ff, &splits, &k2c, &wdt, &summed) == 7) {
        const dfk::BigLaunch l = what == 0 ? dfk::big_gateup_launch(m, ff, splits) : dfk::big_down_launch(m, ff, splits, k2c, wdt, summed);
        printf("%d %d %d %d\\n", l.splits, l.groups, l.tokens, l.row);
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2602_11808_amd", "csrc"), "-x", "c++", "-", "-o", exe],
                   input=SRC, text=True, check=True)

    def run(rows):
        text = "".join("%d %d %d %d %d %d %d\n" % r for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [tuple(map(int, l.split())) for l in out if l]
    return run


def gateup(m, ff, splits):
    return (0, m, ff, splits, 1, 0, 1)


def down(m, ff, splits, k2c, wdt=0, summed=1):
    return (1, m, ff, splits, k2c, wdt, summed)


# tokens, d_ff, configured slices -> slices, groups, tokens per group
GATEUP = [(64, 1024, 128, (128, 1, 64)), (65, 3072, 256, (128, 2, 64)), (65, 3080, 256, (256, 1, 65)), (128, 3072, 256, (128, 2, 64)), (129, 3080, 256, (128, 2, 128)),
          (192, 4096, 256, (128, 2, 128)), (192, 4104, 256, (256, 1, 192)), (193, 4104, 256, (128, 2, 128)), (256, 8192, 256, (128, 2, 128)), (256, 8200, 256, (256, 1, 256)),
          (100, 512, 64, (64, 2, 64)), (100, 1024, 512, (512, 1, 100)),       # fewer slices than half a round stay; more than a round are no groups
          # the wide form: up to 16, 14 and 10 row tiles; one slice of nine; rounds where one does not do; nothing to gain; not for one token tile
          (65, 16384, 256, (256, 1, 65)), (65, 16392, 512, (256, 1, 65)), (128, 32768, 512, (256, 1, 128)), (128, 32776, 768, (512, 1, 128)),
          (129, 28672, 512, (256, 1, 129)), (192, 28680, 512, (512, 1, 192)), (192, 53248, 1024, (512, 1, 192)), (193, 20480, 512, (256, 1, 193)),
          (256, 20488, 512, (512, 1, 256)), (64, 20480, 512, (512, 1, 64)), (150, 28672, 256, (256, 1, 150))]
# tokens, d_ff, configured splits, column blocks, W_down as [d_model, d_ff], summed by a launch -> splits, groups, tokens per group
DOWN = [(64, 1024, 16, 4, 0, 1, (16, 1, 64)), (65, 1024, 16, 4, 0, 1, (16, 2, 64)), (128, 1024, 12, 8, 0, 1, (12, 2, 64)), (193, 1024, 8, 8, 0, 1, (8, 4, 64)),
        (256, 1024, 8, 8, 0, 1, (8, 4, 64)), (256, 1024, 8, 9, 0, 1, (8, 2, 128)), (256, 5376, 8, 16, 0, 1, (8, 2, 128)), (256, 5376, 8, 17, 0, 1, (8, 1, 256)),
        (129, 4096, 4, 32, 0, 1, (4, 2, 128)), (129, 4104, 4, 32, 0, 1, (4, 1, 129)), (128, 4096, 4, 32, 0, 1, (4, 1, 128)), (128, 4096, 4, 32, 1, 1, (4, 2, 64)),
        (128, 4096, 4, 33, 1, 1, (4, 1, 128)), (256, 1024, 8, 8, 0, 0, (8, 1, 256)),
        # bytes of W_down: 20 MB and a little more, 32 and 64 MB and a little more
        (129, 20480, 8, 4, 0, 1, (8, 3, 64)), (129, 20488, 8, 4, 0, 1, (8, 2, 128)), (192, 8192, 8, 16, 0, 1, (8, 2, 128)), (192, 8200, 8, 16, 0, 1, (8, 1, 192)),
        (193, 8200, 8, 16, 0, 1, (8, 2, 128)), (193, 16384, 8, 16, 0, 1, (8, 2, 128)), (193, 16392, 8, 16, 0, 1, (8, 1, 193)),
        # more splits than fit: as many as 128, 80 and 64 workgroups a group make, then the next that cuts d_ff into whole 64-row steps
        (128, 5504, 16, 9, 0, 1, (14, 2, 64)), (128, 9216, 16, 13, 0, 1, (9, 2, 64)), (160, 12288, 24, 7, 0, 1, (16, 2, 128)), (160, 4864, 15, 7, 0, 1, (11, 3, 64)),
        (160, 3840, 12, 8, 0, 1, (10, 3, 64)), (250, 3840, 12, 8, 0, 1, (6, 4, 64)), (250, 3840, 12, 8, 1, 1, (8, 4, 64)), (100, 2560, 14, 5, 0, 1, (14, 2, 64))]


def test_lines_of_the_rules(ask):
    rows = [gateup(*c[:3]) for c in GATEUP] + [down(*c[:6]) for c in DOWN]
    for c, got in zip(GATEUP + DOWN, ask(rows)):
        assert got[:3] == c[-1], (c, got)


def test_every_launch_covers_the_tokens_and_stays_within_its_limits(ask):
    rng = random.Random(11)
    rows = []
    for _ in range(4000):
        m, ff = rng.randint(1, 256), 8 * rng.randint(1, 7000)
        splits = min(ff // 8, rng.choice([1, 64, 128, 200, 256, 512, -(-ff // 64), 1024]))
        k2c = rng.randint(1, 256)
        rows += [gateup(m, ff, splits), down(m, ff, min(ff // 8, rng.randint(1, 512)), k2c, rng.randint(0, 1), rng.randint(0, 1))]
    for r, (splits, groups, tokens, row) in zip(rows, ask(rows)):
        assert 1 <= splits <= r[3] and groups * tokens >= r[1] > (groups - 1) * tokens, (r, splits, groups, tokens)
        assert groups == 1 and tokens == r[1] or tokens % 64 == 0, (r, tokens)
        work = splits * r[4]
        assert row == work if groups == 1 or r[0] == 0 else row == -(-work // 8) * 8, (r, splits, groups, row)
        if r[0] == 0:
            tiles = -(-(r[2] // 8) // splits)
            if -(-(r[2] // 8) // r[3]) <= 8:       # what a valid configuration has
                assert tiles <= (8 if groups > 1 or splits == r[3] else (0, 0, 16, 14, 10)[-(-tokens // 64)]), (r, splits, groups)
        elif groups > 1 and splits > 1:
            assert splits == r[3] or row // 8 * groups <= 32, (r, splits, groups)      # workgroups of an XCD with 32 CUs
