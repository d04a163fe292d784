"""The choice of tiles of a projection launch (csrc/gemm_plan.h, host code
without HIP), compiled on its own (no GPU)."""
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_09768_amd", "csrc")
DRIVER = """
#include <cstdio>
#include "gemm_plan.h"
int main() {
  long long m, n, k;
  while (std::scanf("%lld %lld %lld", &m, &n, &k) == 3) {
    const kvc::GemmPlan p = kvc::gemm_plan(m, n, k);
    const kvc::GemmTile &B = kvc::kGemmBig[p.mode], &S = kvc::kGemmSmall[p.mode];
    std::printf("%d %lld %d %d %d %d\\n", p.mode, p.big_rows, B.rows, B.cols, S.rows, S.cols);
  }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def run(shapes):
        text = "\n".join("%d %d %d" % s for s in shapes)
        r = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True)
        return [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]
    return run


def test_plan_chooses_the_faster_tiles(plans):
    # (mode, row tiles of the larger size) that a measurement on the GPU found
    # the fastest, or within 4 % of it, where the wrong size costs 15 to 60 %
    want = {
        # narrow outputs of many rows, and short K: one or more rounds of the large tile
        (42705, 256, 1024): (0, 167), (48000, 256, 1024): (0, 188), (42705, 256, 4096): (0, 167),
        (30000, 1024, 64): (0, 118), (30000, 4096, 64): (0, 118),   # 58.8 us; 60.7 with (0, 112)
        # a few hundred rows: small tiles, alone or beside a few large ones
        (217, 3584, 18944): (2, 0), (217, 37888, 3584): (1, 1), (696, 4096, 4096): (0, 0), (696, 28672, 4096): (1, 3),
        # thousands: large tiles, small ones for the incomplete round
        (5056, 4096, 4096): (0, 16), (5056, 6144, 4096): (0, 20), (16200, 1024, 4096): (0, 64),
    }
    got = plans(list(want))
    assert {s: p[:2] for s, p in zip(want, got)} == want


def test_plan_stays_within_one_launch(plans):
    # every row has a tile and the workgroups of a launch fit HIP's limit, up
    # to the largest accepted m n (2^23 - 1 tiles of 256 x 256)
    up = lambda a, b: -(-a // b)  # noqa: E731
    rng = random.Random(1)
    shapes = [(1, 8, 64), (2 ** 31 - 256, 8, 64), (2 ** 31 - 256, 256, 64), (1, 2 ** 24, 2 ** 24)]
    for _ in range(2000):
        n = 8 * int(2 ** rng.uniform(0, 21))
        m = int(min(2 ** 31 - 128, 2 ** 39 / n, 2 ** rng.uniform(0, 31)))
        if up(m, 256) * up(n, 256) < 2 ** 23:
            shapes.append((m, n, 64 * int(2 ** rng.uniform(0, 18))))
    for (m, n, k), (mode, big_rows, br, bc, sr, sc) in zip(shapes, plans(shapes)):
        assert 0 <= big_rows <= up(m, br)
        wgs = big_rows * up(n, bc) + (up(m - big_rows * br, sr) * up(n, sc) if big_rows * br < m else 0)
        assert 0 < wgs * 512 < 2 ** 32, (m, n, k)
