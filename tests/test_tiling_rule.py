"""The automatic tiling (paper_1102_4666_amd/csrc/bsde_tiling.h, compiled for
the host): every path is in a tile and no group is empty, no point has more than
32 groups, or more than its paths pay for, and no tile fewer than two blocks or
140 asset steps a lane unless the GPU has fewer than 2048 tiles, over sizes around
its bounds."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1102_4666_amd", "csrc")
DRIVER = r"""
#include "bsde_tiling.h"
#include <cstdio>
int main() {
    int n, M, N, d;
    while (std::scanf("%d %d %d %d", &n, &M, &N, &d) == 4) {
        int g, p;
        bsde::auto_tiling(n, M, N, d, g, p);
        std::printf("%d %d\n", g, p);
    }
}
"""
N_ = [1, 2, 9, 25, 64, 255, 256, 511, 512, 1000, 2047, 2048, 2049, 4096, 8192, 8193, 16384, 1 << 26]
M_ = [1, 255, 256, 257, 512, 513, 777, 4000, 30000, 10 ** 6, 2 ** 31 - 1]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiling")
    (d / "t.cpp").write_text(DRIVER)
    exe = str(d / "t")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, str(d / "t.cpp"), "-o", exe])

    def run(cases):
        text = "".join("%d %d %d %d\n" % c for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in ln.split()) for ln in out.splitlines()]
    return run


def test_tiles_cover_the_paths_and_stay_long(rule):
    cases = [(n, M, N, d) for n in N_ for M in M_ for N in (1, 4, 20, 50, 1000) for d in (1, 2, 5, 10)]
    for (n, M, N, d), (g, p) in zip(cases, rule(cases)):
        what = (n, M, N, d, g, p)
        blocks = -(-M // 256)
        assert g >= 1 and (g - 1) * p < blocks <= g * p, what
        fill = -(-2048 // n)
        assert g <= max(fill, 32, (M * N * d / 400) ** 0.5), what
        if g > fill:
            assert p >= 2 and p * N * d >= 140 and g * n <= 16384, what
        # and the GPU is filled where there are paths for it
        assert 3 * g >= min(fill, blocks), what
