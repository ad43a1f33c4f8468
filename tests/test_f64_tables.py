"""The table functions of the FP64 path kernels that take Philox words and
scaled states (paper_1102_4666_amd/csrc/bsde_f64_math.h), compiled for the
host with g++ and checked against 120-bit references (mpmath): the logarithm
by 512 bins, the square root of a positive radius, and 2^(-y^2/256) of the
bump volatility's state.  No GPU needed."""
import os
import subprocess
import tempfile

import numpy as np
import pytest

mpmath = pytest.importorskip("mpmath")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1102_4666_amd", "csrc")

DRIVER = r"""
#include "bsde_f64_math.h"
#include <cstdio>
int main() {
    static bsde::f64::Tables T;
    bsde::f64::fill_tables(T, 0, 1);
    char kind[8];
    double x;
    while (std::scanf("%7s %lf", kind, &x) == 2) {
        double v = 0;
        if (kind[0] == 'l') v = bsde::f64::log_word_tab((unsigned)x, T);
        else if (kind[0] == 'q') v = bsde::f64::sqrt_pos(x);
        else v = bsde::f64::exp2_neg_sq_tab(x, T);
        std::printf("%.17g\n", v);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver():
    d = tempfile.mkdtemp()
    src, exe = os.path.join(d, "tab.cpp"), os.path.join(d, "tab")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, src, "-o", exe])
    return exe


def _log_words():
    # random words, both ends, and the two sides of every bin's edge in the
    # first and last binades
    rng = np.random.default_rng(11)
    w = [int(v) for v in rng.integers(0, 2 ** 32, 3000, dtype=np.uint64)]
    w += list(range(0, 66)) + [2 ** 32 - 1 - k for k in range(66)]
    w += [2 ** 31 + (j << 22) + o for j in range(512) for o in (-1, 0, 1)]
    w += [2 ** 12 + (j << 3) + o for j in range(512) for o in (-1, 0, 1)]
    return w


CASES = {
    "log": ("l", _log_words, lambda w: mpmath.log((mpmath.mpf(w) + mpmath.mpf(0.5)) / 2 ** 32)),
    "sqrt": ("q", lambda: list(10.0 ** np.random.default_rng(12).uniform(-240, 30, 3000)) +
             [2.0 ** -800, 0.25, 1.0, 2.0, 4.0, 49.0], lambda x: mpmath.sqrt(mpmath.mpf(x))),
    "bump": ("b", lambda: list(np.random.default_rng(13).uniform(-511, 511, 2000)) +
             list(np.random.default_rng(14).uniform(-60, 60, 2000)) +
             # halfway between integers of y^2, where the series argument is largest
             [float(np.sqrt(k + 0.5)) * s for k in range(0, 600, 7) for s in (1, -1)] +
             [0.0, -0.0, 1e-160, 510.99999999999994, 511.0],
             lambda y: mpmath.power(2, -mpmath.mpf(y) ** 2 / 256)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_table_function_within_two_ulp(driver, name):
    # 1.5 ulp for the functions of one table product, 2 for the logarithm's
    # three-term sum: the bounds of the functions they stand beside
    mpmath.mp.prec = 120
    kind, xs, ref = CASES[name]
    xs = xs()
    out = subprocess.run([driver], input="\n".join("%s %.17g" % (kind, x) for x in xs),
                         capture_output=True, text=True, check=True).stdout.split()
    worst = 0.0
    for x, v in zip(xs, out):
        r = ref(x)
        worst = max(worst, float(abs(mpmath.mpf(float(v)) - r)) / np.spacing(abs(float(r))))
    assert worst <= {"log": 2.0, "sqrt": 1.0, "bump": 1.5}[name], worst


def test_bump_beyond_its_clamp(driver):
    # |y| >= 511 stays at 2^(-511^2/256), a normal number far below the
    # volatility's rounding
    out = subprocess.run([driver], input="b 512\nb -1e12\nb 1e300", capture_output=True,
                         text=True, check=True).stdout.split()
    for v in out:
        assert float(v) == pytest.approx(2.0 ** (-(511.0 ** 2) / 256), rel=1e-14)
