"""The plates' densities are correctly rounded quotients: quotient(m, d, 1.0 / d) of
fastdiv.h is m / d, bit for bit (a product with the rounded reciprocal misses the last
bit of about a quarter of them).  m and d over the values densities take and over their
neighbourhood of ones and powers of two."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2302_04741_amd",
                    "csrc")

PROGRAM = r"""
#include <math.h>
#include <stdio.h>
#include <stdint.h>
#include "fastdiv.h"

static uint64_t rng = 88172645463325252ull;
static uint64_t next64(void) { rng ^= rng << 13; rng ^= rng >> 7; rng ^= rng << 17; return rng; }
static double uniform(double lo, double hi) { return lo + (hi - lo) * double(next64() >> 11) * 0x1p-53; }

int main(void)
{
    long bad = 0, product = 0;
    const long n = 4000000;
    for (long k = 0; k < n; ++k) {
        double d = uniform(0.05, 3.0), m = uniform(0.0, 4.0);
        if (k % 4 == 1) d = nextafter(ldexp(1.0, int(next64() % 9) - 4), k % 8 < 4 ? 0.0 : 9e9);
        if (k % 4 == 2) m = -m;
        if (k % 4 == 3) m = d * ldexp(1.0 + double(next64() % 5) * 0x1p-52, int(next64() % 21) - 10);
        const double inv = 1.0 / d;
        bad += lbm::quotient(m, d, inv) != m / d;
        product += m * inv != m / d;
    }
    printf("%ld of %ld differ, of the products %ld\n", bad, n, product);
    return bad != 0 || product == 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_quotient_is_the_rounded_quotient(tmp_path):
    src = tmp_path / "quotient_check.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "quotient_check"
    cmd = ["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-D__host__=", "-D__device__=",
           "-I" + CSRC, str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-2000:]
