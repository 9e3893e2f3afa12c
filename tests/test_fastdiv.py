"""The launch-time division constants of the kernels (fastdiv.h), on the CPU:
divu(make_divu32(d), n) == n / d for divisors 1..70000, every power of two and
its neighbours up to 2^32 - 1, and numerators at every edge (0, multiples of d
and their neighbours, 2^31 and 2^32 neighbours) plus seeded random ones."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2302_04741_amd",
                    "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <stdint.h>
#include "fastdiv.h"

static uint64_t rng = 88172645463325252ull;
static uint32_t next32(void) { rng ^= rng << 13; rng ^= rng >> 7; rng ^= rng << 17; return (uint32_t)rng; }

static int check(uint32_t d, uint32_t n)
{
    const lbm::DivU32 q = lbm::make_divu32(d);
    if (lbm::divu(q, n) != n / d) {
        printf("mismatch d=%u n=%u: %u vs %u\n", d, n, lbm::divu(q, n), n / d);
        return 1;
    }
    return 0;
}

static int sweep(uint32_t d)
{
    const uint32_t edge[] = {0u, 1u, 2u, d - 1u, d, d + 1u, 2u * d - 1u, 2u * d, 0x7fffffffu,
                             0x80000000u, 0x80000001u, 0xfffffffeu, 0xffffffffu};
    int bad = 0;
    for (uint32_t e : edge) bad |= check(d, e);
    const uint32_t top = 0xffffffffu / d;  // largest quotient
    bad |= check(d, top * d) | check(d, top * d - 1u) | check(d, top * d + (d - 1u));
    for (int k = 0; k < 24; ++k) bad |= check(d, next32());
    return bad;
}

int main(void)
{
    int bad = 0;
    for (uint32_t d = 1; d <= 70000u; ++d) bad |= sweep(d);
    for (int k = 1; k < 32; ++k) {
        const uint32_t p = 1u << k;
        bad |= sweep(p - 1u) | sweep(p) | sweep(p + 1u);
    }
    bad |= sweep(0xffffffffu) | sweep(0xfffffffeu) | sweep(0x80000001u);
    for (int k = 0; k < 20000; ++k) bad |= sweep(next32() | 1u);
    puts(bad ? "fastdiv: mismatches" : "fastdiv: all exact");
    return bad;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_division_constants_exact(tmp_path):
    src = tmp_path / "fastdiv_check.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "fastdiv_check"
    # the header's functions carry HIP qualifiers; on the host they are plain
    cmd = ["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-I" + CSRC, str(src),
           "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-2000:]
    assert "all exact" in run.stdout


WRAP_PROGRAM = r"""
#include <stdio.h>
#include <stdint.h>
#include "fastdiv.h"

static int check(uint32_t v, int d, uint32_t n)
{
    const int64_t want = ((int64_t(v) - d) % int64_t(n) + int64_t(n)) % int64_t(n);
    const uint32_t got = lbm::wrap_back(v, d, n);
    if (int64_t(got) == want) return 0;
    printf("mismatch v=%u d=%d n=%u: %u vs %lld\n", v, d, n, got, (long long)want);
    return 1;
}

int main(void)
{
    int bad = 0;
    for (uint32_t n = 1; n <= 300u; ++n)
        for (uint32_t v = 0; v < n; ++v)
            for (int d = -3; d <= 3; ++d) bad |= check(v, d, n);
    for (int k = 9; k <= 31; ++k)
        for (int e = -2; e <= 2; ++e) {
            const uint32_t n = (1u << k) + uint32_t(k < 31 || e < 0 ? e : 0);
            for (uint32_t o = 0; o < 8u; ++o)
                for (int d = -3; d <= 3; ++d)
                    bad |= check(o, d, n) | check(n - 1u - o, d, n) | check(n / 2u + o, d, n);
        }
    puts(bad ? "wrap: mismatches" : "wrap: all exact");
    return bad;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_periodic_wrap_exact(tmp_path):
    """wrap_back(v, d, n) == (v - d) mod n for |d| <= 3: every v of n = 1..300 (n < 4
    takes the shift modulo n), and both ends of the row up to n = 2^31."""
    src = tmp_path / "wrap_check.cpp"
    src.write_text(WRAP_PROGRAM)
    exe = tmp_path / "wrap_check"
    cmd = ["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-I" + CSRC, str(src),
           "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-2000:]
    assert "all exact" in run.stdout
