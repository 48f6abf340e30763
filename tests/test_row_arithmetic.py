"""The row formation's reciprocal, quotient and square root without the
scaling and special cases of the general operations: an estimate, refined by
FMA, then corrected by the exact residual.  The voxel lists are bit-exact
against the oracle only if they are the IEEE results.

Checked on the host, in C with the C library's correctly rounded fma, from
estimates as poor as the hardware's bound allows (2^-23 relative error), for
random operands and for the hard ones: quotients next to the midpoint of two
doubles and squares next to a double's square."""
import os
import shutil
import subprocess

import pytest

SRC = r"""
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
static uint64_t s = 88172645463325252ull;
static uint64_t nx(void) { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return s; }
static double est(double v) { return v * (1.0 + ((double)(int64_t)nx() / 9.3e18) * 0x1p-23); }
static double make(int range)
{
    uint64_t u = nx(), e = 1023 - range / 2 + (u >> 53) % range;
    u = (e << 52) | (u & ((1ull << 52) - 1));
    double v;
    memcpy(&v, &u, 8);
    return v;
}
static double next(double v, int k)
{
    uint64_t u;
    memcpy(&u, &v, 8);
    u += (uint64_t)(int64_t)k;
    memcpy(&v, &u, 8);
    return v;
}
static double refine(double b)
{
    double y = est(1.0 / b);
    y = fma(fma(-b, y, 1.0), y, y);
    return fma(fma(-b, y, 1.0), y, y);
}
static double recip_rn(double b)
{
    double y = refine(b);
    return fma(fma(-b, y, 1.0), y, y);
}
static double quot_rn(double a, double b)
{
    double y = refine(b), q = a * y;
    return fma(fma(-b, q, a), y, q);
}
static double sqrt_rn(double x)
{
    double y = est(1.0 / sqrt(x)), g = x * y, h = 0.5 * y, r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return fma(fma(-g, g, x), h, g);
}
int main(void)
{
    long bad[5] = {0, 0, 0, 0, 0};
    for (long i = 0; i < 3000000; i++) {
        double b = make(600), a = make(300), c = make(40), q = make(4);
        bad[0] += recip_rn(b) != 1.0 / b;
        bad[1] += quot_rn(a, c) != a / c;
        double hi = q * c, lo = fma(q, c, -hi), half = 0.5 * (next(q, 1) - q);
        double m = next(hi + (lo + half * c), (int)(nx() % 5) - 2);
        bad[2] += quot_rn(m, c) != m / c;
        bad[3] += sqrt_rn(b) != sqrt(b);
        double t = next(q * q, (int)(nx() % 7) - 3);
        bad[4] += sqrt_rn(t) != sqrt(t);
    }
    printf("%ld %ld %ld %ld %ld\n", bad[0], bad[1], bad[2], bad[3], bad[4]);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
def test_refined_estimates_give_the_ieee_results(tmp_path):
    c, exe = os.path.join(tmp_path, "a.c"), os.path.join(tmp_path, "a")
    with open(c, "w") as fh:
        fh.write(SRC)
    subprocess.check_call(["gcc", "-O2", "-ffp-contract=off", "-mfma", "-o", exe, c, "-lm"])
    assert subprocess.check_output([exe], text=True).split() == ["0"] * 5
