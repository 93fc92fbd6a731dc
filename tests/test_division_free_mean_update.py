"""The LayerNorm kernel replaces the division d/i of the running-mean update (Eq. 5) by
    t = RN(d*lo),  q = RN(d*hi + t) (one FMA),   hi = RN(1/i), lo = RN(1/i - hi),
which is only legitimate if it returns the bits of the IEEE division for every deviation that the
kernel does not send to the division: d = 0 and 2^-98 <= |d| with a finite quotient.  The proof is at
the table in the source; this file re-checks a slice of that space on every run (all divisors the
table holds, a few thousand significands each, the extreme ones included, at both ends of the
exponent range, where d*lo is subnormal or d is next to the largest number) with a small C program,
so a change of the scheme cannot go unnoticed.  The check is arithmetic on the host: it shares
nothing with the kernel but the formula.  The one-number form with a remainder step,
    q0 = RN(d*rk),  r = d - q0*i (one FMA, exact),  q = RN(q0 + r*rk),   rk = RN(1/i),
is checked beside it: the same quotient from a table of half the size, one more dependent step."""
import os
import subprocess
import tempfile

SRC = r"""
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
int main(void) {
    long long bad = 0, n = 0;
    uint32_t lcg = 12345u;
    for (int k = 1; k <= 4096; ++k) {
        const float kf = (float)k, rk = 1.0f / kf;
        for (int s = 0; s < 6000; ++s) {
            uint32_t m;
            if (s < 64) m = (uint32_t)s;                          /* smallest significands   */
            else if (s < 128) m = (1u << 23) - 1u - (uint32_t)(s - 64);   /* largest           */
            else { lcg = lcg * 1664525u + 1013904223u; m = lcg >> 9; }
            uint32_t bits = 0x3F800000u | m;
            float a; memcpy(&a, &bits, 4);
            for (int e = -60; e <= 60; e += 60) {                 /* the exponent only scales */
                const float d = ldexpf(a, e);
                const float want = d / kf;
                const float q0 = d * rk;
                const float r = fmaf(-q0, kf, d);
                const float q = fmaf(r, rk, q0);
                bad += (q != want); ++n;
            }
        }
    }
    printf("%lld %lld\n", n, bad);
    return bad != 0;
}
"""


def test_corrected_reciprocal_multiply_equals_ieee_division():
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "chk.c"), os.path.join(d, "chk")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.run(["gcc", "-O2", "-ffp-contract=off", "-march=native", src, "-o", exe, "-lm"], check=True)
        out = subprocess.run([exe], capture_output=True, text=True)
        n, bad = (int(v) for v in out.stdout.split())
        assert out.returncode == 0 and bad == 0 and n == 4096 * 6000 * 3


EXPONENTS = [-98, -97, -60, 0, 60, 126, 127]
SRC_TWO_STEP = SRC.replace("const float kf = (float)k, rk = 1.0f / kf;",
                           "const float kf = (float)k, hi = 1.0f / kf, lo = (float)((1.0 - (double)hi * k) / k);") \
    .replace("for (int e = -60; e <= 60; e += 60) {                 /* the exponent only scales */",
             "const int es[] = {%s}; for (int ei = 0; ei < %d; ++ei) { const int e = es[ei];"
             % (", ".join(map(str, EXPONENTS)), len(EXPONENTS))) \
    .replace("const float q0 = d * rk;", "const float t = d * lo;") \
    .replace("const float r = fmaf(-q0, kf, d);", "") \
    .replace("const float q = fmaf(r, rk, q0);", "const float q = fmaf(d, hi, t);")


def test_two_step_quotient_equals_ieee_division():
    """The form the kernel runs: 1/i as a sum hi + lo of two fp32 numbers, t = RN(d*lo), q = RN(d*hi + t)."""
    assert "fmaf(d, hi, t)" in SRC_TWO_STEP and "rk" not in SRC_TWO_STEP and "es[ei]" in SRC_TWO_STEP
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "chk.c"), os.path.join(d, "chk")
        with open(src, "w") as f:
            f.write(SRC_TWO_STEP)
        subprocess.run(["gcc", "-O2", "-ffp-contract=off", "-march=native", src, "-o", exe, "-lm"], check=True)
        out = subprocess.run([exe], capture_output=True, text=True)
        n, bad = (int(v) for v in out.stdout.split())
        assert out.returncode == 0 and bad == 0 and n == 4096 * 6000 * len(EXPONENTS)
