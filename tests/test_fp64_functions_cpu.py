"""The elementary functions of the FP64 paths (csrc/path_fp64.hpp), compiled for
the CPU from the source itself, against long double: the logarithm and the sine
and cosine at every 23-bit uniform, exp(-a) over the arguments of the bridge
test, reciprocal and square root over the magnitudes that paths meet.  The
device's reciprocal and reciprocal square root estimates are stood in for by
the exact values off by 2^-20 either way.

Bars (relative, u = 2^-53), from the steps of each function:
  log   3.2e-16: the nearest argument to 1 takes 2.1 u; below sqrt(1/2), at
        |result| >= 0.347, the constant ln 2 (2.3e-17), the quotient (4.2e-17)
        and the last rounding
  cos, sin  3.6e-16: polynomial 1e-16, its last step and the product u each
  exp   2.5e-16: the reduced argument and the two sums
  1/b, sqrt  1.2e-16: the last rounding of a corrected estimate."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_1504_00084_amd", "csrc", "path_fp64.hpp")
BARS = {"log": 3.2e-16, "cos": 3.6e-16, "sin": 3.6e-16, "exp": 2.5e-16, "rcp": 1.2e-16, "sqrt": 1.2e-16}

MAIN = r"""
static long double worst(long double got, long double want, long double w)
{
    const long double e = fabsl(got / want - 1.0L);
    return e > w || e != e ? e : w;
}
int main()
{
    long double e_log = 0, e_cos = 0, e_sin = 0, e_exp = 0, e_rcp = 0, e_sqrt = 0;
    for (int sign = -1; sign <= 1; sign += 2) {
        g_off = sign * 0x1p-20;
        for (uint32_t k = 0; k < (1u << 23); ++k) {
            const uint32_t w = (k << 9) | (k & 511u);   // the low nine bits are not used
            const uint32_t m = 2u * k + 1u;
            e_log = worst(log_u(w), logl((long double)m * 0x1p-24L), e_log);
            if (sign > 0) continue;
            const uint32_t q = (m + (1u << 21)) >> 22;   // exact quarter turns, and the rest
            const long double r = (long double)((int)m - (int)(q << 22)) * 0x1p-22L * 1.57079632679489661923132169163975L;
            const long double c = cosl(r), s = sinl(r);
            const long double want_c[4] = {c, -s, -c, s}, want_s[4] = {s, c, -s, -c};
            double cs, sn;
            cos_sin_u(w, cs, sn);
            e_cos = worst(cs, want_c[q & 3u], e_cos);
            e_sin = worst(sn, want_s[q & 3u], e_sin);
        }
        for (int k = 0; k <= 2000000; ++k) {
            const double t = k * 0x1p-21 * 1.0485759;   // 0 .. 1
            const double b = std::exp2(40.0 * t - 20.0) * (1.0 + 1e-9 * (k % 1000));
            e_rcp = worst(rcp64(b), 1.0L / b, e_rcp);
            e_sqrt = worst(sqrt64(b), sqrtl(b), e_sqrt);
            if (sign < 0) e_exp = worst(exp_neg(50.0 * t), expl(-(long double)(50.0 * t)), e_exp);
        }
    }
    if (exp_neg(0.0) != 1.0 || !(exp_neg(1e300) >= 0.0 && exp_neg(1e300) < 1e-300)) e_exp = 1;
    printf("log %.3Le\ncos %.3Le\nsin %.3Le\nexp %.3Le\nrcp %.3Le\nsqrt %.3Le\n", e_log, e_cos, e_sin, e_exp, e_rcp, e_sqrt);
}
"""


@pytest.fixture(scope="module")
def errors(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    text = open(HEADER).read()
    body = text[text.index("// Elementary functions"):text.index("// Constants, path state")]
    body, n = re.subn(r'asm volatile\(""[^;]*;', "", body)   # a hint to the device's register allocation
    assert n == 1
    src = os.path.join(str(tmp_path_factory.mktemp("fn")), "fn.cpp")
    with open(src, "w") as f:
        f.write("""#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <algorithm>
using std::fma; using std::fmin; using std::rint; using std::ldexp;
#define __device__
#define __forceinline__ inline
static double g_off;
static double __builtin_amdgcn_rcp(double b) { return 1.0 / b * (1.0 + g_off); }
static double __builtin_amdgcn_rsq(double b) { return 1.0 / std::sqrt(b) * (1.0 + g_off); }
static uint32_t __float_as_uint(float f) { uint32_t u; std::memcpy(&u, &f, 4); return u; }
static float __uint_as_float(uint32_t u) { float f; std::memcpy(&f, &u, 4); return f; }
static uint64_t bits(double d) { uint64_t u; std::memcpy(&u, &d, 8); return u; }
static int __double2hiint(double d) { return (int)(bits(d) >> 32); }
static int __double2loint(double d) { return (int)bits(d); }
static double __hiloint2double(int h, int l)
{
    const uint64_t u = (uint64_t)(uint32_t)h << 32 | (uint32_t)l;
    double d;
    std::memcpy(&d, &u, 8);
    return d;
}
""" + body + MAIN)
    exe = src[:-4]
    res = subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", src, "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    out = subprocess.run([exe], capture_output=True, text=True, check=True, timeout=600).stdout
    return {ln.split()[0]: float(ln.split()[1]) for ln in out.splitlines()}


@pytest.mark.parametrize("name", sorted(BARS))
def test_function_error(errors, name):
    print("%s: %.3e of %.1e" % (name, errors[name], BARS[name]))
    assert errors[name] <= BARS[name]
