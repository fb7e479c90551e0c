"""The square root's Newton steps (host build of the device header): sqrt(x) and 1 / (2 sqrt(x)) from
estimates off by up to 2^-23 either way, over mantissas and exponents, against 80-bit arithmetic.  The
bounds are those of correctly rounded operations: half an ulp for g; for h half an ulp on top of g's,
which counts up to one in ulps of h (g just above a power of two, h just below one).
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = r"""
#include "fr_scalar.hpp"
#include <cmath>
#include <cstdio>
static double ulps(double got, long double want) {
    const double w = (double)want;
    return (double)(fabsl(got - want) / (std::nextafter(w, INFINITY) - w));
}
int main() {
    unsigned long long s = 88172645463325252ull;
    auto next = [&] { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return (double)(s >> 11) * 0x1p-53; };
    double eg = 0, eh = 0;
    for (int i = 0; i < 400000; ++i) {
        const double x = std::ldexp(1.0 + next(), i % 5 ? (int)(next() * 4) - 2 : (int)(next() * 1000) - 500);
        const double y = (double)((1.0L + (2.0L * next() - 1.0L) * 0x1p-23L) / sqrtl((long double)x));
        double g, h;
        sqrt_steps(x, y, g, h);
        const long double q = sqrtl((long double)x);
        eg = std::fmax(eg, ulps(g, q));
        eh = std::fmax(eh, ulps(h, 0.5L / q));
    }
    printf("%.4f %.4f\n", eg, eh);
    return 0;
}
"""


def test_square_root_and_half_reciprocal(tmp_path):
    if shutil.which(HIPCC) is None:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "steps.hip", tmp_path / "steps"
    src.write_text(SOURCE)
    build = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-ffp-contract=off", "-I",
                            os.path.join(ROOT, "paper_1903_06304_amd", "csrc"), str(src), "-o", str(exe)],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stderr[-1000:]
    g, h = map(float, run.stdout.split())
    print(f"[steps] sqrt {g} ulp, half reciprocal {h} ulp", flush=True)
    assert g <= 0.51 and h <= 1.51
