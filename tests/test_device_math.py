"""The kernels' own logarithm, exponential and reciprocal against 80-bit
references (CPU): physics.hpp compiled with g++, the hardware instructions they
start from replaced by their definitions, the reciprocal estimate by one that is
off by as much as the instruction may be (2^29 ulp) and twice that, either way.

Bounds, in ulps of 2^-52: the reciprocal's last Newton step leaves one rounding
of the product and one of the sum, 1; ln, relative to max(1, |ln x|), the
roundings of s (1), of the polynomial's last product and of the sum, 1.5; the
exponential the reduced argument's (1/2) and two of the last two steps, 1.5.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2108_07605_amd", "csrc")

SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <limits>
static double g_off = 0.0;
static inline double est_rcp(double x) { return (1.0 / x) * (1.0 + g_off); }
static inline double est_mant(double x) { int e; return std::frexp(x, &e); }
static inline int est_exp(double x) { int e; std::frexp(x, &e); return e; }
#define __builtin_amdgcn_rcp est_rcp
#define __builtin_amdgcn_frexp_mant est_mant
#define __builtin_amdgcn_frexp_exp est_exp
#define __builtin_amdgcn_ldexp std::ldexp
#include "physics.hpp"
using namespace rlbm;
static double uni() { return std::rand() / (RAND_MAX + 1.0); }
int main() {
    const long double ulp = 0x1p-52L;
    long double e_rcp = 0, e_ln = 0, e_exp = 0;
    const double offs[] = {0.0, 0x1p-23, -0x1p-23, 0x1p-22, -0x1p-22};
    for (double off : offs) {
        g_off = off;
        for (int k = 0; k < 400000; ++k) {
            // the whole normal range, and densely around what the kernels meet
            const double x = std::exp2(k & 1 ? 2000.0 * uni() - 1000.0 : 12.0 * uni() - 6.0) * (1.0 + uni());
            e_rcp = std::fmax(e_rcp, std::fabs((long double)recip(x) * x - 1.0L));
            e_rcp = std::fmax(e_rcp, std::fabs((long double)recip(-x) * -x - 1.0L));
            const long double l = std::log((long double)x);
            e_ln = std::fmax(e_ln, std::fabs(ln(x) - l) / std::fmax(1.0L, std::fabs(l)));
            const double y = k & 1 ? 1400.0 * uni() - 700.0 : 4.0 * uni() - 2.0;
            const long double r = std::exp((long double)y);
            e_exp = std::fmax(e_exp, std::fabs(expo(EXP_E, y) - r) / r);
        }
        for (double x : {0.70710678118654746, 0.70710678118654757, 1.0, std::nextafter(1.0, 0.0), std::nextafter(1.0, 2.0), 2.0})
            e_ln = std::fmax(e_ln, std::fabs(ln(x) - std::log((long double)x)));
    }
    g_off = 0.0;
    const double inf = std::numeric_limits<double>::infinity(), nan = std::nan("");
    const bool edges = ln(1.0) == 0.0 && expo(EXP_E, 0.0) == 1.0 && expo(EXP_E, -inf) == 0.0 && expo(EXP_E, inf) == inf &&
                       expo(EXP_E, 800.0) == inf && expo(EXP_E, -800.0) == 0.0 && std::isnan(expo(EXP_E, nan)) &&
                       std::isnan(ln(-1.0)) && std::isnan(ln(0.0)) && std::isnan(ln(nan));
    std::printf("%.3Lf %.3Lf %.3Lf %d\n", e_rcp / ulp, e_ln / ulp, e_exp / ulp, (int)edges);
}
"""


def test_ln_exp_and_reciprocal_over_their_range(tmp_path):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not shutil.which("g++") or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    src, exe = tmp_path / "math.cpp", tmp_path / "math"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include", f"-I{CSRC}",
                    f"-I{ROOT}/include", str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    rcp, ln, exp = map(float, out[:3])
    assert rcp <= 1.0 and ln <= 1.5 and exp <= 1.5 and out[3] == "1", out
