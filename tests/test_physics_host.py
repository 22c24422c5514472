"""The power of the temperature ratio in the line widths (physics.h), compiled for the host,
against 80-bit arithmetic. The C library's exp is within 0.52 units in the last place and the last
product adds half a unit; a unit is at most 2^-52 of the value, and the logarithm's own error (2^-59
of it, |n ln t| < 5) is below 2^-56: together below 2.2 times 2^-53 (2.1 is asked for)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include "physics.h"
int main() {
  std::mt19937_64 r(7);
  std::uniform_real_distribution<double> T(50.0, 5000.0), N(-0.6, 1.6);
  long double worst = 0.0L, log_worst = 0.0L;
  for (int i = 0; i < 400000; ++i) {
    const double t = i == 0 ? 1.0 : i == 1 ? 0x1.fffffffffffffp-1 : i == 2 ? 0x1.0000000000001p0
                                                                    : 296.0 / T(r);
    const double n = (float)N(r);
    double hi, lo;
    xs::log_two(t, &hi, &lo);
    const long double l = logl((long double)t);
    if (l != 0.0L) log_worst = fmaxl(log_worst, fabsl(((long double)hi + lo - l) / l));
    const long double p = powl((long double)t, (long double)n);
    worst = fmaxl(worst, fabsl(((long double)xs::power_ln(n, hi, lo) - p) / p));
  }
  std::printf("%.4Lf %.4Lg\n", worst * 0x1p53L, log_worst);
  return 0;
}
"""


def test_power_of_the_temperature_ratio(tmp_path):
    cxx = shutil.which("g++")
    inc = "/opt/rocm/include"
    if not cxx or not os.path.isdir(inc):
        pytest.skip("no host compiler or HIP headers")
    src = tmp_path / "power.cpp"
    src.write_text(SOURCE)
    exe = tmp_path / "power"
    subprocess.run([cxx, "-O2", "-std=c++17", "-ffp-contract=off", "-mfma",
                    "-D__HIP_PLATFORM_AMD__=1", "-I" + inc,
                    "-I" + os.path.join(ROOT, "paper_2510_20870_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True, capture_output=True, text=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    print("[power]", out)
    assert float(out[0]) < 2.1
    # 64 bits of the reference's logarithm are 2^-64; 2^-59 leaves both roundings of lo room
    assert float(out[1]) < 2.0 ** -59
