"""The FP64 fields' tanh (tanh.hpp) built with the host compiler, against the
80-bit library over its whole range: the linear part, both ends of the
reduction, the cancellation near -1, the cut at 40 and the special values.

Bar per range: 1 ulp at most (half an ulp of the result's own rounding, and of
m + ml, of dl t and of the last fma less than 2^-3 each) and a mean of 0.28
(0.25: correctly rounded).  The hardware's approximate reciprocal is replaced
by one rounded to float, 2^-24 off; two Newton steps square that twice."""
import shutil
import subprocess

import pytest

from test_f64_shape import CSRC

SRC = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include "tanh.hpp"
struct Host {
  static double rcp(double x) { return (double)(float)(1.0 / x); }
  static double exp2i(int k) { return std::ldexp(1.0, k); }
};
static double f(double x) { return bode::tanh64<Host>(x); }
int main() {
  const double R[][2] = {{1e-300, 1e-100}, {1e-100, 1e-20}, {1e-20, 1e-8},
                         {1e-8, 1e-3}, {1e-3, 0.1}, {0.1, 0.35}, {0.35, 1.0},
                         {1.0, 4.0}, {4.0, 18.0}, {18.0, 41.0}, {41.0, 1e308}};
  std::mt19937_64 g(7);
  int bad = 0;
  for (auto& r : R) {
    std::uniform_real_distribution<double> u(std::log(r[0]), std::log(r[1]));
    double most = 0, sum = 0;
    const int n = 200000;
    for (int i = 0; i < n; ++i) {
      const double x = std::exp(u(g)) * (i & 1 ? 1 : -1);
      const long double t = tanhl((long double)x);
      const double a = std::fabs((double)t);
      const long double ulp = std::ldexp(1.0L, std::ilogb(a >= 1 ? 0.9 : a) - 52);
      const double e = (double)(fabsl((long double)f(x) - t) / ulp);
      most = e > most ? e : most;
      sum += e;
    }
    std::printf("%.0e..%.0e: mean %.3f max %.3f ulp\n", r[0], r[1], sum / n,
                most);
    bad += !(most <= 1.0) || !(sum / n <= 0.28);
  }
  bad += !(f(0.0) == 0.0 && !std::signbit(f(0.0)));
  bad += !(f(-0.0) == 0.0 && std::signbit(f(-0.0)));
  bad += !(f(INFINITY) == 1.0) + !(f(-INFINITY) == -1.0);
  bad += !std::isnan(f(NAN));
  bad += !(f(5e-324) == 5e-324) + !(f(-3e-310) == -3e-310);
  bad += !(f(1.7e308) == 1.0);
  std::printf("%d over\n", bad);
  return bad != 0;
}
"""


def test_tanh64(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    subprocess.run([gxx, "-std=c++17", "-O2", "-ffp-contract=off", "-I", CSRC,
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
