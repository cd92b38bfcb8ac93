"""The NS relaxation of a node (tau_g of eq:N21_1) against extended precision,
on the CPU.  With u = 2^-53 the rounding unit: 3 mu / rho takes two roundings,
its reciprocal a third (3 u); 1/2 + 3 mu / rho adds one to an error of at most
2 u, and its reciprocal another (4 u); 1 - 1 / (2 tau_g) one more, of values
below 1 (4 u / (2 tau_g) + u)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include "relaxation.h"
int main() {
  const long double u = 0x1p-53L;
  std::mt19937_64 g(1904);
  std::uniform_real_distribution<double> U(0.0, 1.0);
  double w[3] = {0, 0, 0};
  for (int i = 0; i < 4000000; ++i) {
    const double rho = std::exp(U(g) * 7 - 3), mu = rho * std::pow(10.0, 5 * U(g) - 4);
    const long double tm = 3.0L * mu / rho, it = 1 / (0.5L + tm), th = 1 / tm;
    double itau, srcg, theta;
    nplbm::ns_relaxation(mu, rho, 1.0 / rho, itau, srcg, theta);
    w[0] = std::max(w[0], (double)(fabsl(itau - it) / (it * u)));
    w[1] = std::max(w[1], (double)(fabsl(srcg - (1 - 0.5L * it)) / ((2 * it + 1) * u)));
    w[2] = std::max(w[2], (double)(fabsl(theta - th) / (th * u)));
  }
  std::printf("%.3f %.3f %.3f\n", w[0], w[1], w[2]);
}
"""


def test_relaxation_is_rounded_once_an_operation(tmp_path):
    src, exe = tmp_path / "r.cpp", tmp_path / "r"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off",
                    "-I", os.path.join(ROOT, "tests", "host_double"),
                    "-I", os.path.join(ROOT, "paper_1904_12553_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    worst = [float(v) for v in subprocess.run([str(exe)], check=True, capture_output=True,
                                              text=True).stdout.split()]
    assert worst[0] <= 4.0 and worst[1] <= 1.0 and worst[2] <= 3.0, worst
