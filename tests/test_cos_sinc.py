"""cos(A) and sin(A)/A of the FP32 vector-potential step (csrc/dirac_cos_sinc.h), the same
source compiled for the host, against long double over its range up to kCosSincMax."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1107_4650_amd", "csrc")

SOURCE = r"""
#include <cmath>
#include <cstdio>
#define __host__
#define __device__
#define __forceinline__ inline
#include "dirac_cos_sinc.h"
using dirac::kCosSincMax;
int main() {
  double ec = 0, es = 0;
  auto at = [&](double z) {
    double c, s;
    dirac::cos_sinc(z, &c, &s);
    const long double A = sqrtl((long double)z);
    const long double sinc = A > 1e-6L ? sinl(A) / A : 1.0L - (long double)z / 6.0L;
    const long double dc = fabsl(c - cosl(A)), ds = fabsl((s - sinc) * (A > 1.0L ? A : 1.0L));
    if (dc > ec) ec = dc;
    if (ds > es) es = ds;
  };
  const int n = 2000000;
  for (int i = 0; i <= n; ++i) at(kCosSincMax * (i / (double)n));
  for (int i = 0; i < 200000; ++i) at(kCosSincMax * (1.0 - i * 1e-9));  // up to the limit
  for (int i = 0; i < 200000; ++i) at(84.10 + (i - 100000) * 1e-6);     // around the worst angle
  for (double z = 1e-300; z < 1.0; z *= 10.0) at(z);
  at(0.0);
  std::printf("%.6e %.6e\n", ec, es);
}
"""


def test_series_errors_over_the_whole_range(tmp_path):
    src = tmp_path / "cos_sinc.cpp"
    src.write_text(SOURCE)
    exe = tmp_path / "cos_sinc"
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-Wno-unknown-pragmas",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True)
    cos_err, sin_err = map(float, subprocess.run([str(exe)], capture_output=True, text=True,
                                                 check=True).stdout.split())
    # the bound beside the source
    assert cos_err < 7e-15 and sin_err < 7e-15, (cos_err, sin_err)
    assert cos_err > 3e-15  # the worst angles were met
