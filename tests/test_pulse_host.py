"""The pulse's integral over a step (csrc/dirac_pulse.h, host code): a step index beyond
32 bits names the step it says, counted from the pass or from the run."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1107_4650_amd", "csrc")

SOURCE = r"""
#include "dirac_pulse.h"
#include <cstdio>
int main() {
  const int64_t far = (int64_t(1) << 32) + 77;
  const dirac::PulseK from_run{3.0, 0.2, 2.0, 1e10, 1.0, 0.5, 0.01, 0};
  dirac::PulseK from_pass = from_run;
  from_pass.n0 = far;
  std::printf("%a %a %a\n", dirac::pulse_step_integral(from_run, far),
              dirac::pulse_step_integral(from_pass, 0), dirac::pulse_step_integral(from_run, 77));
}
"""


def test_step_index_beyond_32_bits(tmp_path):
    src = tmp_path / "pulse.cpp"
    src.write_text(SOURCE)
    exe = tmp_path / "pulse"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wno-narrowing", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True)
    a, b, near = subprocess.run([str(exe)], capture_output=True, text=True,
                                check=True).stdout.split()
    assert a == b and a != near
