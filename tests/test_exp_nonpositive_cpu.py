"""The exponential of the softmax statistics (csrc/exp_nonpositive.h), compiled for the host with an exact 2^p."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2602_06036_amd", "csrc")

DRIVER = r"""
#include <math.h>
#include <stdio.h>
#include <string.h>
#include "exp_nonpositive.h"
static float run(float d) { return exp_nonpositive(d, [](float p) { return (float)exp2((double)p); }); }
int main() {
  double worst = 0, at = 0;
  for (unsigned u = 0x80000000u; ; u += 97) {   // every 97th float from -0 to -87
    float d;
    memcpy(&d, &u, 4);
    if (!(d >= -87.f)) break;
    const double want = exp((double)d), err = fabs((double)run(d) - want) / want * 16777216.0;
    if (err > worst) { worst = err; at = d; }
  }
  printf("%.4f %.6f %g %g %g %d %g\n", worst, at, run(0.f), run(-INFINITY), run(-88.f), isnan(run(NAN)), run(-87.f) / exp(-87.0));
}
"""


def test_relative_error_down_to_the_smallest_normal_numbers(tmp_path):
    """At most 2^-23 relative: half an ulp each of 2^p and of the last operation, the rest second order.  Without the product's rounding put back it would be 33 times
    that at the far end; the instruction's own error (an ulp) comes on top of it on the GPU."""
    (tmp_path / "e.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC, str(tmp_path / "e.cpp"), "-o", str(tmp_path / "e")], check=True)
    worst, at, zero, inf, below, nan, last = subprocess.run([str(tmp_path / "e")], capture_output=True, text=True, check=True).stdout.split()
    assert float(worst) <= 2.0, (worst, at)
    assert (float(zero), float(inf), float(below), int(nan)) == (1.0, 0.0, 0.0, 1)
    assert abs(float(last) - 1.0) < 1e-6
