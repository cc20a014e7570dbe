"""The rotation's sine and cosine (csrc/frontend_core.h), compiled for the host,
against extended precision: the front end's own bounds are BF16 steps and see
nothing of them."""
import os
import shutil
import subprocess

import pytest

from paper_2606_22874_amd import build

SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <cstdint>
#include "frontend_core.h"
static uint64_t state = 88172645463325252ull;
static double uniform() {
  state ^= state << 13; state ^= state >> 7; state ^= state << 17;
  return (double)(state >> 11) * 0x1p-53;
}
int main() {
  // angles up to 2^40, over their logarithm, and around multiples of pi/4
  double worst_s = 0, worst_c = 0;
  for (int i = 0; i < 2000000; ++i) {
    int pos = (int)std::exp2(31 * uniform()) - 1;
    double freq = std::exp2(-20 + 29 * uniform());
    if (i % 4 == 0) {
      pos = i % 8 ? 1 : -1;
      freq = std::floor(4096 * uniform()) * 0.78539816339744831 * (1 + 1e-9 * (uniform() - 0.5));
    }
    float s, c;
    spot::rope_sincos(pos, freq, s, c);
    const long double t = (long double)((double)pos * freq);
    worst_s = std::fmax(worst_s, (double)fabsl(s - sinl(t)));
    worst_c = std::fmax(worst_c, (double)fabsl(c - cosl(t)));
  }
  // any angle the entry points accept (frequencies up to 2^149)
  int bad = 0;
  for (int i = 0; i < 200000; ++i) {
    float s, c;
    spot::rope_sincos((int)(2147483647.0 * (2 * uniform() - 1)), std::exp2(150 * uniform()), s, c);
    bad += !(std::fabs(s) <= 1.0f && std::fabs(c) <= 1.0f);
  }
  float s0, c0;
  spot::rope_sincos(0, 123.0, s0, c0);
  std::printf("%.3e %.3e %d %g %g\n", worst_s, worst_c, bad, s0, c0);
}
"""


def test_sine_and_cosine(tmp_path):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("needs hipcc")
    src, exe = tmp_path / "t.hip", tmp_path / "t"
    src.write_text(SOURCE)
    subprocess.run([build.hipcc(), "--cuda-host-only", "-O2", "-std=c++17", "-I", build.CSRC, "-I",
                    build.INCLUDE, str(src), "-o", str(exe)], check=True, capture_output=True,
                   text=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    print(out)
    assert float(out[0]) <= 1e-7 and float(out[1]) <= 1e-7, out
    assert out[2:] == ["0", "0", "1"], out
