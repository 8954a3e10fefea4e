"""The sine and cosine sums behind the twiddles of lengths without a table (CPU).

eighth_sincos is compiled for the host and evaluated at every angle u / n of an
eighth turn of the transform lengths up to 4096.  Bound: 4.4e-16, two FP64 ulps of
values below one: the angle is rounded twice and the sums once per term, the last
terms well below an ulp.  The entries rounded to FP32 equal those of long double
sines and cosines."""

import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_09775_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include <vector>
#include "common.hpp"
int main() {
  std::vector<double> v;
  for (int n = 2; n <= 4096; ++n) {
    int m = n;
    for (int p : {2, 3, 5}) while (m % p == 0) m /= p;
    if (m != 1) continue;
    const double inv = 1.0 / (double)n;
    for (int u = 0; u <= n; ++u) {
      double s, c;
      wo::eighth_sincos((double)u * inv, &s, &c);
      v.insert(v.end(), {(double)u, (double)n, s, c});
    }
  }
  return fwrite(v.data(), sizeof(double), v.size(), stdout) == v.size() ? 0 : 1;
}
"""


def test_sums_are_fp64(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "sums.hip", tmp_path / "sums"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "--cuda-host-only", "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC, "-o", str(exe), str(src)],
                   check=True, capture_output=True)
    v = np.frombuffer(subprocess.run([str(exe)], check=True, capture_output=True).stdout).reshape(-1, 4)
    a = np.longdouble("0.785398163397448309615660845819875721") * (v[:, 0].astype(np.longdouble) / v[:, 1])
    s, c = np.sin(a), np.cos(a)
    err = max(float(np.max(np.abs(v[:, 2] - s))), float(np.max(np.abs(v[:, 3] - c))))
    assert err <= 4.4e-16
    assert np.array_equal(v[:, 2].astype(np.float32), s.astype(np.float32))
    assert np.array_equal(v[:, 3].astype(np.float32), c.astype(np.float32))
