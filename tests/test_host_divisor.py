"""The kernels' division by a multiplication (Divisor) against the division, for divisors and
numbers at powers of two, around multiples of the divisor and at the ends of the range."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

SOURCE = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "prcr_internal.h"
int main() {
  const uint32_t top = 0x7FFFFFFFu;
  std::mt19937 rng(5);
  std::vector<uint32_t> ds;
  for (uint32_t d = 1; d <= 2000; ++d) ds.push_back(d);
  for (int s = 0; s < 31; ++s)
    for (int e = -2; e <= 2; ++e) ds.push_back(static_cast<uint32_t>((int64_t{1} << s) + e));
  for (int i = 0; i < 2000; ++i) ds.push_back(rng() >> (1 + rng() % 31));
  ds.push_back(top);
  ds.push_back(top - 1);
  long checked = 0;
  for (uint32_t d : ds) {
    if (d < 1 || d > top) continue;
    const prcr::Divisor by = prcr::Divisor::of(static_cast<int32_t>(d));
    auto check = [&](int64_t n) {
      if (n < 0 || n > top) return true;
      ++checked;
      return by.divide(static_cast<uint32_t>(n)) == static_cast<uint32_t>(n) / d;
    };
    bool ok = check(0) && check(1) && check(top) && check(top - 1);
    for (int i = 0; i < 300 && ok; ++i) {
      const int64_t m = static_cast<int64_t>(rng() % (top / d + 1)) * d;
      for (int64_t e = -1; e <= 1; ++e) ok = ok && check(m + e) && check((int64_t{1} << (i % 31)) + e);
    }
    const int64_t last = static_cast<int64_t>(top / d) * d;
    ok = ok && check(last) && check(last - 1);
    if (!ok) {
      std::printf("wrong for %u\n", d);
      return 1;
    }
  }
  std::printf("divisor: ok, %ld\n", checked);
  return 0;
}
"""


def test_division_by_multiplication(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "divisor.cpp", tmp_path / "divisor"
    src.write_text(SOURCE)
    built = subprocess.run([cxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                            "-D__HIP_PLATFORM_AMD__", f"-I{ROOT}/include",
                            f"-I{ROOT}/paper_2606_26631_amd/csrc", f"-I{ROCM}/include", str(src), "-o", str(exe)],
                           capture_output=True, text=True, timeout=300)
    assert built.returncode == 0, built.stderr[-3000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "divisor: ok" in run.stdout, run.stdout + run.stderr
