"""CPU test of the quotients by a divisor's inverse that launches of few rows take their work items from (launch_rules.hpp):
every divisor below 2^15 at the multiples and one below them nearest both ends of the range, and small ones at every number."""
import os
import shutil
import subprocess

import pytest

SOURCE = """
#include <cstdio>
#include "launch_rules.hpp"
int main() {
  const int top = 1 << 15;
  long wrong = 0;
  for (int d = 1; d < top; ++d) {
    const uint32_t inv = astro::inverse_of(d);
    auto check = [&](int n) { if (n >= 0 && n < top && astro::quotient(n, inv) != n / d) ++wrong; };
    if (d < 64) for (int n = 0; n < top; ++n) check(n);
    const int last = (top - 1) / d * d;
    for (int n : {0, d - 1, d, d + 1, 2 * d - 1, 2 * d, last - 1, last, last + 1, top - 1}) check(n);
  }
  std::printf("%ld", wrong);
}
"""


def test_quotients(repo_root, tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "q.cpp", tmp_path / "q"
    src.write_text(SOURCE)
    include = os.path.join(repo_root, "paper_2603_17051_amd", "csrc")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-I", include, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout == "0"
