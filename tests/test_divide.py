"""Division by a multiplication and a shift, as the kernels have it, against the compiler's, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "divide.hpp"
#include <cstdio>
#include <initializer_list>
int main() {
  int64_t wrong = 0, n_checked = 0;
  auto check = [&](int32_t n, int32_t d) { n_checked++; if (n >= 0 && ellm::divide(n, ellm::divisor(d)) != n / d) wrong++; };
  auto around = [&](int32_t d) {
    for (int64_t q : {int64_t(0), int64_t(1), int64_t(2), int64_t(1000), int64_t(0x7fffffff) / d})
      for (int64_t n = q * d - 2; n <= q * d + 2; n++) if (n >= 0 && n <= 0x7fffffff) check((int32_t)n, d);
    check(0x7fffffff, d); check(0x7ffffffe, d);
  };
  for (int32_t d = 1; d < 70000; d++) around(d);
  for (int b = 1; b < 31; b++) for (int k = -2; k <= 2; k++) if ((1ll << b) + k >= 1) around((int32_t)((1ll << b) + k));
  around(0x7fffffff);
  for (int32_t n = 0; n < 20000; n++) for (int32_t d = 1; d < 700; d += 3) check(n, d);
  std::printf("%lld %lld\n", (long long)wrong, (long long)n_checked);
}
"""


def test_division_is_exact(tmp_path):
    """Every divisor up to 70000 and around the powers of two, around multiples of it up to the largest 31-bit number."""
    src, exe = tmp_path / "d.cpp", tmp_path / "d"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2506_15155_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    wrong, n = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert wrong == 0 and n > 1_000_000
