"""CPU test: the products that the kernels divide by, compiled for the host, against the division."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_02043_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include <random>
#include "fl_params.hpp"
int main() {
  std::mt19937_64 rng(1);
  auto check = [&](uint32_t d) {
    const fl::Divisor f = fl::Divisor::of(d);
    auto one = [&](int64_t n) {
      if (n < 0 || n > 0x7fffffffLL) return true;
      int q, r;
      f.split((int)n, q, r);
      if (q == n / d && r == n % d && f.div((int)n) == q) return true;
      std::printf("%lld / %u\n", (long long)n, d);
      return false;
    };
    const int64_t top = 0x7fffffffLL / d * d;
    for (int64_t n : {(int64_t)0, (int64_t)1, (int64_t)d - 1, (int64_t)d, (int64_t)d + 1, top - 1, top, top + 1, (int64_t)0x7fffffff})
      if (!one(n)) return false;
    for (int i = 0; i < 50; ++i)
      if (!one((int64_t)(rng() & 0x7fffffff))) return false;
    return true;
  };
  for (uint32_t d = 1; d < 5000; ++d)
    if (!check(d)) return 1;
  for (int k = 0; k < 31; ++k)
    for (int e = -1; e <= 1; ++e)
      if ((1LL << k) + e >= 1 && !check((uint32_t)((1LL << k) + e))) return 1;
  for (int i = 0; i < 20000; ++i)
    if (!check((uint32_t)(rng() % 0x7fffffff) + 1)) return 1;
  return fl::Divisor::of(0).d == 1 ? 0 : 1;
}
"""


def test_products_divide_exactly(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    src = tmp_path / "d.hip"
    src.write_text(SOURCE)
    exe = str(tmp_path / "d")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True, timeout=300)
    assert subprocess.run([exe], timeout=120).returncode == 0
