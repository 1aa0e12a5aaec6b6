"""The product-and-shift division of csrc/fastdiv.h against the integer division, for every divisor up to
4096 and a spread of larger ones, at multiples of the divisor and their neighbours over the whole range
of indices (0 .. 2^31 - 1)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include "fastdiv.h"
#include <cstdio>
int main() {
  long bad = 0;
  const long top = 0x7fffffffL;
  for (long d = 1; d <= top; d = d < 4096 ? d + 1 : d + d / 3) {
    const whmc::FastDiv f = whmc::fast_div((int)d);
    for (long k = 0; k <= 64; ++k) {
      const long q = top / d * k / 64;
      for (long n = q * d - 1; n <= q * d + 1; ++n)
        if (n >= 0 && n <= top && f.div((int)n) != n / d) ++bad;
    }
    if (f.div((int)top) != top / d) ++bad;
  }
  std::printf("%ld\n", bad);
  return bad != 0;
}
"""


def test_fast_division_is_exact(tmp_path):
    src = tmp_path / "fd.cpp"
    src.write_text(SRC)
    exe = str(tmp_path / "fd")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1805_03560_amd", "csrc"), str(src),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "0"
