"""The division by a runtime constant that the kernels decode pixel indices with (csrc/fastdiv.h), on the CPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_23186_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "fastdiv.h"
int main() {
  const long long top = 2147483647LL;
  long long bad = 0;
  auto check = [&](const FastDiv& f, long long x) {
    if (x < 0 || x > top) return;
    int q, r;
    f.divmod((int)x, &q, &r);
    if (q != x / f.d || r != x % f.d) {
      if (bad++ < 5) printf("%lld / %u: %d rest %d\n", x, f.d, q, r);
    }
  };
  for (int step = 0; step < 2; ++step)
    for (unsigned d = 1; d < 2147483648u; d = step ? d * 2 + 1 : d + (d < 4200 ? 1 : d / 7 + 1)) {
      FastDiv f;
      f.init(d);
      const long long rows = top / d, every = rows / 4000 + 1;      // both sides of the ends of rows, the last ones among them
      for (long long k = 0; k <= rows; k += every)
        for (long long x = k * d - 1; x <= k * d + 1; ++x) check(f, x);
      for (long long k = rows > 50 ? rows - 50 : 0; k <= rows; ++k)
        for (long long x = k * d - 1; x <= k * d + 1; ++x) check(f, x);
      check(f, top);
    }
  printf("%lld wrong\n", bad);
  return bad != 0;
}
"""


def test_division_by_a_constant_is_exact_over_the_whole_index_range(tmp_path):
    """Quotient and remainder on both sides of the ends of rows up to the largest 32-bit index, for every width up to
    4200 and larger ones: one too large at a row's end is a pixel in column -1 of the next row."""
    src, exe = tmp_path / "fastdiv.cpp", tmp_path / "fastdiv"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", CSRC, str(src),
                           "-o", str(exe)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
