"""Device arithmetic that has a header of its own, compiled for the CPU: the division by a runtime constant that the
kernels decode pixel indices with (csrc/fastdiv.h), GELU's derivative (csrc/gelu.h), the compensated sum
(csrc/compensated.h)."""
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


def run_on_cpu(tmp_path, program):
    src, exe = tmp_path / "program.cpp", tmp_path / "program"
    src.write_text(program)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                           "-D__builtin_amdgcn_rcpf(x)=(1.0f/(x))", "-D__builtin_amdgcn_exp2f=exp2f", "-I", CSRC, str(src), "-o", str(exe)])
    return subprocess.run([str(exe)], capture_output=True, text=True)


def test_division_by_a_constant_is_exact_over_the_whole_index_range(tmp_path):
    """Quotient and remainder on both sides of the ends of rows up to the largest 32-bit index, for every width up to
    4200 and larger ones: one too large at a row's end is a pixel in column -1 of the next row."""
    run = run_on_cpu(tmp_path, PROGRAM)
    assert run.returncode == 0, run.stdout


GELU_PROGRAM = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
using std::fmaf;
#include "gelu.h"
int main() {
  double worst[2] = {0, 0}, square[2] = {0, 0};
  int bad = 0;
  for (uint32_t i = 0; i < 65536; ++i) {
    const uint32_t bits = i << 16;
    float u;
    memcpy(&u, &bits, 4);
    if (!std::isfinite(u)) continue;
    const double x = u, want = 0.5 * erfc(-x / std::sqrt(2.0)) + x * std::exp(-0.5 * x * x) / std::sqrt(2 * M_PI);
    const float got[2] = {gelu_grad_f(u), 0.5f * (1.0f + erff(u * 0.70710678118654752f)) + u * expf(-0.5f * u * u) * 0.39894228040143268f};
    for (int f = 0; f < 2; ++f) {
      const double e = std::fabs(got[f] - want);
      if (!(e < 1e-3)) ++bad;
      if (e > worst[f]) worst[f] = e;
      square[f] += e * e;
    }
  }
  printf("largest %g against %g, rms %g against %g, %d bad\n", worst[0], worst[1], std::sqrt(square[0] / 65536), std::sqrt(square[1] / 65536), bad);
  return bad || worst[0] > worst[1] || square[0] > square[1];
}
"""


def test_gelu_derivative_is_as_exact_as_the_textbook_form_in_fp32(tmp_path):
    """Over every finite bf16 argument, against fp64: largest and rms error no larger than those of the same formula
    with erff and expf."""
    run = run_on_cpu(tmp_path, GELU_PROGRAM)
    assert run.returncode == 0, run.stdout


SUM_PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <vector>
#include "compensated.h"
float sum_of(const std::vector<float>& v) {
  float s = 0.f, lost = 0.f;
  for (float x : v) compensated_add(x, s, lost);
  return s;
}
int main() {
  const float inf = INFINITY;
  int bad = 0;
  auto expect = [&](bool ok, const char* what) { if (!ok) { printf("%s\n", what); ++bad; } };
  expect(sum_of({1, inf, 2, -3, 4}) == inf, "an infinity among finite terms");
  expect(sum_of({inf}) == inf && sum_of({inf, inf, 1}) == inf, "infinities of one sign");
  expect(sum_of({5, -inf, 2, 3}) == -inf, "a negative infinity");
  expect(std::isnan(sum_of({inf, 1, -inf, 2})), "infinities of both signs");
  expect(std::isnan(sum_of({1, NAN, 2})), "a NaN");
  expect(sum_of({3e38f, 3e38f, 1, 2}) == inf && sum_of({-3e38f, -3e38f, 1}) == -inf, "a sum past the largest number");
  std::vector<float> v;
  double want = 0;
  unsigned r = 1;
  for (int i = 0; i < 100000; ++i) {
    r = r * 1664525u + 1013904223u;
    v.push_back((float)(r >> 8) * 0x1p-24f + 0.5f);
    want += v.back();
  }
  expect(std::fabs(sum_of(v) - want) <= want * 0x1p-23, "1e5 terms: two roundings");
  return bad;
}
"""


def test_compensated_sum_keeps_what_it_rounds_off_and_passes_infinities_on(tmp_path):
    run = run_on_cpu(tmp_path, SUM_PROGRAM)
    assert run.returncode == 0, run.stdout + run.stderr
