"""The arithmetic of light nodes (csrc/device.h), run on the CPU: the quotient by a
tabled reciprocal against IEEE division, and the bins at the ends of their range with
signed overflow trapped."""
import os
import subprocess

from tests._native import PKG, ROCM

PROGRAM = r"""
#include <cstdio>
#include "device.h"
int main() {
  // squares of sums of up to 511 responses of at most 2^22, small and large ones, and
  // squares next to multiples of b: the quotient is IEEE's
  uint64_t x = 88172645463325252ull, bad = 0, n = 0;
  auto check = [&](double a, int b) {
    if (aiwc::div_recip(a, (double)b, 1.0 / (double)b) != a / (double)b) ++bad;
    ++n;
  };
  for (int b = 1; b < 512; ++b) {
    for (int i = 0; i < 60000; ++i) {
      x ^= x << 13; x ^= x >> 7; x ^= x << 17;
      const double s = (double)(int64_t)(x >> (33 + i % 30));
      check(s * s, b);
      // any double of the range, and the neighbours of b times a double
      const double a = (double)(x >> 2);
      check(a, b);
      const double m = (double)(x >> 11) * (double)b;
      check(m, b);
      check(__builtin_nextafter(m, 0.0), b);
      check(__builtin_nextafter(m, 1e300), b);
    }
    check(0.0, b);
    check(1.0, b);
  }
  check(270392545247081.0, 123);
  if (aiwc::div_recip(0.0, 0.0, 0.0) != 0.0) ++bad;
  // bins: every weight at the extreme responses, alone and summed to a weight of 511
  uint64_t wrong = 0;
  for (int64_t y : {-(int64_t)(1 << 22), (int64_t)-1, (int64_t)0, (int64_t)77, (int64_t)(1 << 22)})
    for (uint32_t w = 0; w < 512; ++w) {
      const uint64_t v = aiwc::light_word(w, w * y);
      if (v >> 32 != w || aiwc::light_sum(w, (uint32_t)v) != w * y) ++wrong;
      const uint64_t t = v + aiwc::light_word(511 - w, (int64_t)(511 - w) * y);
      if (t >> 32 != 511 || aiwc::light_sum(511, (uint32_t)t) != 511 * y) ++wrong;
    }
  std::printf("%llu %llu %d\n", (unsigned long long)bad, (unsigned long long)wrong, n > 1000000);
}
"""


def test_light_arithmetic(tmp_path):
    src, exe = tmp_path / "light.hip", tmp_path / "light"
    src.write_text(PROGRAM)
    # host code only; -ffp-contract=off as in the library
    subprocess.run([f"{ROCM}/bin/hipcc", "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-ffp-contract=off",
                    "-Xarch_host", "-fsanitize=signed-integer-overflow", "-Xarch_host",
                    "-fsanitize-trap=signed-integer-overflow", f"-I{PKG}/csrc", str(src), "-o", str(exe)],
                   check=True, capture_output=True, env=dict(os.environ))
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120).stdout
    assert out.split() == ["0", "0", "1"]
