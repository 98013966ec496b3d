"""The quantizer's quotient without a division (Quant::code of pack_kernels.hip): a first quotient from the approximate
reciprocal of the scale and one exact remainder, the scheme of P. W. Markstein, "Computation of elementary functions on the
IBM RISC System/6000 processor" (1990).  His theorem asks for a correctly rounded reciprocal; the hardware's is within one
unit in the last place, so the result is compared with the IEEE quotient here: for every positive fp16 scale, with the
correctly rounded reciprocal and both its neighbours, at the numerators where a code changes (half-integers times the scale,
two numbers on either side) and at differences of bf16 numbers.  The scale's own quotient, a group's range by the largest code,
goes the same way with the correctly rounded reciprocal: all numerators of two binades, and the sign of a zero."""
import shutil
import subprocess

import pytest

PROGRAM = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <initializer_list>
static float from_bits(uint32_t u) { float f; std::memcpy(&f, &u, 4); return f; }
static float half_value(uint32_t h) {                 // positive, finite
  const int e = h >> 10, m = h & 1023;
  return e == 0 ? std::ldexp(float(m), -24) : std::ldexp(float(1024 + m), e - 25);
}
static long n = 0, bad = 0;
static void check(float d, float s, float y) {
  const float q0 = d * y, q = std::fma(std::fma(-q0, s, d), y, q0), want = d / s;
  ++n;
  if (std::memcmp(&q, &want, 4) != 0 && bad++ < 5) std::printf("d %a s %a y %a: %a instead of %a\n", d, s, y, q, want);
}
int main() {
  uint64_t rng = 88172645463325252ull;
  const auto next = [&] { rng ^= rng << 13; rng ^= rng >> 7; rng ^= rng << 17; return uint32_t(rng >> 32); };
  for (uint32_t h = 1; h < 0x7C00; ++h) {
    const float s = half_value(h), y1 = 1.0f / s;
    const float ys[3] = {y1, std::nextafter(y1, 0.0f), std::nextafter(y1, INFINITY)};
    for (const float y : ys) {
      for (int k = 0; k < 256; ++k) {
        float d = (k + 0.5f) * s;
        d = std::nextafter(std::nextafter(d, 0.0f), 0.0f);
        for (int i = 0; i < 5; ++i, d = std::nextafter(d, INFINITY)) check(d, s, y);
      }
      for (int k = 0; k < 64; ++k) {                  // x - m of bf16 numbers, up to the largest code and a half
        const float m = from_bits(next() & 0xBFFF0000u) * s, x = m + from_bits((0x3F000000u + (next() % 0x04800000u)) & 0xFFFF0000u) * s;
        const float d = from_bits([](float f) { uint32_t u; std::memcpy(&u, &f, 4); return u & 0xFFFF0000u; }(x)) - m;
        if (d >= 0.0f && d <= 256.0f * s) check(d, s, y);
      }
    }
  }
  for (const float Q : {3.0f, 15.0f, 255.0f}) {
    const float inv = 1.0f / Q;
    for (uint32_t u = 0x3F800000u; u < 0x40800000u; ++u) check(from_bits(u), Q, inv);
    for (const float zero : {0.0f, -0.0f}) {
      const float q0 = zero * inv, q = std::copysign(std::fma(std::fma(-q0, Q, zero), inv, q0), zero), want = zero / Q;
      bad += std::memcmp(&q, &want, 4) != 0;
    }
  }
  std::printf("%ld quotients, %ld differ\n", n, bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_quotient_from_reciprocal_and_remainder_is_the_ieee_quotient(tmp_path):
    (tmp_path / "quotient.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-march=native", "-ffp-contract=off", "-o", "quotient", "quotient.cpp"],
                   cwd=tmp_path, check=True)
    p = subprocess.run([tmp_path / "quotient"], capture_output=True, text=True)
    print(p.stdout)
    assert p.returncode == 0, p.stdout


def test_window_row_by_a_product_is_the_remainder():
    """limit_of in weights_kernels.hip: row % s_obs from row * (65536 / s_obs + 1) / 65536, for every window length."""
    for s in range(1, 65):
        for row in range(768):
            assert row - (row * (65536 // s + 1) >> 16) * s == row % s
