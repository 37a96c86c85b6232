"""Bits of the Sobol estimator's points, on the CPU: the kernel's -ln and
barycentric coordinates (csrc/morea_sobol_point.h, compiled for the host with
either FP32 neighbour of 1 / d as the reciprocal) against the definition's
plain FP32 operations with divisions: -ln for every word, the reciprocal of
the sum for every mantissa, and the coordinates of four million points."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include "morea_sobol_point.h"

static uint32_t bits(float f) { return __builtin_bit_cast(uint32_t, f); }
static float from_bits(uint32_t u) { return __builtin_bit_cast(float, u); }

// The FP32 neighbour of 1 / d at or below it (side 0) or at or above (1); the
// nearest one for the mantissa of all ones.
static float reciprocal(float d, int side) {
  const float t = 1.0f / d;
  const double exact = 1.0 / static_cast<double>(d);
  if ((bits(d) & 0x7fffffu) == 0x7fffffu) return t;
  if (side == 0) return t > exact ? from_bits(bits(t) - 1) : t;
  return t < exact ? from_bits(bits(t) + 1) : t;
}

// The definition: r = m 2^e, s = (m - 1) / (m + 1), -ln r = -(e ln 2 + 2 s
// (1 + s^2/3 + ... + s^10/11)).
static float neg_log(uint32_t v) {
  const uint32_t u = bits(static_cast<float>(v) * 0x1p-24f);
  int e = static_cast<int>(u >> 23) - 127;
  float m = from_bits((u & 0x007fffffu) | 0x3f800000u);
  if (m > 0x1.6a09e6p+0f) {
    m = m * 0.5f;
    e = e + 1;
  }
  const float s = (m - 1.0f) / (m + 1.0f), s2 = s * s;
  float c = std::fmaf(s2, 0x1.745d18p-4f, 0x1.c71c72p-4f);
  c = std::fmaf(s2, c, 0x1.24924ap-3f);
  c = std::fmaf(s2, c, 0x1.99999ap-3f);
  c = std::fmaf(s2, c, 0x1.555556p-2f);
  c = std::fmaf(s2, c, 1.0f);
  return -std::fmaf(static_cast<float>(e), 0x1.62e430p-1f, (s + s) * c);
}

int main() {
  for (uint32_t v = 1; v < (1u << 24); v += 2)
    for (int side = 0; side < 2; side++) {
      const float h = morea::sobol::half_neg_log(v, [=](float d) { return reciprocal(d, side); });
      if (bits(h + h) != bits(neg_log(v))) return printf("-ln of word %u, side %d\n", v, side), 1;
    }
  for (uint32_t k = 0; k < (1u << 23); k++)
    for (int side = 0; side < 2; side++) {
      const float d = from_bits(0x3f800000u | k), r = reciprocal(d, side);
      if (std::fmaf(std::fmaf(-d, r, 1.0f), r, r) != 1.0f / d) return printf("reciprocal of %a, side %d\n", d, side), 1;
    }
  uint64_t z = 1;
  for (int i = 0; i < 4000000; i++) {
    uint32_t v[4];
    for (int j = 0; j < 4; j++) {
      z = z * 6364136223846793005ull + 1442695040888963407ull;
      const uint32_t w = static_cast<uint32_t>(z >> 40);
      // some near both ends of the range
      v[j] = (i % 16 == j ? w & 255u : (i % 16 == 4 + j ? 0xffff00u | (w & 255u) : w)) | 1u;
    }
    float l[3], e[4];
    morea::sobol::lambdas(v, l, [=](float d) { return reciprocal(d, i & 1); });
    for (int j = 0; j < 4; j++) e[j] = neg_log(v[j]);
    const float sum = ((e[0] + e[1]) + e[2]) + e[3];
    for (int j = 0; j < 3; j++)
      if (bits(l[j]) != bits(e[j + 1] / sum)) return printf("point %d: words %u %u %u %u\n", i, v[0], v[1], v[2], v[3]), 1;
  }
  return 0;
}
"""


def test_bits_of_logarithms_and_coordinates(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ is not installed")
    src, exe = tmp_path / "points.cpp", tmp_path / "points"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-D__device__=", "-D__forceinline__=inline",
                           "-I", os.path.join(ROOT, "paper_2303_04873_amd", "csrc"), "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout
