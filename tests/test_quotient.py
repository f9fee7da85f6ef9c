"""The logarithm of the Gaussian draws, on the host, for every reciprocal estimate within 8 ulp: its
quotient is the IEEE one for every mantissa but one, and the Box-Muller radius is the one that
the IEEE quotient gives for every u, so the draws do not depend on how the estimate is rounded."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "tmz_math.h"
static float number(uint32_t b) { return __builtin_bit_cast(float, b); }
static uint32_t nearest_rcp(float d) { return __builtin_bit_cast(uint32_t, (float)(1.0 / (double)d)); }
static float radius(float ln) { return std::sqrt(-2.0f * ln); }
int main() {
  long long bad = 0, one = 0, draws = 0;
  for (uint32_t i = 0; i < (1u << 23); ++i) {
    const float m = number((i | 0x3F800000u) - (i > 0x3504F3u ? 0x00800000u : 0u));
    const float n = m - 1.0f, d = m + 1.0f, want = n / d;
    const uint32_t r = nearest_rcp(d);
    bad += tmz::quotient_from_rcp(n, d, number(r)) != want;
    for (int e = -8; e <= 8; ++e)
      if (tmz::quotient_from_rcp(n, d, number(r + e)) != want) ++(m == 1.0f - 0x1p-23f ? one : bad);
  }
  for (uint32_t k : {0xFFFFFEu, 0x7FFFFFu}) {            // the u of 24 bits with that mantissa
    const float u = (float)k * 0x1p-24f;
    const float want = radius(tmz::ln_unit_with(u, [](float n, float d) { return n / d; }));
    for (int e = -8; e <= 8; ++e)
      draws += radius(tmz::ln_unit_with(u, [e](float n, float d) {
                 return tmz::quotient_from_rcp(n, d, number(nearest_rcp(d) + e));
               })) != want;
  }
  std::printf("quotients %lld, of the one mantissa %lld of 16, radii %lld\n", bad, one, draws);
  return bad != 0 || one == 0 || draws != 0;
}
"""


def test_draws_do_not_depend_on_the_reciprocal_estimate(tmp_path):
    src = tmp_path / "quotient.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "quotient")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_2609_33548_amd", "csrc"), str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
