"""The branch-free GELU and tanh of the bf16 low-rank kernels (csrc/feature_maps.h), built for the host with
a correctly rounded reciprocal and the C library's exponential, against erfc and tanh in 64 bits."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_06712_amd", "csrc")

# Bounds in units of u = 2^-24 (half an fp32 ulp of 1):
#   GELU, x < 0: |x| tail. The tail is a product of t (2 roundings), P(t) (9 steps of Horner's scheme whose
#     terms are at most 1.6 times the sum: 12 u), two products, and exp (1 ulp = 2 u) of an argument that
#     carries the rounding of z twice and of z^2 once: 3 u z^2. The product with x adds one more, the fit
#     1.5e-8 up to z = 5: (20 + 3 z^2) u in all.
#   GELU, x >= 0: the same error of the tail (at most 1/2) against Phi >= 1/2, and two roundings.
#   tanh below 0.6: the fit, the rounding of x^2 and x^3 Q (at most 0.12 of x, 8 u of it) and the last: 3 u.
#   tanh beyond: 2 / (1 + e^2a) < 0.47, its exp and reciprocal (6 u, and 2 a u from the argument, exact) against
#     tanh >= 0.53, and the last rounding: 8 u.
PROGRAM = r"""
#include <math.h>
#include <stdio.h>
#define MAP_FN static inline
#define MAP_RCP(x) (1.0f / (x))
#define MAP_EXP(x) expf(x)
#include "feature_maps.h"
static int failed = 0;
static void check(const char* what, float x, double got, double want, double bound) {
  if (!(fabs(got - want) <= bound) && failed++ < 10)
    printf("%s(%.9g) = %.9g, want %.9g, bound %.3g\n", what, x, got, want, bound);
}
static void both(float x) {
  const double u = 1.0 / 16777216, d = x, z = fabs(d) * 0.70710678118654752440, tail = 0.5 * erfc(z);
  const double rel = (20 + 3 * z * z) * u + (z <= 5 ? 1.5e-8 : 1e-4);
  const double want = d < 0 ? d * tail : d * (1 - tail);
  check("gelu", x, rola::gelu_fast(x), want, d < 0 ? fabs(want) * rel + 1e-38 : d * (tail * rel + 2 * u));
  const double th = tanh(d);
  check("tanh", x, rola::tanh_fast(x), th, fabs(th) * (fabs(d) < 0.6 ? 3 * u + 3e-9 : 8 * u));
}
int main(void) {
  for (int i = -12000000; i <= 12000000; i += 7) both(i * 1e-6f);
  for (float x = 1e-38f; x < 1e-3f; x *= 1.5f) both(x), both(-x);   // towards zero: x / 2 and x
  for (int i = -2000; i <= 2000; ++i) {                              // around the crossover
    float x = 0.6f + i * 5.9604645e-8f;
    both(x), both(-x);
  }
  for (float x = 12; x < 1e30f; x *= 2) {                            // saturation
    check("gelu", x, rola::gelu_fast(x), x, 0), check("gelu", -x, rola::gelu_fast(-x), 0, 1e-29);
    check("tanh", x, rola::tanh_fast(x), 1, 0), check("tanh", -x, rola::tanh_fast(-x), -1, 0);
  }
  check("gelu", 0, rola::gelu_fast(0.f), 0, 0), check("tanh", 0, rola::tanh_fast(0.f), 0, 0);
  check("tanh", INFINITY, rola::tanh_fast(INFINITY), 1, 0), check("tanh", -INFINITY, rola::tanh_fast(-INFINITY), -1, 0);
  if (rola::gelu_fast(INFINITY) != INFINITY) ++failed;
  printf("%d failed\n", failed);
  return failed != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_feature_maps_against_64_bits(tmp_path):
    src, exe = tmp_path / "maps.cpp", str(tmp_path / "maps")
    src.write_text(PROGRAM)
    res = subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", f"-I{CSRC}", str(src), "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
