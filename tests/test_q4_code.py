"""Host-side check (no GPU needed) of the packers' quotient: q4_code replaces the divide by a
multiplication with the reciprocal and one correction step.  The kernels' own function, compiled
for the host, against the correctly rounded fp32 quotient over every pair of fp16 significands
whose quotient can matter, with the reciprocal exact and one unit off either way (what the
hardware's approximation guarantees), at scales from the smallest subnormal to the largest."""
import ctypes
import os
import subprocess

import pytest

from paper_2504_08378_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCE = """
#include <cmath>
#include <cstring>
#include "q4_code.h"
static unsigned divided(float w, float s) {
  const float q = std::rint(w / s);  // ties to even
  return (unsigned)((int)std::fmin(7.f, std::fmax(-7.f, q)) + 8);
}
// pairs of significands (1024 .. 2047) at scale 2^e and quotients of 2^-3 to 2^4; returns the
// mismatches and counts what was compared
extern "C" long long mismatches(int e, long long* compared) {
  long long bad = 0, n = 0;
  for (int a = 1024; a < 2048; ++a) {
    const float s = std::ldexp((float)a, e - 10);
    const float inv = 1.0f / s;
    float near[3] = {std::nextafterf(inv, 0.f), inv, std::nextafterf(inv, INFINITY)};
    for (int b = 1024; b < 2048; ++b)
      for (int d = -3; d <= 3; ++d) {
        const float w = std::ldexp((float)b, e - 10 + d);
        if (w > 65504.f) continue;
        const unsigned up = divided(w, s), down = divided(-w, s);
        for (int r = 0; r < 3; ++r) {
          bad += q4_code(w, s, near[r]) != up;
          bad += q4_code(-w, s, near[r]) != down;
          n += 2;
        }
      }
  }
  *compared = n;
  return bad;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("q4")
    src, so = str(d / "q4.hip"), str(d / "q4.so")
    open(src, "w").write(SOURCE)
    subprocess.run([HIPCC, *build.HIPCC_FLAGS, "-ffp-contract=off", "-I", build.CSRC, "-shared", src, "-o", so], check=True,
                   stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    so = ctypes.CDLL(so)
    so.mismatches.restype = ctypes.c_longlong
    return so


# scales of 2^e: subnormal halves (their significands are some of these), ordinary ones, the largest
@pytest.mark.parametrize("e", [-24, -15, -6, 0, 9, 13])
def test_code_is_that_of_the_divide(lib, e):
    n = ctypes.c_longlong()
    assert lib.mismatches(e, ctypes.byref(n)) == 0
    assert n.value > 2e7
