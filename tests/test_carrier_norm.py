"""The carrier matcher's reciprocal norm, its device code built for the CPU.

inv_norm corrects the hardware's estimates of 1 / sqrt(x) and 1 / x; its result
is within one unit in the last place of the IEEE square root's and division's,
and equal to it but for a few in ten million, whatever the estimates within an
ulp of the exact values are.  The function is taken from the kernel's source
text, with estimates an ulp low, rounded and an ulp high in place of the
instructions, over two octaves (the square root's) of the mantissas."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_31105_amd import build as B

MAIN = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
static int off_rsq, off_rcp;
static float ulps(double exact, int off) {
  float f = (float)exact;
  for (; off > 0; --off) f = nextafterf(f, INFINITY);
  for (; off < 0; ++off) f = nextafterf(f, 0.f);
  return f;
}
static float est_rsq(float x) { return ulps(1.0 / sqrt((double)x), off_rsq); }
static float est_rcp(float x) { return ulps(1.0 / (double)x, off_rcp); }
#define __builtin_amdgcn_rsqf est_rsq
#define __builtin_amdgcn_rcpf est_rcp
#define __device__
#define __forceinline__ inline
using std::fma;
%s
static float bits(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static uint32_t word(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
int main() {
  long n = 0, differ = 0, far = 0;
  const uint32_t bases[4] = {0x3f800000u, 0x40000000u, 0x0d000000u, 0x00800000u};
  for (uint32_t base : bases)
    for (uint32_t m = 0; m < (1u << 23); m += base >= 0x3f800000u ? 3 : 61)
      for (int r = -1; r <= 1; ++r)
        for (int c = -1; c <= 1; ++c) {
          off_rsq = r;
          off_rcp = c;
          const float x = bits(base + m), want = 1.f / sqrtf(x), got = inv_norm(x);
          const long d = (long)word(got) - (long)word(want);
          ++n;
          differ += d != 0;
          far += d > 1 || d < -1;
        }
  const bool ends = inv_norm(0.f) == 0.f && inv_norm(INFINITY) == 0.f;
  printf("%%ld %%ld %%ld %%d\n", n, differ, far, (int)ends);
}
"""


def test_inv_norm_against_ieee(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ missing")
    src = open(os.path.join(B.CSRC, "carrier.hip")).read()
    fn = re.search(r"^__device__ __forceinline__ float inv_norm\(float ss\) \{.*?^\}", src, re.S | re.M)
    (tmp_path / "norm.cpp").write_text(MAIN % fn.group(0))
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "norm.cpp", "-o",
                    "norm"], check=True, cwd=tmp_path)
    n, differ, far, ends = map(int, subprocess.run([str(tmp_path / "norm")], check=True,
                                                   capture_output=True, text=True).stdout.split())
    print(n, differ, far)
    assert n > 50_000_000 and ends and far == 0
    assert differ <= 1e-6 * n
